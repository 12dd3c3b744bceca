"""Two-segment gradients split at a level whose special masks (vertex 0 visited
twice, no other once) open the cycle of the last head: the memory that halves of
about equal size need, the sums of the sweep that stores every level, and with
reproducible gradients the same bits."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _run(G, st, ob, n, nflav, variant, mask, det, segments, w=-1.0, limit=0):
    import torch
    from paper_2507_12349_amd import _binding as B
    nconf = ob.numel()
    B.set_workspace_limit(limit)
    b = B.Batch(np.full(nconf, n, dtype=np.int32), nflav, variant, stubs=st is not None, mask_only=mask,
                deterministic=det)
    B.set_workspace_limit(0)
    b.set_adjoint_segments(segments)
    S = torch.full((nconf,), float("nan"), dtype=torch.float64, device=G.device)
    Gb, sb = torch.full_like(G, float("nan")), None if st is None else torch.full_like(st, float("nan"))
    b.adjoint(G, None, st, w, ob, S, Gb, sb)
    torch.cuda.synchronize()
    plan = b.adjoint_plan(n)
    b.close()
    return [x.cpu().numpy() for x in (S, Gb, sb) if x is not None], plan


# per group, two segments against every level stored, with the best split of any level
RATIO = {3: 0.78, 6: 0.73, 7: 0.70, 8: 0.68, 9: 0.66, 10: 0.65, 12: 0.63}


@pytest.mark.parametrize("n,nflav,variant,stubs,mask,nconf", [
    (3, 2, 0, True, False, 70), (6, 3, 1, True, False, 130), (6, 2, 1, False, True, 64), (7, 2, 0, True, False, 65),
    (8, 2, 0, True, False, 200), (8, 3, 1, True, False, 65), (9, 2, 0, False, False, 64), (10, 2, 1, True, False, 66),
    (10, 2, 1, False, True, 3), (12, 2, 0, True, False, 5)])
def test_split_at_any_level(n, nflav, variant, stubs, mask, nconf):
    import torch
    announce("two segments: n=%d nflav=%d variant=%d stubs=%s mask_only=%s nconf=%d" % (n, nflav, variant, stubs, mask, nconf))
    rng = np.random.default_rng(300 + n)
    dev = torch.device("cuda:0")
    nmat = nflav if variant else 1
    G = torch.as_tensor(rng.normal(size=nconf * nmat * n * n) * 0.35, device=dev)
    st = torch.as_tensor(rng.normal(size=(nconf, nmat)) * 0.3, device=dev) if stubs else None
    ob = torch.as_tensor(rng.normal(size=nconf), device=dev)
    one, p1 = _run(G, st, ob, n, nflav, variant, mask, True, 1)
    two, p2 = _run(G, st, ob, n, nflav, variant, mask, True, 2)
    print("  split at level %d, %.3f of the memory" % (p2["split_level"], p2["bytes_per_group"] / p1["bytes_per_group"]),
          flush=True)
    for x, y in zip(one, two):
        assert np.array_equal(x, y)
    for limit in (0, 1):   # the default reverse; one group per chunk
        atom, _ = _run(G, st, ob, n, nflav, variant, mask, False, 2, limit=limit)
        assert np.array_equal(atom[0], one[0])
        if mask:   # the clows cancel only for w = -1: a bound from the entries' size
            assert np.allclose(atom[1], one[1], rtol=0, atol=1e-12 * np.abs(one[1]).max())
            continue
        ref, _ = _run(G.abs(), None if st is None else -st.abs(), ob.abs(), n, nflav, variant, False, False, 1, 1.0)
        for x, y, z in zip(atom[1:], one[1:], ref[1:]):
            assert np.all(np.abs(x - y) <= 2 * 8 * n * (n + 2) * EPS * np.abs(z) + 1e-300)
    assert p2["bytes_per_group"] <= RATIO[n] * p1["bytes_per_group"]
