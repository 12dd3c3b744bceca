"""Orders that run a whole sweep in one launch (one workgroup per 64
configurations, barriers between levels) against the level kernels, which the
same batch takes when the reverse sweep is told to use two segments: the same
sums bit for bit (heads and flavours are added in the same order) and the same
gradients up to the order of their accumulation, bounded by the same sweep over
absolute values.  Group edges (1, 64, 65 configurations), shifts, several
flavours, and more flavours than fit LDS."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("nconf", [1, 64, 65])
@pytest.mark.parametrize("nflav,variant,stubs,mask_only", [(3, 0, True, False), (2, 1, False, True), (3, 1, True, False),
                                                           (9, 1, False, False)])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6])
def test_one_launch_against_levels(n, nflav, variant, stubs, mask_only, nconf):
    import torch
    from paper_2507_12349_amd import _binding as B
    announce("one launch against levels: n=%d nflav=%d variant=%d stubs=%s mask_only=%s nconf=%d"
             % (n, nflav, variant, stubs, mask_only, nconf))
    rng = np.random.default_rng(1000 * n + 10 * nflav + nconf)
    nmat = nflav if variant else 1
    dev = torch.device("cuda:0")
    G = torch.as_tensor(rng.normal(size=nconf * nmat * n * n) * 0.4, device=dev)
    st = torch.as_tensor(rng.normal(size=(nconf, nmat)) * 0.3, device=dev) if stubs else None
    ob = torch.as_tensor(rng.normal(size=nconf), device=dev)

    def sweep(G, st, w, ob, segments):
        b = B.Batch(np.full(nconf, n, dtype=np.int32), nflav, variant, stubs=stubs, mask_only=mask_only)
        b.set_adjoint_segments(segments)
        S, S2 = (torch.full((nconf,), float("nan"), dtype=torch.float64, device=dev) for _ in range(2))
        Gb, sb = torch.full_like(G, float("nan")), None if st is None else torch.full_like(st, float("nan"))
        b.forward(G, None, st, w, S)
        b.adjoint(G, None, st, w, ob, S2, Gb, sb)
        torch.cuda.synchronize()
        b.close()
        return [None if x is None else x.cpu().numpy() for x in (S, S2, Gb, sb)]

    one = sweep(G, st, -1.0, ob, 1)
    lev = sweep(G, st, -1.0, ob, 2)
    assert np.array_equal(one[0], one[1]) and np.array_equal(one[0], lev[1])
    if mask_only:   # the clows cancel only for w = -1: a bound from the entries' size
        assert np.allclose(one[2], lev[2], rtol=0, atol=1e-12 * np.abs(lev[2]).max())
        return
    ref = sweep(G.abs(), None if st is None else -st.abs(), 1.0, ob.abs(), 1)
    tol = 2 * 8 * n * (n + 2) * EPS
    assert np.all(np.abs(one[2] - lev[2]) <= tol * np.abs(ref[2]) + 1e-300)
    if stubs:
        assert np.all(np.abs(one[3] - lev[3]) <= tol * np.abs(ref[3]) + 1e-300)
