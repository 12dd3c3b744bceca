"""Order 5 with several flavours: small batches run by levels, large ones in one
launch.  Both sides of the rule give the sums and gradients of the level kernels
(a reproducible batch), and no batch takes longer than the reproducible one, which
does the same work on the level kernels with its adds in order (one launch took 1.5
times as long for four flavours in one group)."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _batch(nconf, nflav, det):
    from paper_2507_12349_amd import _binding as B
    return B.Batch(np.full(nconf, 5, dtype=np.int32), nflav, B.FLAVOUR, stubs=True, deterministic=det)


@pytest.mark.parametrize("nflav", [3, 4])
@pytest.mark.parametrize("nconf", [64, 300, 2048, 2049])
def test_both_sides(nflav, nconf):
    import torch
    announce("order 5, %d flavours, %d configurations" % (nflav, nconf))
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(5 * nflav + nconf)
    G = torch.as_tensor(rng.normal(size=nconf * nflav * 25) * 0.4, device=dev)
    st = torch.as_tensor(rng.normal(size=(nconf, nflav)) * 0.3, device=dev)
    ob = torch.as_tensor(rng.normal(size=nconf), device=dev)

    def sweep(b, G, st, w, ob):
        S, Gb, sb = torch.empty_like(ob), torch.empty_like(G), torch.empty_like(st)
        b.adjoint(G, None, st, w, ob, S, Gb, sb)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in (S, Gb, sb)]

    best, res = {}, {}
    for det in (False, True):
        b = _batch(nconf, nflav, det)
        res[det] = sweep(b, G, st, -1.0, ob)
        bound = sweep(b, G.abs(), -st.abs(), 1.0, ob.abs())
        S, Gb, sb = torch.empty_like(ob), torch.empty_like(G), torch.empty_like(st)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            e0.record()
            for _ in range(20):
                b.adjoint(G, None, st, -1.0, ob, S, Gb, sb)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) / 20)
        b.close()
        best[det] = min(times[1:])
    print("  default %.3f ms, reproducible %.3f ms" % (best[False], best[True]), flush=True)
    assert np.array_equal(res[False][0], res[True][0])
    for x, y, z in zip(res[False][1:], res[True][1:], bound[1:]):
        assert np.all(np.abs(x - y) <= 2 * 8 * 5 * 7 * EPS * np.abs(z) + 1e-300)
    assert best[False] <= 1.25 * best[True]
