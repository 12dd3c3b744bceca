"""Phase times of orders whose sweep is one launch: the forward inside an
adjoint is reported as forward, not as reverse, and a batch whose phases are
timed gives the results of one that is not."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("n,nflav,variant,limit", [(4, 3, 0, 0), (5, 3, 0, 0), (5, 3, 1, 0), (5, 3, 0, 1)])
def test_phases_of_one_launch_orders(n, nflav, variant, limit):
    import torch
    from paper_2507_12349_amd import _binding as B
    announce("phase times of a one-launch order: n=%d nflav=%d variant=%d limit=%d" % (n, nflav, variant, limit))
    rng = np.random.default_rng(70 + n)
    nconf, nmat = 300, nflav if variant else 1
    dev = torch.device("cuda:0")
    G = torch.as_tensor(rng.normal(size=nconf * nmat * n * n) * 0.4, device=dev)
    st = torch.as_tensor(rng.normal(size=(nconf, nmat)) * 0.3, device=dev)
    ob = torch.as_tensor(rng.normal(size=nconf), device=dev)
    B.set_workspace_limit(limit)   # 1: one group of 64 configurations per chunk
    b = B.Batch(np.full(nconf, n, dtype=np.int32), nflav, variant, stubs=True)
    b.set_adjoint_segments(1)
    B.set_workspace_limit(0)

    def adjoint(G, st, w, ob):
        S = torch.full((nconf,), float("nan"), dtype=torch.float64, device=dev)
        Gb, sb = torch.full_like(G, float("nan")), torch.full_like(st, float("nan"))
        b.adjoint(G, None, st, w, ob, S, Gb, sb)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in (S, Gb, sb)]

    plain = adjoint(G, st, -1.0, ob)
    bound = adjoint(G.abs(), -st.abs(), 1.0, ob.abs())
    b.timing(True)
    out = torch.empty(nconf, dtype=torch.float64, device=dev)
    b.forward(G, None, st, -1.0, out)
    b.timing_read()
    for _ in range(20):
        b.forward(G, None, st, -1.0, out)
    fwd, calls = b.timing_read()
    assert calls == 20
    for _ in range(20):
        timed = adjoint(G, st, -1.0, ob)
    both, calls = b.timing_read()
    b.close()
    print("  forward calls %s\n  adjoint calls %s" % (fwd, both), flush=True)
    assert calls == 20
    # the same levels as in a forward call, in the phase that bears their name
    assert both["forward"] > 0.5 * fwd["forward"]
    assert both["reverse"] > 0.5 * fwd["forward"]
    assert np.array_equal(timed[0], plain[0])
    for x, y, z in zip(timed[1:], plain[1:], bound[1:]):
        assert np.all(np.abs(x - y) <= 2 * 8 * n * (n + 2) * EPS * np.abs(z) + 1e-300)
