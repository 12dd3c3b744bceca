"""Deterministic gradients of large batches, where one workgroup serves several
parts of a level: bit for bit those of the same configurations in a small batch
(one part per workgroup) and in chunks, within the rounding bound of the default
reverse sweep, and in a time of its order.

The level kernels of orders 2 to 5, which a deterministic batch takes, against
the one-launch sweeps, which a default batch takes, and the oracle."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _gradients(G, st, ob, n, nflav, variant, mask, det, w=-1.0, limit=0):
    import torch
    from paper_2507_12349_amd import _binding as B
    nconf = ob.numel()
    B.set_workspace_limit(limit)
    b = B.Batch(np.full(nconf, n, dtype=np.int32), nflav, variant, stubs=st is not None, mask_only=mask,
                deterministic=det)
    B.set_workspace_limit(0)
    S = torch.full((nconf,), float("nan"), dtype=torch.float64, device=G.device)
    Gb, sb = torch.full_like(G, float("nan")), None if st is None else torch.full_like(st, float("nan"))
    b.adjoint(G.view(-1), None, st, w, ob, S, Gb.view(-1), sb)
    torch.cuda.synchronize()
    b.close()
    return [x.cpu().numpy() for x in (S, Gb, sb) if x is not None]


def _inputs(n, nconf, nmat, stubs, seed):
    import torch
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(seed)
    G = torch.as_tensor(rng.normal(size=(nconf, nmat, n, n)) * 0.4, device=dev)
    st = torch.as_tensor(rng.normal(size=(nconf, nmat)) * 0.3, device=dev) if stubs else None
    return G, st, torch.as_tensor(rng.normal(size=nconf), device=dev)


def _close(a, b, n, G, st, ob, nflav, variant, mask):
    """Two sweeps of the same inputs: equal sums, gradients within the bound."""
    assert np.array_equal(a[0], b[0])
    if mask:   # the clows cancel only for w = -1: a bound from the entries' size
        assert np.allclose(a[1], b[1], rtol=0, atol=1e-12 * np.abs(b[1]).max())
        return
    ref = _gradients(G.abs(), None if st is None else -st.abs(), ob.abs(), n, nflav, variant, False, False, 1.0)
    for x, y, z in zip(a[1:], b[1:], ref[1:]):
        assert np.all(np.abs(x - y) <= 2 * 8 * n * (n + 2) * EPS * np.abs(z) + 1e-300)


@pytest.mark.parametrize("n,nflav,variant,stubs,mask,nconf", [
    (3, 2, 0, True, False, 65536 + 3), (4, 3, 1, True, False, 8192 + 1), (4, 2, 1, False, True, 16384),
    (5, 2, 0, True, False, 8192 + 65), (5, 3, 1, False, False, 4096), (6, 2, 0, True, False, 4096 + 1),
    (6, 2, 1, False, True, 2048), (7, 3, 1, True, False, 1024 + 1), (8, 2, 0, False, False, 2048)])
def test_bits_do_not_depend_on_the_batch(n, nflav, variant, stubs, mask, nconf):
    announce("deterministic reverse of a large batch: n=%d nflav=%d variant=%d stubs=%s mask_only=%s nconf=%d"
             % (n, nflav, variant, stubs, mask, nconf))
    G, st, ob = _inputs(n, nconf, nflav if variant else 1, stubs, 40 + n)
    large = _gradients(G, st, ob, n, nflav, variant, mask, True)
    chunks = _gradients(G, st, ob, n, nflav, variant, mask, True, limit=8 << 20)
    k = 65
    small = _gradients(G[:k].contiguous(), None if st is None else st[:k].contiguous(), ob[:k], n, nflav, variant, mask,
                       True)
    for x, y, z in zip(large, chunks, small):
        assert np.array_equal(x, y) and np.array_equal(x[:k], z)
    _close(large, _gradients(G, st, ob, n, nflav, variant, mask, False), n, G, st, ob, nflav, variant, mask)


@pytest.mark.parametrize("n,nconf", [(6, 8192), (7, 8192)])
def test_cost_of_large_batches(n, nconf):
    """Both reverse sweeps read and write the same states; the deterministic one
    adds its terms in turn.  At these sizes that took less than twice the time
    of the default; a launch of a workgroup per part took three times as long."""
    import torch
    from paper_2507_12349_amd import _binding as B
    announce("deterministic reverse, time against the default: n=%d nconf=%d" % (n, nconf))
    G, _, ob = _inputs(n, nconf, 1, False, 3)
    S, Gb = torch.empty_like(ob), torch.empty_like(G)
    best = {}
    for det in (False, True):
        b = B.Batch(np.full(nconf, n, dtype=np.int32), 2, B.UNIFORM, deterministic=det)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            e0.record()
            for _ in range(4):
                b.adjoint(G.view(-1), None, None, -1.0, ob, S, Gb.view(-1), None)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) / 4)
        b.close()
        best[det] = min(times[1:])
    print("  default %.3f ms, deterministic %.3f ms" % (best[False], best[True]), flush=True)
    assert best[True] <= 2.25 * best[False]


@pytest.mark.parametrize("nconf", [1, 64, 65])
@pytest.mark.parametrize("nflav,variant,stubs,mask", [(3, 0, True, False), (2, 1, False, True), (3, 1, True, False),
                                                      (9, 1, True, False)])
@pytest.mark.parametrize("n", [2, 3, 4, 5])
def test_level_kernels_of_small_orders(oracle_mod, n, nflav, variant, stubs, mask, nconf):
    announce("level kernels of small orders: n=%d nflav=%d variant=%d stubs=%s mask_only=%s nconf=%d"
             % (n, nflav, variant, stubs, mask, nconf))
    G, st, ob = _inputs(n, nconf, nflav if variant else 1, stubs, 60 + n)
    lev = _gradients(G, st, ob, n, nflav, variant, mask, True)
    _close(lev, _gradients(G, st, ob, n, nflav, variant, mask, False), n, G, st, ob, nflav, variant, mask)
    if mask:
        return
    for c in {0, nconf - 1}:
        M = G[c].cpu().numpy()
        M, s, o = M if variant else M[0], st[c].cpu().numpy(), float(ob[c])
        S, gref, sref = oracle_mod.dp_adjoint(M, nflav, variant, s, -1.0)
        sabs, gabs, sbabs = oracle_mod.dp_adjoint(np.abs(M), nflav, variant, -np.abs(s), 1.0)
        tol = 8 * n * (n + 2) * EPS
        assert abs(lev[0][c] - S) <= tol * sabs
        assert np.all(np.abs(lev[1][c].reshape(gref.shape) - o * gref) <= tol * np.abs(o * gabs) + 1e-300)
        assert np.all(np.abs(lev[2][c] - o * np.reshape(sref, -1)) <= tol * np.abs(o * np.reshape(sbabs, -1)) + 1e-300)
