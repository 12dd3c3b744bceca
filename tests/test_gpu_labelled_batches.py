"""Labelled (bipartite) sums over batch sizes: a few configurations (levels split
by rows, groups that are not full) and the same ones repeated to a large batch
(blocks of many masks), bit for bit the same sums, gradients within the bound of
their order of accumulation, and both against the oracle's sum over label
assignments where that is quick.

Tolerances: |S_gpu - S| <= 8 n (n + 2) eps S_abs, and per gradient entry the
same factor times the gradient over absolute values."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _sweep(A, nflav, variant, mask_only, w, ob):
    import torch
    from paper_2507_12349_amd import _binding as B
    nconf, n = A.shape[0], A.shape[-1] // 2
    dev = torch.device("cuda:0")
    G = torch.as_tensor(A.reshape(-1), device=dev)
    S, S2 = (torch.full((nconf,), float("nan"), dtype=torch.float64, device=dev) for _ in range(2))
    Gb = torch.full_like(G, float("nan"))
    b = B.Batch(np.full(nconf, n, dtype=np.int32), nflav, variant, sublattice=True, mask_only=mask_only)
    b.forward(G, None, None, w, S)
    b.adjoint(G, None, None, w, torch.as_tensor(ob, device=dev), S2, Gb, None)
    torch.cuda.synchronize()
    b.close()
    S, S2 = S.cpu().numpy(), S2.cpu().numpy()
    assert np.array_equal(S, S2)
    return S, Gb.cpu().numpy().reshape(A.shape)


@pytest.mark.parametrize("n,nflav,variant,mask_only,repeat", [(2, 3, 1, False, 50), (4, 2, 1, False, 700), (5, 3, 1, False, 300),
                                                              (5, 4, 0, False, 300), (6, 2, 1, True, 200), (7, 2, 1, False, 100),
                                                              (8, 3, 1, False, 22)])
def test_few_and_many(oracle_mod, n, nflav, variant, mask_only, repeat):
    from oracle import sublattice as SL
    announce("labelled n=%d nflav=%d variant=%d mask_only=%s: 3 and %d configurations" % (n, nflav, variant, mask_only, 3 * repeat))
    rng = np.random.default_rng(17 * n + nflav)
    nmat = nflav if variant else 1
    A, ob = rng.normal(size=(3, nmat, 2 * n, 2 * n)) * 0.4, rng.normal(size=3)
    S, Gb = _sweep(A, nflav, variant, mask_only, -1.0, ob)
    Sm, Gm = _sweep(np.tile(A, (repeat, 1, 1, 1)), nflav, variant, mask_only, -1.0, np.tile(ob, repeat))
    assert np.array_equal(Sm, np.tile(S, repeat))
    if mask_only:   # the clows cancel only for w = -1: a bound from the entries' size
        assert np.allclose(Gm, np.tile(Gb, (repeat, 1, 1, 1)), rtol=0, atol=1e-12 * np.abs(Gb).max())
        return
    _, Ga = _sweep(np.abs(A), nflav, variant, False, 1.0, np.abs(ob))
    tol = 8 * n * (n + 2) * EPS
    assert np.all(np.abs(Gm - np.tile(Gb, (repeat, 1, 1, 1))) <= 2 * tol * np.tile(Ga, (repeat, 1, 1, 1)) + 1e-300)
    if n > 5:
        return
    for i in range(3):
        M = A[i] if variant else A[i, 0]
        ref, g = SL.by_assignment_adjoint(M, nflav, variant)
        sabs, gabs = SL.by_assignment_adjoint(np.abs(M), nflav, variant, 1.0)
        assert abs(S[i] - ref) <= tol * sabs, i
        assert np.all(np.abs(Gb[i] - ob[i] * np.reshape(g, Gb[i].shape)) <= tol * abs(ob[i]) * np.reshape(gabs, Gb[i].shape) + 1e-300), i
