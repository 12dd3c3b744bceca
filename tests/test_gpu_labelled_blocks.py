"""Blocks of masks of the labelled level kernels: whatever the batch size and the
launch shape cut the levels into (blocks that are not full, more or fewer blocks
than fit the chip, masks or row pairs as the items), the sums of a configuration
are the same bit for bit and its gradients agree within the rounding bound."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _sweep(A, nconf, nflav, mask_only, w, shape=None):
    """S and dS/dG of `nconf` configurations that repeat those of A in turn."""
    import torch
    from paper_2507_12349_amd import _binding as B
    k, n = A.shape[0], A.shape[-1] // 2
    dev = torch.device("cuda:0")
    idx = torch.arange(nconf, device=dev) % k
    G = torch.as_tensor(A, device=dev)[idx].reshape(-1)
    S = torch.full((nconf,), float("nan"), dtype=torch.float64, device=dev)
    Gb = torch.full_like(G, float("nan"))
    b = B.Batch(np.full(nconf, n, dtype=np.int32), nflav, B.FLAVOUR, sublattice=True, mask_only=mask_only)
    if shape:
        b.set_launch_shape(n, *shape)
    b.adjoint(G, None, None, w, torch.ones_like(S), S, Gb, None)
    torch.cuda.synchronize()
    b.close()
    return S.cpu().numpy(), Gb.cpu().numpy().reshape((nconf,) + A.shape[1:])


@pytest.mark.parametrize("n,nflav,mask_only,sizes", [(3, 1, False, (1, 130, 4000)), (3, 2, False, (64, 4000)),
                                                     (4, 1, False, (63, 1000, 4100)), (5, 2, True, (1, 700)),
                                                     (6, 1, False, (1, 129, 1000)), (6, 2, False, (300, 900)),
                                                     (7, 1, False, (22, 300)), (8, 1, False, (1, 65, 200)),
                                                     (8, 2, False, (64,))])
def test_blocks_do_not_change_the_sums(n, nflav, mask_only, sizes):
    announce("labelled blocks: n=%d nflav=%d mask_only=%s" % (n, nflav, mask_only))
    rng = np.random.default_rng(90 + n)
    A = rng.normal(size=(3, nflav, 2 * n, 2 * n)) * 0.4
    S, Gb = _sweep(A, 3, nflav, mask_only, -1.0)
    if mask_only:   # the clows cancel only for w = -1: a bound from the entries' size
        bound = 1e-12 * np.abs(Gb).max(axis=(1, 2, 3), keepdims=True) + np.zeros_like(Gb)
    else:
        bound = 2 * 8 * n * (n + 2) * EPS * _sweep(np.abs(A), 3, nflav, False, 1.0)[1] + 1e-300
    for nconf in sizes:
        for shape in (None, (8, 3, 5), (5, 1, 1), (16, 16, 64)):
            Sm, Gm = _sweep(A, nconf, nflav, mask_only, -1.0, shape)
            i = np.arange(nconf) % 3
            assert np.array_equal(Sm, S[i]), (nconf, shape)
            assert np.all(np.abs(Gm - Gb[i]) <= bound[i]), (nconf, shape)
