"""Propagator kernels over batches: several configurations share a workgroup
(from 4096 on), ragged orders share its threads, and matrices whose tables do
not fit LDS together are served in turns.  Sampled configurations, among them
those next to workgroup edges, against the oracle's builders, entry by entry
within 1e-12 relative or 1e-13 of the matrix's largest entry (a sum of L^2
terms of that size)."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _batch(nconf, n_lo, n_hi, L, beta, per, seed):
    rng = np.random.default_rng(seed)
    n = rng.integers(n_lo, n_hi + 1, size=nconf).astype(np.int32)
    voff = np.concatenate([[0], np.cumsum(n[:-1])]).astype(np.int64)
    sizes = per * n.astype(np.int64) ** 2
    off = np.concatenate([[0], np.cumsum(sizes[:-1])]).astype(np.int64)
    sites = rng.integers(0, L, size=(int(n.sum()), 2)).astype(np.int32)
    tau = rng.uniform(0.0, beta, size=int(n.sum()))
    picks = sorted({0, min(nconf - 1, 1), nconf // 2, nconf - 1, min(nconf - 1, 2), min(nconf - 1, 7), min(nconf - 1, 8)})
    return n, voff, sizes, off, sites, tau, picks


def _close(got, ref):
    return np.allclose(got, ref, rtol=1e-12, atol=1e-13 * np.max(np.abs(ref)))


@pytest.mark.parametrize("nconf,n_lo,n_hi,L,nmat", [(1, 4, 4, 4, 1), (4096, 1, 5, 8, 1), (6149, 3, 3, 7, 2),
                                                    (20000, 2, 4, 3, 1), (37, 9, 12, 16, 6), (5, 2, 6, 32, 16),
                                                    (4100, 1, 12, 6, 3)])
def test_square_batches(nconf, n_lo, n_hi, L, nmat):
    import torch
    from oracle import g0
    from paper_2507_12349_amd import _binding as B
    announce("square-lattice propagators: %d configurations, n=%d..%d L=%d nmat=%d" % (nconf, n_lo, n_hi, L, nmat))
    beta = 4.0
    n, voff, sizes, off, sites, tau, picks = _batch(nconf, n_lo, n_hi, L, beta, nmat, nconf + L)
    mu, alpha = np.linspace(-1.5, 0.8, nmat), np.linspace(0.2, -0.1, nmat)
    dev = torch.device("cuda:0")
    dn, dv, ds, dt, do = (torch.as_tensor(x, device=dev) for x in (n, voff, sites.reshape(-1), tau, off))
    G, dG, G2 = (torch.full((int(sizes.sum()),), float("nan"), dtype=torch.float64, device=dev) for _ in range(3))
    B.build_g0(nconf, dn, dv, ds, dt, L, 1.0, beta, mu, alpha, do, G, dG)
    B.build_g0(nconf, dn, dv, ds, dt, L, 1.0, beta, mu, alpha, do, G2, None)
    torch.cuda.synchronize()
    assert torch.equal(G, G2) and bool(torch.isfinite(G).all()) and bool(torch.isfinite(dG).all())
    Gh, dGh = G.cpu().numpy(), dG.cpu().numpy()
    for c in picks:
        k, v = int(n[c]), int(voff[c])
        Go, dGo = g0.build_g0(L, 1.0, beta, mu, alpha, sites[v:v + k], tau[v:v + k])
        assert _close(Gh[off[c]:off[c] + sizes[c]].reshape(nmat, k, k), Go), c
        assert _close(dGh[off[c]:off[c] + sizes[c]].reshape(nmat, k, k), dGo), c


@pytest.mark.parametrize("nconf,n_lo,n_hi,L,nmat", [(1, 3, 3, 4, 1), (4099, 1, 3, 5, 2), (9, 6, 8, 16, 2), (3, 2, 4, 32, 5)])
def test_honeycomb_batches(nconf, n_lo, n_hi, L, nmat):
    import torch
    from oracle import g0_honeycomb as GH
    from paper_2507_12349_amd import _binding as B
    announce("honeycomb propagators: %d configurations, n=%d..%d L=%d nmat=%d" % (nconf, n_lo, n_hi, L, nmat))
    beta = 4.0
    n, voff, sizes, off, cells, tau, picks = _batch(nconf, n_lo, n_hi, L, beta, 4 * nmat, nconf + L)
    mu, alpha, delta = np.linspace(-0.5, 0.4, nmat), np.linspace(0.1, -0.1, nmat), 0.3 * (1.0 - 2.0 * (np.arange(nmat) % 2))
    dev = torch.device("cuda:0")
    dn, dv, ds, dt, do = (torch.as_tensor(x, device=dev) for x in (n, voff, cells.reshape(-1), tau, off))
    G, dG = (torch.full((int(sizes.sum()),), float("nan"), dtype=torch.float64, device=dev) for _ in range(2))
    B.build_g0_honeycomb(nconf, dn, dv, ds, dt, L, 1.0, beta, mu, alpha, delta, do, G, dG=dG)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(G).all()) and bool(torch.isfinite(dG).all())
    Gh, dGh = G.cpu().numpy(), dG.cpu().numpy()
    for c in picks:
        k, v = int(n[c]), int(voff[c])
        args = (L, 1.0, beta, mu, alpha, delta, cells[v:v + k], tau[v:v + k])
        Go, dGo = GH.build_g0(*args), GH.build_dg0(*args)
        assert _close(Gh[off[c]:off[c] + sizes[c]].reshape(nmat, 2 * k, 2 * k), Go), c
        assert _close(dGh[off[c]:off[c] + sizes[c]].reshape(nmat, 2 * k, 2 * k), dGo), c
