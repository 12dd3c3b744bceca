"""Several flavour slots on the level kernels: every flavour's workgroups store
their own part of a closed cycle and the readers add the parts up.  A few
configurations (levels split by heads) and the same ones repeated to a large
batch (levels split by masks) against the oracle's sums and gradients, and
against each other: sums bit for bit (heads and flavours are added in the same
order), gradients within the bound of their order of accumulation.

Tolerances as for the uniform form: |S_gpu - S| <= 8 n (n + 2) eps S_abs, and
per gradient entry the same factor times the gradient over absolute values."""
import numpy as np
import pytest

from gpu_util import announce, gpu_forward

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("n,nflav,stubs,repeat", [(6, 2, True, 500), (6, 6, True, 200), (7, 3, False, 300),
                                                  (8, 5, True, 60), (9, 2, False, 40), (10, 3, True, 7)])
def test_flavour_slots(oracle_mod, n, nflav, stubs, repeat):
    announce("flavour slots: n=%d nflav=%d stubs=%s, 3 and %d configurations" % (n, nflav, stubs, 3 * repeat))
    rng = np.random.default_rng(31 * n + nflav)
    mats = [rng.normal(size=(nflav, n, n)) * 0.5 for _ in range(3)]
    st = rng.normal(size=(3, nflav)) * 0.3 if stubs else None
    ob = rng.normal(size=3)
    few = gpu_forward(mats, nflav, 1, st, adjoint=True, out_bar=ob)
    many = gpu_forward(mats * repeat, nflav, 1, None if st is None else np.tile(st, (repeat, 1)), adjoint=True,
                       out_bar=np.tile(ob, repeat))
    assert np.array_equal(few[0], few[1]) and np.array_equal(many[0], many[1])
    assert np.array_equal(many[0], np.tile(few[0], repeat))
    tol = 8 * n * (n + 2) * EPS
    for i, M in enumerate(mats[:1 if n > 8 else 3]):
        s = None if st is None else st[i]
        Sref, gref, sref = oracle_mod.dp_adjoint(M, nflav, 1, s)
        Sabs, gabs, sabs = oracle_mod.dp_adjoint(np.abs(M), nflav, 1, None if s is None else -np.abs(s), 1.0)
        assert abs(few[0][i] - Sref) <= tol * Sabs
        for c, r in ((i, few), (i, many), (i + 3 * (repeat - 1), many)):
            assert np.all(np.abs(r[2][c] - ob[i] * gref) <= tol * abs(ob[i]) * np.abs(gabs) + 1e-300), (i, c)
            if stubs:
                assert np.all(np.abs(r[3][c] - ob[i] * sref) <= tol * abs(ob[i]) * np.abs(sabs) + 1e-300), (i, c)
