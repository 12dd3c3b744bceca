"""Injected launch failures count the steps of a sweep: packing (and zeroing and
unpacking) once per order and 2n levels per chunk of its groups, whether the
levels are launches of their own (order 6) or one launch does them all."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limit,chunks", [(0, 1), (1, 3)])
@pytest.mark.parametrize("n", [2, 4, 5, 6])
def test_steps_of_a_call(n, limit, chunks):
    import torch
    from paper_2507_12349_amd import _binding as B
    announce("steps counted by injected launch failures: n=%d, %d chunk(s)" % (n, chunks))
    nconf = 150   # three groups
    dev = torch.device("cuda:0")
    G = torch.as_tensor(np.random.default_rng(n).normal(size=nconf * n * n) * 0.4, device=dev)
    out, ob = torch.empty(nconf, dtype=torch.float64, device=dev), torch.ones(nconf, dtype=torch.float64, device=dev)
    Gb = torch.empty_like(G)
    B.set_workspace_limit(limit)   # 1: one group of 64 configurations per chunk
    b = B.Batch(np.full(nconf, n, dtype=np.int32), 2, B.UNIFORM)
    b.set_adjoint_segments(1)
    b.adjoint(G, None, None, -1.0, ob, out, Gb, None)
    B.set_workspace_limit(0)
    try:
        for steps, call in ((1 + 2 * n * chunks, lambda: b.forward(G, None, None, -1.0, out)),
                            (4 + 4 * n * chunks, lambda: b.adjoint(G, None, None, -1.0, ob, out, Gb, None))):
            B.inject_failures(1, steps, 1)   # the step after the call's last
            call()
            B.inject_failures(1, steps - 1, 1)   # its last
            with pytest.raises(B.CosError) as e:
                call()
            assert e.value.status == -4
    finally:
        B.inject_failures(1, 0, 0)
        torch.cuda.synchronize()
        b.close()
