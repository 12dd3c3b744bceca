"""The autotuner on orders whose forward is one launch: there is no forward shape to
time, so it stays what it was, also where the reverse runs by levels and is tuned."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,segments", [(3, 2), (4, 2), (5, 2), (5, 1)])
def test_forward_shape_is_kept(n, segments):
    import torch
    from paper_2507_12349_amd import _binding as B
    announce("autotuner, one-launch forward: n=%d segments=%d" % (n, segments))
    nconf = 500
    dev = torch.device("cuda:0")
    G = torch.as_tensor(np.random.default_rng(n).normal(size=nconf * n * n) * 0.4, device=dev)
    S, ob = torch.empty(nconf, dtype=torch.float64, device=dev), torch.ones(nconf, dtype=torch.float64, device=dev)
    Gb = torch.empty_like(G)
    b = B.Batch(np.full(nconf, n, dtype=np.int32), 2, B.UNIFORM)
    b.set_adjoint_segments(segments)
    try:
        for waves, masks in ((3, 5), (7, 11)):   # no candidates of the tuner
            b.set_launch_shape(n, waves, masks, 7)
            b.autotune(G, None, None, -1.0, S, ob, Gb, None)
            shape = b.launch_shape(n)
            assert (shape["fwd_waves"], shape["fwd_masks"]) == (waves, masks)
            assert (shape["adj_masks"] == 7) == (segments == 1)
        tuned = S.clone()
        b.forward(G, None, None, -1.0, S)
        torch.cuda.synchronize()
        assert torch.equal(S, tuned)
    finally:
        b.close()
