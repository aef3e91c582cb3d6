"""The whole-frame background sums of an observation, for tile counts around the quads and rounds
in which one workgroup adds them.  A hand out of view costs the background alone, so the oracle's
terms of the empty render give its cost: FP64 sums of whole numbers, exact, then one rounding to
FP32 (relative 2^-24, doubled)."""
import numpy as np
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda
from oracle import cost as ocost

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(8, 8), (5, 3), (17, 8), (40, 8), (256, 128), (512, 512), (513, 512),
                                 (1025, 257)])
def test_background_cost_of_uneven_tile_counts(W, H):
    torch = torch_cuda()
    dev = torch.device("cuda:0")
    cfg, model, fr = frame_for(1)
    rng = np.random.default_rng(W * 7 + H)
    bg = 900.0
    depth = rng.integers(860, 940, (H, W)).astype(np.uint16)
    depth[rng.random((H, W)) < 0.1] = 0
    skin = (rng.random((H, W)) < 0.3).astype(np.uint8)
    skin[0, 0] = 1
    ctx = make_ctx(model, [{"depth": depth, "skin": skin, "cam": fr["cam"], "bg": bg}])
    x = particles_for(model, fr, 3, seed=5)
    x[:, 20] = 1.0e5                                # out of view
    got = ctx.eval(torch.tensor(x, device=dev), torch.zeros(1, dtype=torch.int32, device=dev))
    none = np.zeros((H, W), bool)
    D = ocost.discrepancy(depth, skin, np.full((H, W), bg), none)[0]
    for p in range(3):
        want = D + ocost.LAMBDA_K * ocost.kc(model, x[p].astype(np.float64))
        assert abs(float(got[p]) - want) <= 2.0 ** -23 * abs(want)
    ctx.close()
