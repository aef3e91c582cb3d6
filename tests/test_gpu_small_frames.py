"""Many particles of a frame of few tiles: up to three workgroups per CU (768 particles on 256 CUs)
they go in one launch, beyond that in separate ones.  Costs on both sides are those of a gradient
evaluation, which never takes the one launch, bit for bit."""
import numpy as np
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("primitive_set", ["cylinders", "paper"])
@pytest.mark.parametrize("side,n", [(64, 384), (64, 385), (32, 767), (32, 768), (32, 769), (8, 4096)])
def test_one_launch_and_separate_launches_agree(primitive_set, side, n):
    torch = torch_cuda()
    cfg, model, fr = frame_for(0, primitive_set=primitive_set)
    o = (fr["depth"].shape[0] - side) // 2
    cut = dict(fr, depth=np.ascontiguousarray(fr["depth"][o:o + side, o:o + side]),
               skin=np.ascontiguousarray(fr["skin"][o:o + side, o:o + side]),
               cam=(*fr["cam"][:2], fr["cam"][2] - o, fr["cam"][3] - o))
    ctx = make_ctx(model, [cut])
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    x = torch.tensor(particles_for(model, fr, n, seed=n), device="cuda:0")
    ctx.eval_counts(reset=True)
    cost = ctx.eval(x, slots)
    assert ctx.eval_counts() == (n, 0)
    assert torch.equal(cost, ctx.eval_grad(x, slots)[0])
    assert torch.equal(cost, ctx.eval_noalloc(x, slots))
    ctx.close()
