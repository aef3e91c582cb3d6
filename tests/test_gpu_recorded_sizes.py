"""A recorded evaluation is replayed on larger observations than it was recorded with (the
reservation covers them): its work then comes from the queues, each of which needs a workgroup even
where the recording had few items.  Costs are those of an eager call bit for bit (the FP64 depth
sums are exact); gradients agree to 1e-5 of their largest component (their FP32 row sums take
other tiles together)."""
import numpy as np
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 5])
@pytest.mark.parametrize("grad", [False, True])
def test_recorded_on_a_small_observation_replayed_on_a_large_one(n, grad):
    torch = torch_cuda()
    cfg, model, fr = frame_for(5)
    small = dict(fr, depth=np.ascontiguousarray(fr["depth"][:24, :24]),
                 skin=np.ascontiguousarray(fr["skin"][:24, :24]))
    H, W = fr["depth"].shape
    ctx = make_ctx(model, [small])
    ctx.reserve(8, H * W)
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    x = torch.tensor(particles_for(model, fr, n, seed=60 + n), device="cuda:0")

    def call():
        return ctx.eval_grad(x, slots) if grad else (ctx.eval(x, slots), None)
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cost, gr = call()
    for frame in (fr, small, fr):
        ctx.set_observation(0, frame["depth"], frame["skin"], frame["cam"], frame["bg"])
        g.replay()
        torch.cuda.synchronize()
        ref, ref_g = call()
        assert torch.equal(cost, ref)
        if grad:
            scale = ref_g.abs().amax(1, keepdim=True)
            assert (frame is small or scale.min() > 0) and torch.all((gr - ref_g).abs() <= 1e-5 * scale)
    ctx.close()
