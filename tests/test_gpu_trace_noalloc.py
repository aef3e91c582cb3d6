"""ht_eval_particles_noalloc allocates nothing, so tracing (whose events are allocated) leaves its
launches out, whichever launches a call takes."""
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 300])
def test_noalloc_calls_are_not_traced(n):
    torch = torch_cuda()
    cfg, model, fr = frame_for(1)
    ctx = make_ctx(model, [fr])
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    x = torch.tensor(particles_for(model, fr, n, seed=2), device="cuda:0")
    ctx.eval(x, slots)
    ctx.profile_begin()
    ctx.eval_noalloc(x, slots)
    assert all(v["launches"] == 0 for v in ctx.profile_end().values())
    ctx.profile_begin()
    ctx.eval(x, slots)
    assert ctx.profile_end()["raycast"]["particles"] == n
    ctx.close()
