"""The autotuner chooses only among launches that differ: groups_per_cu stays at 8 where the timed
launch takes no account of it, and is never 4, which launches as 8 does."""
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg_idx,n", [(0, 1), (0, 16), (1, 64), (0, 512), (4, 128), (1, 300), (1, 4000)])
def test_the_tuner_does_not_choose_by_noise(cfg_idx, n):
    torch = torch_cuda()
    cfg, model, fr = frame_for(cfg_idx)
    ctx = make_ctx(model, [fr])
    x = torch.tensor(particles_for(model, fr, n, seed=8)[None], device="cuda:0")
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    ref = ctx.eval(x, slots)
    one_launch = n <= 128
    for _ in range(12 if one_launch else 3):
        tpi, gpc, cull = ctx.autotune(x, slots, repeats=2)
        assert tpi == 64 and gpc in ((8,) if one_launch else (8, 2, 1)) and cull in (0, 1)
        assert ctx.launch_config() == (tpi, gpc, cull)
    assert torch.equal(ctx.eval(x, slots), ref)
    ctx.close()
