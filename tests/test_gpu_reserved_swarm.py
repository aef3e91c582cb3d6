"""A reservation covers a swarm's generation: nothing is left to be allocated when the first one is
recorded, whichever kernels it takes (the one-launch update, or the separate ones with their
flags).  Replays go on as eager generations do, bit for bit."""
import pytest

import paper_2005_07068_amd as ht
from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [64, 128, 300])
def test_a_first_generation_can_be_recorded_after_a_reservation(P):
    torch = torch_cuda()
    cfg, model, fr = frame_for(1)
    out = []
    for recorded in (True, False):
        ctx = make_ctx(model, [fr])
        ctx.reserve(P, fr["depth"].size)
        slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
        x = torch.tensor(particles_for(model, fr, 2, seed=6), device="cuda:0")
        sw = ctx.swarm(slots, P, x.amin(0)[None], x.amax(0)[None], seed=9)
        ctx.pso_init(sw)
        if recorded:
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                ctx.pso_step(sw, ht.pso_params(mutate_every=2))
        for _ in range(4):
            if recorded:
                g.replay()
            else:
                ctx.pso_step(sw, ht.pso_params(mutate_every=2))
        torch.cuda.synchronize()
        out.append({k: sw[k].cpu() for k in ("x", "v", "pbest_cost", "gbest_x", "gen")})
        ctx.close()
    assert out[0]["gen"].item() == 4
    for k in out[0]:
        assert torch.equal(out[0][k], out[1][k]), k
