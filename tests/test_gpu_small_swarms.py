"""The edges of the one-launch swarm update: 96 particles of a frame, and 3328 pose parameters (64
two-hand particles).  One generation on both sides against the oracle's update of the same costs,
and the trace of which launches it took (the one-launch update assembles the costs itself)."""
import pytest

import paper_2005_07068_amd as ht
import test_gpu_launch_split as split
from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu

EDGES = [(1, 95), (1, 96), (1, 97), (4, 63), (4, 64), (4, 65)]


@pytest.mark.parametrize("cfg_idx,P", EDGES)
def test_the_update_matches_the_oracle_on_both_sides(cfg_idx, P):
    split.test_swarm_update_in_one_launch_matches_the_oracle(cfg_idx, P)


@pytest.mark.parametrize("cfg_idx,P", EDGES)
def test_the_launches_of_a_generation(cfg_idx, P):
    torch = torch_cuda()
    cfg, model, fr = frame_for(cfg_idx)
    ctx = make_ctx(model, [fr, fr])
    slots = torch.tensor([0, 1], dtype=torch.int32, device="cuda:0")
    x = torch.tensor(particles_for(model, fr, 2, seed=4), device="cuda:0")
    sw = ctx.swarm(slots, P, x, x, seed=5)
    ctx.pso_init(sw)
    ctx.profile_begin()
    ctx.pso_step(sw, ht.pso_params())
    st = ctx.profile_end()
    one = P <= 96 and P * model["n_dof"] <= 3328
    # 2 P > 128 particles: kinematics and cast apart, in parts
    assert 2 * P <= 128 or st["fk"]["launches"] == 1
    assert st["finalize"]["launches"] == int(not one)
    assert st["pso"]["launches"] == 1
    ctx.close()
