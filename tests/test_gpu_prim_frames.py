"""A primitive's local frame counts only as far as its type's definition names it: a sphere has the
frame's origin, a cylinder and a cone its origin and z axis.  The other columns are free (zeros,
or anything), and every result must be that of a model whose frames are orthonormal."""
import numpy as np
import pytest

from gpu_util import eval_debug, frame_for, make_ctx, oracle_renders, particles_for, torch_cuda
from oracle.raycast import CONE, CYLINDER, SPHERE

pytestmark = pytest.mark.gpu


def _with_free_columns(model, fill):
    rng = np.random.default_rng(3)
    m = dict(model)
    m["prim_frame"] = np.array(model["prim_frame"], np.float64)
    for k, t in enumerate(np.asarray(model["prim_type"])):
        free = {SPHERE: 3, CYLINDER: 2, CONE: 2}.get(int(t), 0)
        m["prim_frame"][k, :, :free] = {"zeros": 0.0, "random": rng.uniform(-3, 3, (3, free)),
                                        "nan": np.nan}[fill]
    return m


@pytest.mark.parametrize("primitive_set", ["cylinders", "paper"])
@pytest.mark.parametrize("fill", ["zeros", "random", "nan"])
@pytest.mark.parametrize("cull", [0, 1])
@pytest.mark.parametrize("n", [5, 300])
def test_free_frame_columns_change_nothing(primitive_set, fill, cull, n):
    torch = torch_cuda()
    cfg, model, fr = frame_for(0, primitive_set=primitive_set)
    H, W = fr["depth"].shape
    x = particles_for(model, fr, n, seed=21, angle_deg=40.0)
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    got = []
    for m in (model, _with_free_columns(model, fill)):
        ctx = make_ctx(m, [fr])
        ctx.set_launch_config(16, 8, cull)
        xt = torch.tensor(x, device="cuda:0")
        cost, (c_g, g) = ctx.eval(xt, slots), ctx.eval_grad(xt, slots)
        _, dbg = eval_debug(ctx, x[:5], 0, W, H)
        got.append((cost.cpu().numpy(), c_g.cpu().numpy(), g.cpu().numpy(),
                    *(dbg[k] for k in ("depth", "hit", "rm", "winner", "margin"))))
        ctx.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_free_frame_columns_against_the_oracle():
    """Spheres and cylinders, whose oracle reads no other column either."""
    torch_cuda()
    cfg, model, fr = frame_for(0)
    m = _with_free_columns(model, "zeros")
    H, W = fr["depth"].shape
    x = particles_for(model, fr, 8, seed=22, angle_deg=40.0)
    ctx = make_ctx(m, [fr])
    _, dbg = eval_debug(ctx, x, 0, W, H)
    ctx.close()
    for i, (res, cls) in enumerate(oracle_renders(m, [(fr, p) for p in x])):
        bad = (dbg["hit"][i].astype(bool) != res["hit"]) & ~cls["ambiguous"]
        assert not bad.any(), f"pose {i}: {int(bad.sum())} hit/miss mismatches"
