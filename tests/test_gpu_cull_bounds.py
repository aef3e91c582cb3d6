"""The tile test's pixel boxes round inwards and its reach is padded by an eighth of a pixel: no
primitive may be left out of a tile that holds one of its pixels.  Poses spread widely (foreshortened
and overlapping fingers, hands cut by the frame's border, primitives of a pixel or two), hit masks
against the oracle's render outside its ambiguous pixels."""
import numpy as np
import pytest

from gpu_util import eval_debug, frame_for, make_ctx, oracle_renders, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("primitive_set", ["cylinders", "paper"])
@pytest.mark.parametrize("cull", [0, 1])
@pytest.mark.parametrize("scale", [1.0, 0.25])
def test_no_hit_is_culled(primitive_set, cull, scale):
    torch_cuda()
    cfg, model, fr = frame_for(0, primitive_set=primitive_set)
    fr = dict(fr)
    fx, fy, cx, cy = fr["cam"]
    # a shorter focal length about the image centre: the whole hand in a quarter of the pixels
    H, W = fr["depth"].shape
    fr["cam"] = (fx * scale, fy * scale, W / 2 + (cx - W / 2) * scale, H / 2 + (cy - H / 2) * scale)
    ctx = make_ctx(model, [fr])
    ctx.set_launch_config(16, 8, cull)
    poses = particles_for(model, fr, 24, seed=11, angle_deg=60.0, trans_mm=60.0)
    _, dbg = eval_debug(ctx, poses, 0, W, H)
    ctx.close()
    for i, (res, cls) in enumerate(oracle_renders(model, [(fr, p) for p in poses])):
        bad = (dbg["hit"][i].astype(bool) != res["hit"]) & ~cls["ambiguous"]
        assert not bad.any(), f"pose {i}: {int(bad.sum())} hit/miss mismatches"
