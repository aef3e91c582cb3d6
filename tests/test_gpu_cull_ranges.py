"""Tile culling far from the ordinary view: 4096-pixel strips, crops whose principal point lies
thousands of pixels away, hands close to the camera and far from it, wide and narrow lenses, unequal
focal lengths.  A primitive may be left out of no tile that holds one of its pixels: hit masks
against the oracle's render outside its ambiguous pixels."""
import numpy as np
import pytest

from gpu_util import (MARGIN_TAU, eval_debug, frame_for, make_ctx, oracle_render, particles_for,
                      torch_cuda)
from oracle import raycast

pytestmark = pytest.mark.gpu

# image size, focal lengths, where the hand's centre is seen, its depth, the principal point
VIEWS = {
    "strip across": ((4096, 24), (575.0, 575.0), (3900.0, 12.0), 500.0, (2047.5, 12.0)),
    "strip down": ((24, 4096), (575.0, 575.0), (12.0, 150.0), 500.0, (12.0, 2047.5)),
    "crop right of the axis": ((120, 104), (1200.0, 1200.0), (60.0, 52.0), 900.0, (-6000.0, 40.0)),
    "crop far off both axes": ((104, 120), (3000.0, 3000.0), (52.0, 60.0), 2500.0, (-20000.0, 9000.0)),
    "wide lens, grazing": ((160, 120), (150.0, 150.0), (80.0, 60.0), 250.0, (-1500.0, -300.0)),
    "close": ((200, 160), (60.0, 60.0), (100.0, 80.0), 130.0, (100.0, 80.0)),
    "close to the corner": ((200, 160), (90.0, 90.0), (180.0, 20.0), 170.0, (60.0, 110.0)),
    "far, a few pixels": ((64, 64), (575.0, 575.0), (30.2, 33.7), 4000.0, (31.5, 31.5)),
    "unequal focal lengths": ((160, 160), (300.0, 700.0), (70.0, 90.0), 600.0, (900.0, -700.0)),
}


@pytest.mark.parametrize("primitive_set", ["cylinders", "paper"])
@pytest.mark.parametrize("view", VIEWS)
def test_no_hit_is_culled(primitive_set, view):
    torch_cuda()
    (W, H), (fx, fy), (u, v), z, (cx, cy) = VIEWS[view]
    cfg, model, fr = frame_for(0, primitive_set=primitive_set)
    P = 6
    poses = particles_for(model, fr, P, seed=17, angle_deg=50.0, trans_mm=25.0)
    at = np.array([(u - cx) / fx * z, (v - cy) / fy * z, z])
    poses[:, 20:23] += (at - np.asarray(fr["h_true"])[20:23]).astype(np.float32)
    rng = np.random.default_rng(5)
    frame = {"depth": rng.integers(0, 2000, (H, W)).astype(np.uint16),
             "skin": (rng.random((H, W)) < 0.3).astype(np.uint8), "cam": (fx, fy, cx, cy),
             "bg": 30000.0}
    ctx = make_ctx(model, [frame])
    hits = []
    for cull in (0, 1):
        ctx.set_launch_config(16, 8, cull)
        hits.append(eval_debug(ctx, poses, 0, W, H)[1]["hit"].astype(bool))
    ctx.close()
    # FP32 rays are off by 2^-23 of their distance from the principal point (pixels), which moves a
    # margin by at most four times that over the smallest radius in pixels
    off = 2.0 ** -23 * max(abs(cx) + W, abs(cy) + H)
    tau = MARGIN_TAU + 4 * off / (min(fx, fy) * np.min(model["prim_size"][:, 0]) / z)
    seen = 0
    for i, pose in enumerate(poses):
        res, _ = oracle_render(model, frame, pose)
        amb = raycast.classify_pixels(res, tau)["ambiguous"]
        for cull in (0, 1):
            bad = (hits[cull][i] != res["hit"]) & ~amb
            assert not bad.any(), f"pose {i}, cull {cull}: {int(bad.sum())} hit/miss mismatches"
        seen += int((res["hit"] & ~amb).sum())
    assert seen > 20 * P
