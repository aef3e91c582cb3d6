"""Forward launches of more than 128 particles of a 128x128 frame: split into parts and assembled
(a finalize launch), one workgroup per particle, or from the work queues, at every edge between
these for one, two and all workgroups per CU.  The trace says which it was; costs are those of
launches of 64, which take the kinematics and the cast in one kernel, bit for bit (the FP64 depth
sums are exact)."""
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu

SIZES = [129, 255, 256, 257, 511, 512, 513, 1024, 1025, 2047, 2048, 2049]


@pytest.mark.parametrize("primitive_set", ["cylinders", "paper"])
def test_parts_single_workgroups_and_queues_agree(primitive_set):
    torch = torch_cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    cfg, model, fr = frame_for(1, primitive_set=primitive_set)
    ctx = make_ctx(model, [fr])
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    x = torch.tensor(particles_for(model, fr, max(SIZES), seed=31), device="cuda:0")
    x[77, 3] = float("nan")
    ref = torch.cat([ctx.eval(x[i:i + 64].contiguous(), slots) for i in range(0, len(x), 64)])
    assert torch.isinf(ref[77])
    split = 0
    for gpc in (1, 2, 8):
        for tpi in (4, 64):
            ctx.set_launch_config(tpi, gpc, 1)
            for n in SIZES:
                ctx.eval_counts(reset=True)
                ctx.profile_begin()
                cost = ctx.eval(x[:n].contiguous(), slots)
                launches = {k: v["launches"] for k, v in ctx.profile_end().items()}
                assert ctx.eval_counts() == (n, 0)
                assert torch.equal(cost, ref[:n]), (gpc, tpi, n)
                assert launches["fk"] == launches["raycast"] == 1 and not launches["sched"]
                if gpc < 8:
                    assert launches["finalize"] == int(gpc * cus // n >= 2), (gpc, n)
                split += launches["finalize"]
    assert split >= 10
    ctx.close()


@pytest.mark.parametrize("n", [129, 255, 257, 600])
def test_gradients_do_not_depend_on_the_workgroups(n):
    """The work items of a gradient launch follow from the configured shape alone: with four, five
    and more workgroups per CU asked for, the same items run on other grids.  8 and 64 give the
    same bits; costs are the same with every shape."""
    torch = torch_cuda()
    cfg, model, fr = frame_for(4)
    ctx = make_ctx(model, [fr])
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    x = torch.tensor(particles_for(model, fr, n, seed=33), device="cuda:0")
    cost = ctx.eval(x, slots)
    got = {}
    for gpc in (1, 2, 4, 8, 64):
        ctx.set_launch_config(64, gpc, 1)
        got[gpc] = ctx.eval_grad(x, slots)
        assert torch.equal(got[gpc][0], cost), gpc
    assert torch.equal(got[8][1], got[64][1])
    scale = got[8][1].abs().amax(1, keepdim=True)
    for gpc in (1, 2, 4):      # FP32 row sums of other tiles
        assert torch.all((got[gpc][1] - got[8][1]).abs() <= 1e-5 * scale), gpc
    ctx.close()
