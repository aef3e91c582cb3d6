"""Small evaluations count a particle's finished parts in device memory that outlives the call.  A
count may not carry over: not from call to call, not into or out of recorded launches, and not from
calls that overlapped on two streams (which a program must not let happen: they share one
workspace and spoil each other's results, but nothing after them)."""
import numpy as np
import pytest

from gpu_util import frame_for, make_ctx, particles_for, torch_cuda

pytestmark = pytest.mark.gpu


def _setup():
    torch = torch_cuda()
    cfg, model, fr = frame_for(1)
    ctx = make_ctx(model, [fr])
    slots = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    xs = [torch.tensor(particles_for(model, fr, n, seed=50 + n), device="cuda:0")
          for n in (5, 16, 40, 100)]
    # (a gradient evaluation counts nothing)
    refs = [ctx.eval_grad(x, slots)[0].cpu().numpy() for x in xs]
    return torch, ctx, slots, xs, refs


def test_calls_after_overlapping_ones_are_right():
    torch, ctx, slots, xs, refs = _setup()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for rnd in range(10):
        for k in range(8):                       # overlapping, of other sizes: results unused
            with torch.cuda.stream(streams[k % 2]):
                ctx.eval(xs[(k + rnd) % 4], slots)
        torch.cuda.synchronize()
        for x, ref in zip(xs, refs):
            assert np.array_equal(ctx.eval(x, slots).cpu().numpy(), ref), rnd
    ctx.close()


def test_many_calls_in_a_row():
    torch, ctx, slots, xs, refs = _setup()
    got = [(k % 4, ctx.eval(xs[k % 4], slots)) for k in range(203)]
    for k, (i, c) in enumerate(got):
        assert np.array_equal(c.cpu().numpy(), refs[i]), k
    ctx.close()


def test_recorded_and_eager_calls_take_turns():
    torch, ctx, slots, xs, refs = _setup()
    outs = [torch.empty((1, len(x)), device="cuda:0") for x in xs]
    graphs = []
    for x, out in zip(xs, outs):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            ctx.eval(x[None], slots, cost=out)
        graphs.append(g)
    for rnd in range(4):
        for g, x, out, ref in zip(graphs, xs, outs, refs):
            out.fill_(-1.0)
            g.replay()
            if rnd % 2:
                g.replay()
            assert np.array_equal(ctx.eval(x, slots).cpu().numpy(), ref)
            assert np.array_equal(out[0].cpu().numpy(), ref), rnd
    ctx.close()
