"""Local steps of the residual networks captured in a HIP graph.

Inside a call the weight gradients run on a stream of the library's.  Outside a capture the launch that stores their factor carries the
event they wait for; a captured stream (and one whose launches are timed) records events instead.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("make,init", [("resnet_cifar", "resnet_init"), ("wide_resnet", "wrn_init")])
def test_a_captured_step_replays_the_eager_result(make, init, act):
    import torch
    import paper_2508_08540_amd as bls
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = bls.Context(0, stream.cuda_stream)
        try:
            wide = make == "wide_resnet"
            widths, extra = ((32, 64, 64), dict(stem=16)) if wide else ((16, 32, 64), {})
            model = getattr(bls.Model, make)(widths=widths, blocks=1, classes=10, image_hw=16, act_dtype=act, **extra)
            p, b = synth.wrn_init(3, widths, 1, 10, 16) if wide else synth.resnet_init(3, widths, 1, 10)
            x, y = synth.image_pool(3, 21, 10, hw=16)
            dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
            p0, b0, dx, dy = dev(model.pack(p)), dev(model.pack(b, buffers=True)), dev(x), dev(y)
            sel = dev(np.arange(20, -1, -1, dtype=np.int32))
            ps, bs, ms, ls = torch.empty_like(p0), torch.empty_like(b0), torch.empty_like(p0), torch.empty(3 * 8, device="cuda")

            def steps():
                ps.copy_(p0)
                bs.copy_(b0)
                ms.zero_()
                bls.local_step(ctx, model, ps, bs, ms, dx, dy, sel, 8, 3, 0.05, 0.9, 1e-4, ls)

            def result():
                stream.synchronize()
                return [t.cpu().numpy().copy() for t in (ps, bs, ms, ls)]

            steps()
            eager = result()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                steps()
            for _ in range(3):
                for t in (ps, bs, ms, ls):
                    t.fill_(-1.0)
                graph.replay()
                replayed = result()
                steps()
                again = result()
                for e, r, a in zip(eager, replayed, again):
                    np.testing.assert_array_equal(r, e)
                    np.testing.assert_array_equal(a, e)
            del graph
        finally:
            ctx.close()
