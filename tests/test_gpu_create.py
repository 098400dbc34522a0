"""Creating a context waits for no work that is under way on the device and is possible while a stream is captured (relaxed mode)."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


def test_create_does_not_wait_for_other_streams():
    rg.Context(256, 4, 64, 1024, 64, 256).close()            # the library and the device are up
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(other):
        torch.cuda._sleep(400_000_000)                         # some 0.2 s
        done.record(other)
    ctx = rg.Context(256, 4, 64, 1024, 64, 256, stream=mine)
    waited = done.query()
    torch.cuda.synchronize()
    ctx.close()
    assert not waited


@pytest.mark.parametrize("on_default_stream", [False, True])
def test_create_during_a_relaxed_capture(on_default_stream):
    m, n, k = 70, 130, 512
    x, w = torch.randn((m, k), device="cuda").to(torch.bfloat16), torch.randn((n, k), device="cuda").to(torch.bfloat16)
    captured = torch.cuda.Stream()
    graph, buf = torch.cuda.CUDAGraph(), torch.zeros(16, device="cuda")
    mine = torch.cuda.current_stream() if on_default_stream else captured
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=captured, capture_error_mode="relaxed"):
        buf += 1.0
        ctx = rg.Context(256, 4, 64, 1024, 64, 256, stream=mine)
    plain = rg.Context(256, 4, 64, 1024, 64, 256)
    out = []
    for c in (ctx, plain):
        y = torch.zeros((m, n), device="cuda")
        torch.cuda.synchronize()
        rg.regione_tune_gemm(c, 222, 3)                      # K splits: finished through the counters that were cleared at creation
        rg.regione_linear(c, x, rg.pack_weight(plain, w), None, m, n, k, rg.ACT_NONE, rg.FP32, y)
        torch.cuda.synchronize()
        out.append(y)
        c.close()
    assert torch.equal(out[0], out[1]) and float(out[0].abs().max()) > 0.0
    for i in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.all(buf == i + 1.0)
