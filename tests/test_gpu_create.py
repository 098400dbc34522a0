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


def test_a_small_context_holds_little_attention_scratch():
    """400 rows of 8 heads of 128: the products' 128 MiB, 35 MB of partial rows of attentions and a few MB of rows, not the 69 MB that full chips need."""
    torch.zeros(1, device="cuda")
    rg.Context(1024, 8, 128, 1024, 400, 16).close()          # what the first context sets up for all
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx = rg.Context(1024, 8, 128, 1024, 400, 16)
    held = before - torch.cuda.mem_get_info()[0]
    ctx.close()
    rows = 400 * (4 * 1024 + 2 * 1024 + 1024) * 2 + 400 * 1024 * 4    # u q k v, a, m in bf16; h1 in float32
    assert held <= (128 << 20) + 256 * 2 * 128 * 132 * 4 + rows + (12 << 20)    # and a dozen allocations' rounding to pages


@pytest.mark.parametrize("heads,rows", [(8, 129), (8, 400), (8, 1024), (4, 2048)])
def test_small_contexts_deal_attentions_as_large_ones_do(heads, rows):
    torch.zeros(1, device="cuda")
    small, large = (rg.Context(128 * heads, heads, 128, 256, n, 16) for n in (rows, 4096))
    for n_q in (rows, rows - 1, 3 * rows // 4, rows // 2):
        for n_keys in (65, 129, 400, 801, 1409, 2500, 4097, 6304, 8704, 12000, 19456):
            for source in (rg.KEYS_CONTIGUOUS, rg.KEYS_TWO, rg.KEYS_INDEXED):
                plans = [rg.regione_attention_workgroups(c, n_q, n_keys, heads, 128, source) for c in (small, large)]
                assert plans[0] == plans[1], (n_q, n_keys, source)
    small.close()
    large.close()
