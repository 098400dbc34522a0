"""E4M3 blocks of one group of rows, whose attention result is quantised by the launch that merges its key ranges (head dimension 128) or by the quantiser: one query to more than a query
tile, few and many heads, few keys (one range) and many.  Codes and scales are the quantiser's on the attention's rows bit for bit, and the block gives the same bits whether or not
the rows are handed out."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,d", [(2, 128), (9, 128), (24, 128), (32, 128), (4, 64)])
@pytest.mark.parametrize("n,n_all", [(1, 700), (33, 64), (205, 4608), (300, 4608), (820, 4608), (4608, 4608)])
def test_codes(heads, d, n, n_all):
    hidden, mlp = heads * d, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(heads + n)
    rnd = lambda *s, k=1.0: torch.empty(s, device="cuda").normal_(generator=g) * k
    ctx = rg.Context(hidden, heads, d, mlp, n, 16)
    raw = {"w_qkv": rnd(3 * hidden, hidden, k=0.05), "w_o": rnd(hidden, hidden, k=0.05), "w_1": rnd(mlp, hidden, k=0.05), "w_2": rnd(hidden, mlp, k=0.05)}
    raw = {k: v.to(torch.bfloat16) for k, v in raw.items()}
    t = {"b_qkv": rnd(3 * hidden), "b_o": rnd(hidden), "b_1": rnd(mlp), "b_2": rnd(hidden)}
    for i in (1, 2):
        t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = rnd(hidden, k=0.1), rnd(hidden, k=0.1), rnd(hidden)
    bw, w8 = rg.BlockWeights(), rg.BlockWeightsFp8()
    bw.img = rg.make_stream_weights(t)
    w8.img, held = rg.make_stream_weights_fp8(ctx, raw)
    h = rnd(n, hidden).to(torch.bfloat16)
    k, v = (rnd(n_all, heads, d).to(torch.bfloat16) for _ in range(2))
    slots = torch.randperm(n_all, device="cuda", generator=g)[:n].sort().values.to(torch.int32).contiguous()
    attn = torch.zeros((n, hidden), dtype=torch.bfloat16, device="cuda")
    codes, want = (torch.full((n + 1, hidden), 0x55, dtype=torch.uint8, device="cuda") for _ in range(2))
    scale, want_scale = (torch.full((n + 1,), -1.0, device="cuda") for _ in range(2))
    taps = rg.Fp8Taps()
    taps.attn, taps.a_codes, taps.a_scale = attn.data_ptr(), codes.data_ptr(), scale.data_ptr()
    outs = []
    for tap in (taps, None, taps):
        out = torch.zeros_like(h)
        rg.regione_block_forward_fp8(ctx, bw, w8, rg.BLOCK_DOUBLE, h, out, rg.BF16, n, 0, slots, 0, k, v, n_all, rg.FLAG_RETRIEVE, tap)
        outs.append(out)
    rg.regione_quantize_rows_fp8(ctx, attn, n, hidden, want, want_scale)
    torch.cuda.synchronize()
    ctx.close()
    assert bool(torch.isfinite(outs[0].float()).all()) and float(attn.float().abs().max()) > 0
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert torch.equal(codes, want) and torch.equal(scale, want_scale)
