"""Double-stream blocks whose text and image products share launches.  With the same weights for both streams it does not matter where the rows are split: every split gives the bits of
the block that has image rows only, whose products are launches of one product.  Rows around the edges of the 16-row tiles and of the sizes up to which products are paired."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [rg.BF16, rg.FP32])
@pytest.mark.parametrize("hidden,heads,mlp", [(256, 4, 1024), (512, 8, 320), (1024, 8, 4096), (1152, 9, 256)])
@pytest.mark.parametrize("n,splits", [(2, (1,)), (33, (1, 16, 17, 32)), (130, (15, 64)), (352, (64, 333))])
def test_any_split(dtype, hidden, heads, mlp, n, splits):
    g = torch.Generator(device="cuda")
    g.manual_seed(hidden + n)
    rnd = lambda *s, k=1.0: torch.empty(s, device="cuda").normal_(generator=g) * k
    ctx = rg.Context(hidden, heads, hidden // heads, mlp, n, 16, compute_dtype=dtype)
    t = {"w_qkv": rnd(3 * hidden, hidden, k=0.05), "w_o": rnd(hidden, hidden, k=0.05), "w_1": rnd(mlp, hidden, k=0.05), "w_2": rnd(hidden, mlp, k=0.05),
         "b_qkv": rnd(3 * hidden), "b_o": rnd(hidden), "b_1": rnd(mlp), "b_2": rnd(hidden)}
    t = {k: rg.pack_weight(ctx, v.to(ctx.torch_dtype)) if k.startswith("w_") else v for k, v in t.items()}
    for i in (1, 2):
        t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = rnd(hidden, k=0.1), rnd(hidden, k=0.1), rnd(hidden)
    copy = {k: v.clone() for k, v in t.items()}
    bw = rg.BlockWeights()
    bw.txt, bw.img = rg.make_stream_weights(copy), rg.make_stream_weights(t)
    h = rnd(n, hidden)
    outs = []
    for n_txt in (0,) + splits:
        if n_txt and rg.regione_block_lanes_host(n_txt, n - n_txt, hidden, mlp, dtype) != 1:
            continue
        out = torch.full((n + 1, hidden), 7.0, device="cuda")
        rg.regione_block_forward(ctx, bw, rg.BLOCK_DOUBLE, h, out, rg.FP32, n, n_txt, None, 0, None, None, 0, 0)
        outs.append(out)
    torch.cuda.synchronize()
    ctx.close()
    assert bool(torch.isfinite(outs[0]).all()) and bool((outs[0][n] == 7).all())
    # larger products take their sums in an order that depends on the rows: there the roundings to bf16 between the products decide
    products = [(3 * hidden, hidden), (hidden, hidden), (mlp, hidden), (hidden, mlp)]
    small = all((n + 63) // 64 * ((o + 63) // 64) < 256 if dtype == rg.FP32 else rg.regione_gemm_plan_host(n, o, i, 0)[0] == 0 for o, i in products)
    for out in outs[1:]:
        if small:
            assert torch.equal(out, outs[0])
        else:
            assert (out - outs[0]).norm() <= 4 * 2.0 ** -8 * outs[0].norm() and bool((out[n] == 7).all())
