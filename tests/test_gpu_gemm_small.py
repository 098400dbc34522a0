"""The kernel of 16-row tiles: products of few rows and narrow results at the edges of its tiles, its K dealing and its range, and products that take their
rows before the LayerNorm, against float32 products of the same bf16 operands and against the tile kernels."""
import numpy as np
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [
    (1, 1, 64), (15, 33, 64), (16, 64, 128), (17, 65, 192), (36, 256, 1024), (33, 96, 320), (100, 520, 704), (544, 768, 256), (820, 64, 3072), (2049, 64, 576),
    (5000, 63, 64), (16, 3072, 3072), (70, 1000, 5120), (160, 1024, 1024), (255, 129, 2048), (160, 1024, 1792),
])
def test_products(m, n, k):
    assert rg.regione_gemm_plan_host(m, n, k, rg.GEMM_BF16) == (0, 1)        # the kernel in question
    rng = np.random.default_rng(m + n + k)
    up = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16).cuda()
    x, w = up(rng.standard_normal((m, k))), up(rng.standard_normal((n, k)))
    b = torch.from_numpy(rng.standard_normal(n).astype(np.float32)).cuda()
    ctx = rg.Context(256, 4, 64, 1024, 64, 16)
    packed = rg.pack_weight(ctx, w)
    y = [torch.full((m + 1, n), 7.0, dtype=torch.float32, device="cuda") for _ in range(3)]
    rg.regione_linear(ctx, x, packed, b, m, n, k, rg.ACT_NONE, rg.FP32, y[0])
    rg.regione_linear(ctx, x, packed, b, m, n, k, rg.ACT_NONE, rg.FP32, y[1])
    rg.regione_tune_gemm(ctx, 222, 1)
    rg.regione_linear(ctx, x, packed, b, m, n, k, rg.ACT_NONE, rg.FP32, y[2])
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(y[0], y[1]) and torch.all(y[0][m] == 7.0)
    scale = x.float().norm(dim=1, keepdim=True) * w.float().norm(dim=1)       # |error| of a float32 sum of k products <= k 2^-24 |x| |w|, far less in practice
    want = x.double() @ w.double().T.contiguous() + b
    for got in (y[0], y[2]):
        assert torch.all((got[:m].double() - want).abs() <= 2.0 ** -20 * scale + 2.0 ** -22 * want.abs() + 1e-6)


@pytest.mark.parametrize("kind", ["double", "single"])
@pytest.mark.parametrize("hidden,heads,d,mlp,n", [(256, 4, 64, 1024, 1), (256, 4, 64, 1024, 37), (256, 4, 64, 1024, 544), (1024, 8, 128, 4096, 17), (1024, 8, 128, 4096, 100), (128, 2, 64, 192, 50),
                                                   (256, 4, 64, 1024, 300), (1024, 8, 128, 4096, 60)])     # one round of tiles of 64 columns, full or nearly so
@pytest.mark.parametrize("f32", [False, True])
def test_rows_before_the_layernorm(kind, hidden, heads, d, mlp, n, f32):
    """A block whose products normalise their rows themselves, against the same block with a LayerNorm of its own before tile kernels."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    r = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    ctx = rg.Context(hidden, heads, d, mlp, n, 16)
    shapes = {"w_qkv": (3 * hidden, hidden), "w_o": (hidden, hidden), "w_1": (mlp, hidden), "w_2": (hidden, mlp)} if kind == "double" else \
             {"w_1": (3 * hidden + mlp, hidden), "w_2": (hidden, hidden + mlp)}
    t = {}
    for name, (o, i) in shapes.items():
        t[name], t["b" + name[1:]] = rg.pack_weight(ctx, (0.05 * r(o, i)).to(torch.bfloat16)), 0.05 * r(o)
    for j in (1, 2):
        t[f"shift{j}"], t[f"scale{j}"], t[f"gate{j}"] = 0.1 * r(hidden), 0.1 * r(hidden), 1.0 + 0.1 * r(hidden)
    bw = rg.BlockWeights()
    bw.img = rg.make_stream_weights(t)
    h = (3.0 * r(n, hidden) + 1.0).to(torch.float32 if f32 else torch.bfloat16)
    outs = []
    for plan in ((0, 0), (0, 0), (222, 1)):
        rg.regione_tune_gemm(ctx, *plan)
        out = torch.zeros_like(h)
        rg.regione_block_forward(ctx, bw, rg.BLOCK_DOUBLE if kind == "double" else rg.BLOCK_SINGLE, h, out, rg.FP32 if f32 else rg.BF16, n, 0, None, 0, None, None, 0, 0)
        torch.cuda.synchronize()
        outs.append(out.double())
    ctx.close()
    assert torch.equal(outs[0], outs[1])
    # sums in another order, rounded to bf16 between the stages: a few ulps (2^-8) of what the block adds
    assert float((outs[0] - outs[2]).norm()) <= 2.0 ** -8 * float((outs[2] - h.double()).norm()) + 2.0 ** -9 * float(outs[2].norm()) * (not f32)


@pytest.mark.parametrize("hidden,heads,d,n,launches", [(1024, 8, 128, 30, 0), (1024, 8, 128, 34, 1), (768, 6, 128, 32, 0), (768, 6, 128, 50, 1), (256, 4, 64, 128, 0), (256, 4, 64, 150, 1)])
def test_rows_are_normalised_twice_only_for_one_round(hidden, heads, d, n, launches):
    """A single-stream block of width 768 and 50 rows took 33.2 us with its 336 workgroups in two rounds, each normalising its rows, and 30.0 with a LayerNorm launch."""
    mlp = 4 * hidden
    r = lambda *s: torch.randn(s, device="cuda")
    ctx = rg.Context(hidden, heads, d, mlp, n, 16)
    t = {}
    for name, (o, i) in {"w_1": (3 * hidden + mlp, hidden), "w_2": (hidden, hidden + mlp)}.items():
        t[name], t["b" + name[1:]] = rg.pack_weight(ctx, (0.05 * r(o, i)).to(torch.bfloat16)), 0.05 * r(o)
    t["shift1"], t["scale1"], t["gate1"] = 0.1 * r(hidden), 0.1 * r(hidden), 1.0 + 0.1 * r(hidden)
    bw = rg.BlockWeights()
    bw.img = rg.make_stream_weights(t)
    h = r(n, hidden).to(torch.bfloat16)
    out = torch.empty_like(h)
    rg.regione_profile_enable(ctx, True)
    rg.regione_profile_read(ctx)
    rg.regione_block_forward(ctx, bw, rg.BLOCK_SINGLE, h, out, rg.BF16, n, 0, None, 0, None, None, 0, 0)
    profile = rg.regione_profile_read(ctx)
    ctx.close()
    assert profile["layernorm"][1] == launches and profile["gemm"][1] == 2
