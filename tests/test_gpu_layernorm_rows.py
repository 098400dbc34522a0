"""LayerNorm + modulation around the edges of the kernel that reads a row in 16-byte groups: one group, whole and partly filled rounds of 64 lanes, one, two and more of them, the longest
row, and rows that only the kernel for any width takes; bf16 and float32 in and out, tensors off the 16-byte grid.  The oracle is float64."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f32_ctx", [False, True])
@pytest.mark.parametrize("f32_in", [False, True])
@pytest.mark.parametrize("n,hidden,shifted", [(1, 8, 0), (3, 256, 0), (5, 520, 0), (3, 1024, 0), (5, 1032, 0), (2, 4096, 0), (4, 4104, 0), (3, 100, 0), (6, 512, 1)])
def test_rows(f32_ctx, f32_in, n, hidden, shifted):
    g = torch.Generator(device="cuda")
    g.manual_seed(hidden + n)
    t_in, t_out = (torch.float32 if f else torch.bfloat16 for f in (f32_in, f32_ctx))
    h = torch.empty(n * hidden + shifted, dtype=t_in, device="cuda").normal_(generator=g)[shifted:].view(n, hidden)
    shift, scale = (torch.empty(hidden, dtype=torch.float32, device="cuda").normal_(generator=g) for _ in range(2))
    ctx = rg.Context(256, 4, 64, 256, 16, 16, compute_dtype=rg.FP32 if f32_ctx else rg.BF16)
    u = torch.full((n + 1, hidden), 7.0, dtype=t_out, device="cuda")
    rg.regione_layernorm(ctx, h, rg.FP32 if f32_in else rg.BF16, n, hidden, shift, scale, u)
    torch.cuda.synchronize()
    ctx.close()
    x = h.double()
    y = (x - x.mean(1, keepdim=True)) / torch.sqrt(x.var(1, unbiased=False, keepdim=True) + 1e-6)
    want = y * (1 + scale.double()) + shift.double()
    # float32 throughout: sums of at most 4104 terms in 64 chains, a handful of roundings; then one rounding to bf16
    size = y.abs() * (1 + scale.double().abs()) + (1 + scale.double().abs()) + shift.double().abs()
    bound = size * 2.0 ** -20 + (0 if f32_ctx else want.abs() * 2.0 ** -8)
    assert torch.all((u[:n].double() - want).abs() <= bound)
    assert torch.all(u[n] == 7.0)
