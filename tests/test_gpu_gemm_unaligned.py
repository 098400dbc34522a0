"""Results whose rows are not 16-byte aligned (odd widths, tensors that start inside a piece) hold the same bits as aligned ones,
in bf16 and float32, with and without the activation and with K splits, and nothing beyond them is written."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [222, 426, 244, 44])
@pytest.mark.parametrize("out_dtype", [rg.BF16, rg.FP32])
def test_rows_out_of_alignment(tile, out_dtype):
    m, k, wide = 70, 320, 168
    g = torch.Generator(device="cuda")
    g.manual_seed(tile)
    r = lambda *shape: torch.empty(shape, device="cuda").normal_(generator=g)
    x, w, b = r(m, k).to(torch.bfloat16), r(wide, k).to(torch.bfloat16), r(wide)
    ctx = rg.Context(256, 4, 64, 1024, 128, 16)
    dt = torch.bfloat16 if out_dtype == rg.BF16 else torch.float32
    for act in (rg.ACT_NONE, rg.ACT_GELU_TANH):
        for splits in (1, 2):
            rg.regione_tune_gemm(ctx, tile, splits)
            want = torch.zeros((m, wide), dtype=dt, device="cuda")
            rg.regione_linear(ctx, x, rg.pack_weight(ctx, w), b, m, wide, k, act, out_dtype, want)
            for n, start in ((wide, 1), (wide, 3), (wide - 1, 0), (wide - 3, 5), (wide - 8, 2), (97, 0), (98, 7), (100, 0), (66, 1)):
                buf = torch.full((start + m * n + 16,), 7.0, dtype=dt, device="cuda")
                rg.regione_linear(ctx, x, rg.pack_weight(ctx, w[:n]), b, m, n, k, act, out_dtype, buf[start:])
                torch.cuda.synchronize()
                assert torch.equal(buf[start:start + m * n].view(m, n), want[:, :n]), (act, splits, n, start)
                assert torch.all(buf[:start] == 7.0) and torch.all(buf[start + m * n:] == 7.0), (act, splits, n, start)
    ctx.close()
