"""The tuning knob of the GEMMs: K splits forced without a tile split the tile that the product gets by itself, in bf16 and in
E4M3, and a number that names no tile is refused at once."""
import numpy as np
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [rg.GEMM_BF16, rg.GEMM_E4M3])
@pytest.mark.parametrize("n", [72, 520])
def test_splits_without_a_tile(kind, n):
    m, k, forced = 70, 1920, 2
    ctx = rg.Context(256, 4, 64, 1024, 128, 16)
    rng = np.random.default_rng(n)
    y = lambda: torch.zeros((m, n), dtype=torch.float32, device="cuda")
    if kind == rg.GEMM_BF16:
        x = torch.from_numpy(rng.standard_normal((m, k)).astype(np.float32)).to(torch.bfloat16).cuda()
        w = rg.pack_weight(ctx, torch.from_numpy(rng.standard_normal((n, k)).astype(np.float32)).to(torch.bfloat16).cuda())
        call = lambda out: rg.regione_linear(ctx, x, w, None, m, n, k, rg.ACT_NONE, rg.FP32, out)
    else:
        # no NaN, and exponents far enough apart that the sums are rounded
        x = torch.from_numpy((rng.integers(0, 256, (m, k)) & 0xF7).astype(np.uint8)).cuda()
        codes = torch.from_numpy((rng.integers(0, 256, (n, k)) & 0xF7).astype(np.uint8)).cuda()
        sx, sw = (torch.from_numpy(rng.uniform(0.5, 1.5, c).astype(np.float32)).cuda() for c in (m, n))
        w = torch.zeros(rg.regione_packed_weight_elems(n, k), dtype=torch.uint8, device="cuda")
        rg.regione_pack_weight_fp8(ctx, codes, n, k, w)
        call = lambda out: rg.regione_linear_fp8(ctx, x, sx, w, sw, None, m, n, k, rg.ACT_NONE, rg.FP32, out)
    tile, own = rg.regione_gemm_plan_host(m, n, k, kind)
    assert own != forced
    out = {}
    for plan in ((0, forced), (tile, forced), (tile, own)):
        out[plan] = y()
        rg.regione_tune_gemm(ctx, *plan)
        call(out[plan])
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(out[0, forced], out[tile, forced])
    assert not torch.equal(out[tile, own], out[tile, forced])      # the split shows in the last bits of the sums


def test_only_tiles_are_taken():
    ctx = rg.Context(256, 4, 64, 1024, 64, 16)
    for code, splits in ((-1, 0), (7, 0), (41, 0), (85, 0), (223, 1), (499, 0), (0, -1), (0, 17)):
        with pytest.raises(rg.RegionEError):
            rg.regione_tune_gemm(ctx, code, splits)
    for code in (0, 1, 6, 42, 54, 84, 222, 242, 284, 436, 446):
        rg.regione_tune_gemm(ctx, code, 1)
    ctx.close()
