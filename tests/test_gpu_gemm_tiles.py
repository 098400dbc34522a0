"""Every tile of the GEMM at the sizes where it can go wrong: one row, a tile's rows and columns less and plus one, the last
32-column block ragged, K of one step, fewer steps than the copies run ahead, and K splits whose last part is short."""
import numpy as np
import pytest
import torch

from paper_2510_25590_amd import binding as rg
from oracle import fp8_reference as f8

pytestmark = pytest.mark.gpu

TILES = {222: (64, 64), 224: (64, 128), 242: (128, 64), 244: (128, 128), 274: (224, 128), 284: (256, 128), 426: (128, 96), 436: (192, 96), 446: (256, 96),
         44: (128, 256), 64: (192, 256), 74: (224, 256), 84: (256, 256)}
TILES_FP8 = {42: (128, 128), 62: (192, 128), 82: (256, 128), 44: (128, 256),
             222: (64, 64), 224: (64, 128), 274: (224, 128), 426: (128, 96), 446: (256, 96),
             54: (160, 256), 64: (192, 256), 74: (224, 256), 84: (256, 256)}


@pytest.fixture(scope="module")
def ctx():
    c = rg.Context(256, 4, 64, 1024, 1024, 16)
    yield c
    c.close()


def _sizes(rows, cols):
    return [(1, cols - 8, 64), (rows - 1, cols + 1, 128), (rows, cols, 192), (rows + 1, 2 * cols + 40, 64 * 5), (2 * rows + 17, cols + 100, 64 * 13)]


@pytest.mark.parametrize("tile", sorted(TILES))
def test_tile_edges(ctx, tile):
    rng = np.random.default_rng(tile)
    for m, n, k in _sizes(*TILES[tile]):
        x = torch.from_numpy(rng.standard_normal((m, k)).astype(np.float32)).to(torch.bfloat16)
        w = torch.from_numpy((rng.standard_normal((n, k)) * 0.05).astype(np.float32)).to(torch.bfloat16)
        b = rng.standard_normal(n).astype(np.float32)
        xd, wd = x.float().numpy().astype(np.float64), w.float().numpy().astype(np.float64)
        want, mag = xd @ wd.T + b, np.abs(xd) @ np.abs(wd).T + np.abs(b)
        wp = rg.pack_weight(ctx, w.cuda())
        xg, bg = x.cuda(), torch.from_numpy(b).cuda()
        for splits in (1, 2, 5):
            if splits > k // 64:
                continue
            runs = []
            rg.regione_tune_gemm(ctx, tile, splits)
            try:
                for _ in range(2):
                    y = torch.full((m + 1, n), 7.0, dtype=torch.float32, device="cuda")
                    rg.regione_linear(ctx, xg, wp, bg, m, n, k, rg.ACT_NONE, rg.FP32, y)
                    runs.append(y.cpu().numpy())
            finally:
                rg.regione_tune_gemm(ctx, 0, 0)
            assert np.array_equal(runs[0], runs[1]), (m, n, k, splits)        # whichever split arrives last
            assert np.all(runs[0][m] == 7.0)
            # exact products, float32 sums of at most 13 x 64 of them: well within 2^-19 of the sum of magnitudes
            assert np.all(np.abs(runs[0][:m] - want) <= mag * 2.0 ** -19 + 1e-30), (m, n, k, splits)


@pytest.mark.parametrize("tile", sorted(TILES_FP8))
def test_fp8_tile_edges(ctx, tile):
    rng = np.random.default_rng(1000 + tile)
    for m, n, k2 in _sizes(*TILES_FP8[tile]):
        k = 2 * k2
        xq = ((rng.integers(0, 256, (m, k)).astype(np.uint8) & 0x87) | 0x30).astype(np.uint8)
        wq = ((rng.integers(0, 256, (n, k)).astype(np.uint8) & 0x87) | 0x28).astype(np.uint8)
        sx, sw = rng.uniform(0.5, 1.5, m).astype(np.float32), rng.uniform(0.5, 1.5, n).astype(np.float32)
        want = f8.linear_fp8(xq, sx, wq, sw)
        mag = (np.abs(f8.e4m3_decode(xq)) @ np.abs(f8.e4m3_decode(wq)).T) * sx[:, None].astype(np.float64) * sw[None, :]
        packed = torch.zeros(rg.regione_packed_weight_elems(n, k), dtype=torch.uint8, device="cuda")
        rg.regione_pack_weight_fp8(ctx, torch.from_numpy(wq).cuda(), n, k, packed)
        for splits in (1, 3):
            if splits > k2 // 64:
                continue
            y = torch.full((m + 1, n), 7.0, dtype=torch.float32, device="cuda")
            rg.regione_tune_gemm(ctx, tile, splits)
            try:
                rg.regione_linear_fp8(ctx, torch.from_numpy(xq).cuda(), torch.from_numpy(sx).cuda(), packed, torch.from_numpy(sw).cuda(), None,
                                      m, n, k, rg.ACT_NONE, rg.FP32, y)
            finally:
                rg.regione_tune_gemm(ctx, 0, 0)
            got = y.cpu().numpy()
            assert np.all(got[m] == 7.0)
            assert np.all(np.abs(got[:m] - want) <= mag * 2.0 ** -11 + 1e-30), (m, n, k, splits)   # the instruction's alignment cut
