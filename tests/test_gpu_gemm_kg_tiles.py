"""The tiles of 192 columns whose wave groups take the two halves of every K-step, at the sizes where a tile can go wrong (test_gpu_gemm_tiles.py), and
in every epilogue that a block uses: 224 x 192 does not fit
into LDS when the groups exchange their sums and does it in two turns."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg
from test_gpu_gemm_tiles import TILES, ctx, test_tile_edges  # noqa: F401 (the fixture and the check)

pytestmark = pytest.mark.gpu
KG_TILES = {266: (192, 192), 276: (224, 192)}
del test_tile_edges


@pytest.mark.parametrize("tile", sorted(KG_TILES))
def test_tile_edges_of_half_steps(ctx, tile, monkeypatch):
    import test_gpu_gemm_tiles as tiles
    monkeypatch.setitem(tiles.TILES, tile, KG_TILES[tile])
    tiles.test_tile_edges(ctx, tile)
