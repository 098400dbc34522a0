"""The tiles of 192 columns whose wave groups take the two halves of every K-step, at the sizes where a tile can go wrong (test_gpu_gemm_tiles.py), and in every epilogue: Q, K and V with and
without slots and for two branches, the single-stream blocks' joint product, the gated residual, the activation, the velocity step, both storage types, odd widths and rows out of
alignment, one K split and two.  224 x 192 does not fit into LDS when the groups exchange their sums and does it in two turns.
For the epilogues every row of a weight holds one value, at a K of its own: sums are exact then, and whatever the tile all results are the same bits as those of the smallest tile."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg
from test_gpu_gemm_tiles import TILES, ctx, test_tile_edges  # noqa: F401 (the fixture and the check)

pytestmark = pytest.mark.gpu
KG_TILES = {266: (192, 192), 276: (224, 192)}
PLANS = [(222, 1)] + [(tile, splits) for tile in sorted(KG_TILES) for splits in (1, 2)]
del test_tile_edges


@pytest.mark.parametrize("tile", sorted(KG_TILES))
def test_tile_edges_of_half_steps(ctx, tile, monkeypatch):
    import test_gpu_gemm_tiles as tiles
    monkeypatch.setitem(tiles.TILES, tile, KG_TILES[tile])
    tiles.test_tile_edges(ctx, tile)


class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, k=1.0):
        return torch.empty(shape, device="cuda").normal_(generator=self.g) * k

    def weight(self, n, k):
        """[n, k] bf16, one value a row"""
        w = torch.zeros((n, k), device="cuda")
        at = torch.randint(k, (n, 1), generator=self.g, device="cuda")
        return w.scatter_(1, at, self.normal(n, 1)).to(torch.bfloat16)


def _same(results):
    assert all(torch.isfinite(t.float()).all() for t in results[0]) and float(results[0][0].float().abs().max()) > 0
    for plan, other in zip(PLANS[1:], results[1:]):
        for i, (a, b) in enumerate(zip(results[0], other)):
            assert torch.equal(a, b), (plan, i)


@pytest.mark.parametrize("kind,flags,n_txt,branches", [("double", rg.FLAG_STORE, 193, 1), ("double", rg.FLAG_RETRIEVE, 0, 2), ("double", rg.FLAG_RETRIEVE, 40, 1), ("double", 0, 0, 1),
                                                       ("single", rg.FLAG_STORE, 0, 2), ("single", rg.FLAG_RETRIEVE, 0, 1)])
@pytest.mark.parametrize("hidden,mlp,n", [(256, 320, 191), (256, 448, 450), (320, 192, 225)])
@pytest.mark.parametrize("h_dtype", [rg.BF16, rg.FP32])
def test_blocks(kind, flags, n_txt, branches, hidden, mlp, n, h_dtype):
    r = _Draws(hidden + n + n_txt)
    n, heads = n + n_txt, hidden // 64
    n_all = n if flags != rg.FLAG_RETRIEVE else n + 70
    ctx = rg.Context(hidden, heads, 64, mlp, branches * n, 16)
    shapes = {"w_qkv": (3 * hidden, hidden), "w_o": (hidden, hidden), "w_1": (mlp, hidden), "w_2": (hidden, mlp)} if kind == "double" else \
             {"w_1": (3 * hidden + mlp, hidden), "w_2": (hidden, hidden + mlp)}
    bw, held = rg.BlockWeights(), []
    for stream in ("txt", "img"):
        t = {}
        for name, (a, b) in shapes.items():
            t[name], t["b" + name[1:]] = rg.pack_weight(ctx, r.weight(a, b)), r.normal(a)
        for i in (1, 2):
            t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = r.normal(hidden, k=0.1), r.normal(hidden, k=0.1), r.normal(hidden)
        held.append(t)
        setattr(bw, stream, rg.make_stream_weights(t))
    h = r.normal(branches * n, hidden).to(torch.bfloat16 if h_dtype == rg.BF16 else torch.float32)
    slots = torch.randperm(n_all, device="cuda", generator=r.g)[:n].to(torch.int32).contiguous()
    k0, v0 = (r.normal(branches * n_all, hidden).to(torch.bfloat16) for _ in range(2))
    results = []
    for plan in PLANS:
        out, k, v = torch.full((branches * n + 1, hidden), 7.0, dtype=h.dtype, device="cuda"), k0.clone(), v0.clone()
        rg.regione_tune_gemm(ctx, *plan)
        rg.regione_block_forward_batched(ctx, bw, rg.BLOCK_DOUBLE if kind == "double" else rg.BLOCK_SINGLE, h, out, h_dtype, branches, n, n_txt, slots if flags else None, 0,
                                         k if flags else None, v if flags else None, n_all if flags else 0, flags)
        results.append((out, k, v))
    torch.cuda.synchronize()
    ctx.close()
    assert bool((results[0][0][branches * n] == 7).all()) and (not flags) == torch.equal(results[0][1], k0)
    _same(results)


@pytest.mark.parametrize("channels", [65, 136, 191, 200, 388])
@pytest.mark.parametrize("n", [191, 225, 450])
@pytest.mark.parametrize("dtype", [rg.BF16, rg.FP32])
def test_velocity_head(channels, n, dtype):
    r = _Draws(channels + n)
    hidden, total, dt = 320, n + 30, torch.bfloat16 if dtype == rg.BF16 else torch.float32
    ctx = rg.Context(hidden, 5, 64, 64, n, 16)
    w, b, h = rg.pack_weight(ctx, r.weight(channels, hidden)), r.normal(channels), r.normal(n, hidden).to(torch.bfloat16)
    x = r.normal(n, channels).to(dt)
    index = torch.randperm(total, device="cuda", generator=r.g)[:n].to(torch.int32).contiguous()
    results = []
    for plan in PLANS:
        v, ca, full = (torch.full((rows, channels), 7.0, dtype=dt, device="cuda") for rows in (n + 1, n + 1, total))
        xe = torch.cat([x, torch.full((1, channels), 7.0, dtype=dt, device="cuda")])
        rg.regione_tune_gemm(ctx, *plan)
        rg.regione_velocity_head(ctx, h, w, b, n, channels, hidden, 0.04, v, ca, xe, full, index, dtype)
        results.append((v, ca, xe, full))
    torch.cuda.synchronize()
    ctx.close()
    assert all(bool((t[n] == 7).all()) for t in results[0][:3]) and torch.equal(results[0][0], results[0][1]) and torch.equal(results[0][3][index.long()], results[0][2][:n])
    _same(results)


@pytest.mark.parametrize("act", [rg.ACT_NONE, rg.ACT_GELU_TANH])
@pytest.mark.parametrize("out_dtype", [rg.BF16, rg.FP32])
@pytest.mark.parametrize("m", [191, 193, 223, 225])
def test_linear_out_of_alignment(m, out_dtype, act):
    r = _Draws(m)
    k, dt = 320, torch.bfloat16 if out_dtype == rg.BF16 else torch.float32
    ctx = rg.Context(256, 4, 64, 1024, 1024, 16)
    x = r.normal(m, k).to(torch.bfloat16)
    for n, start in ((191, 0), (192, 1), (193, 0), (194, 3), (200, 0), (385, 2)):
        w, b = rg.pack_weight(ctx, r.weight(n, k)), r.normal(n)
        results = []
        for plan in PLANS:
            buf = torch.full((start + m * n + 16,), 7.0, dtype=dt, device="cuda")
            rg.regione_tune_gemm(ctx, *plan)
            rg.regione_linear(ctx, x, w, b, m, n, k, act, out_dtype, buf[start:])
            results.append((buf,))
        torch.cuda.synchronize()
        assert bool((results[0][0][:start] == 7).all()) and bool((results[0][0][start + m * n:] == 7).all())
        _same(results)
    ctx.close()
