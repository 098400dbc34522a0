"""LayerNorms of forwards that store K and V: one wave per row whatever its length, in kernels for as many rounds of 512 values as the row has.  The stored rows against float64, and bit for
bit against the order of sums that they are meant to keep."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_dtype", [rg.BF16, rg.FP32])
@pytest.mark.parametrize("hidden,n", [(1024, 300), (1152, 65), (2048, 64), (2176, 33), (3072, 257), (3200, 5), (4096, 130)])
def test_stored_rows(hidden, n, h_dtype):
    heads, d, mlp = hidden // 128, 128, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(hidden + n)
    rnd = lambda *s, k=1.0: torch.empty(s, device="cuda").normal_(generator=g) * k
    ctx = rg.Context(hidden, heads, d, mlp, n, 16)
    raw = {"w_qkv": rnd(3 * hidden, hidden, k=0.05), "w_o": rnd(hidden, hidden, k=0.05), "w_1": rnd(mlp, hidden, k=0.05), "w_2": rnd(hidden, mlp, k=0.05)}
    raw = {k: v.to(torch.bfloat16) for k, v in raw.items()}
    t = {k: rg.pack_weight(ctx, v) for k, v in raw.items()}
    t.update({"b_qkv": rnd(3 * hidden), "b_o": rnd(hidden), "b_1": rnd(mlp), "b_2": rnd(hidden)})
    for i in (1, 2):
        t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = rnd(hidden, k=0.1), rnd(hidden, k=0.1), rnd(hidden)
    bw = rg.BlockWeights()
    bw.img = rg.make_stream_weights(t)
    h = rnd(n, hidden) + 3.0
    h = h.to(torch.bfloat16) if h_dtype == rg.BF16 else h
    out = torch.zeros_like(h)
    k, v = (torch.full((n + 1, heads, d), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    slots = torch.arange(n, dtype=torch.int32, device="cuda")
    rg.regione_block_forward(ctx, bw, rg.BLOCK_DOUBLE, h, out, h_dtype, n, 0, slots, 0, k, v, n, rg.FLAG_STORE)
    torch.cuda.synchronize()
    ctx.close()
    u = torch.nn.functional.layer_norm(h.double(), (hidden,), eps=1e-6) * (1 + t["scale1"].double()) + t["shift1"].double()
    for part, got in ((1, k), (2, v)):
        w, b = raw["w_qkv"][part * hidden:(part + 1) * hidden].double(), t["b_qkv"][part * hidden:(part + 1) * hidden].double()
        want, size = u @ w.T.contiguous() + b, u.abs() @ w.abs().T.contiguous()
        # a row value is rounded to bf16 once (2^-9 of it), the sums are float32, the result is rounded to bf16
        bound = size * (2.0 ** -9 * 1.01 + hidden * 2.0 ** -24) + want.abs() * 2.0 ** -8
        assert bool((got[n] == 7).all())
        assert bool(((got[:n].reshape(n, hidden).double() - want).abs() <= bound).all())
    assert bool(torch.isfinite(out.float()).all())


def _fma(a, b, c):
    """float32 a * b + c with one rounding (but for double roundings, one in 2^29)"""
    return (a.double() * b.double() + c.double()).float()


def _wave_layernorm(h, shift, scale):
    """LayerNorm + modulation as a wave of 64 lanes forms it: groups of eight values dealt to the lanes in turn, every lane's sums in the order of its values, then partners 32, 16, 8, 4, 2
    and 1 lanes away.  Three results: the reciprocal square root of the GPU is within one unit in the last place of the exact one, so with that and with its two neighbours."""
    n, hidden = h.shape
    rounds = -(-hidden // 512)
    live = (torch.arange(512 * rounds, device=h.device) < hidden).view(rounds, 64, 8)
    x = torch.zeros((n, 512 * rounds), device=h.device)
    x[:, :hidden] = h.float()
    x = x.view(n, rounds, 64, 8)

    def total(term):
        s = torch.zeros((n, 64), device=h.device)
        for i in range(rounds):
            for e in range(8):
                s = torch.where(live[i, :, e], term(s, x[:, i, :, e]), s)
        lanes = torch.arange(64, device=h.device)
        for partner in (32, 16, 8, 4, 2, 1):
            s = s + s[:, lanes ^ partner]
        assert torch.equal(s, s[:, :1].expand(n, 64))
        return s[:, :1]

    mean = (total(lambda s, v: s + v).double() / hidden).float()
    squares = total(lambda s, v: _fma(v - mean, v - mean, s))
    exact = (1.0 / ((squares.double() / hidden).float() + torch.tensor(1e-6, device=h.device)).double().sqrt()).float()
    results = []
    for rstd in (exact, torch.nextafter(exact, exact * 2), torch.nextafter(exact, exact * 0)):
        y = (h.float() - mean) * rstd
        results.append(_fma(y, 1.0 + scale, shift.expand_as(y)).to(torch.bfloat16))
    return results


@pytest.mark.parametrize("h_dtype", [rg.BF16, rg.FP32])
@pytest.mark.parametrize("hidden,n", [(1152, 1024), (2048, 1200), (3072, 820), (3072, 2048), (4096, 515)])
def test_stored_bits(hidden, n, h_dtype):
    """K and V are those of the wave's LayerNorm and of the tile and K splits that regione_gemm_plan_host names for them; the LayerNorm of several waves, or its own tile, gives other bits."""
    heads, mlp = hidden // 128, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(hidden + n)
    rnd = lambda *s, k=1.0: torch.empty(s, device="cuda").normal_(generator=g) * k
    ctx = rg.Context(hidden, heads, 128, mlp, n, 16)
    shapes = {"w_qkv": (3 * hidden, hidden), "w_o": (hidden, hidden), "w_1": (mlp, hidden), "w_2": (hidden, mlp)}
    t = {name: rg.pack_weight(ctx, rnd(*shape, k=0.05).to(torch.bfloat16)) for name, shape in shapes.items()}
    t.update({"b_qkv": rnd(3 * hidden), "b_o": rnd(hidden), "b_1": rnd(mlp), "b_2": rnd(hidden)})
    for i in (1, 2):
        t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = rnd(hidden, k=0.1), rnd(hidden, k=0.1), rnd(hidden)
    bw = rg.BlockWeights()
    bw.img = rg.make_stream_weights(t)
    h = (rnd(n, hidden) + 3.0).to(torch.bfloat16 if h_dtype == rg.BF16 else torch.float32)
    k, v = (torch.zeros((n, hidden), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    rg.regione_block_forward(ctx, bw, rg.BLOCK_DOUBLE, h, torch.zeros_like(h), h_dtype, n, 0, torch.arange(n, dtype=torch.int32, device="cuda"), 0, k, v, n, rg.FLAG_STORE)
    stored = torch.cat([k, v], 1)

    def projected(u):
        rg.regione_tune_gemm(ctx, *rg.regione_gemm_plan_host(n, 3 * hidden, hidden, rg.GEMM_BF16_STORED))
        y = torch.zeros((n, 3 * hidden), dtype=torch.bfloat16, device="cuda")
        rg.regione_linear(ctx, u, t["w_qkv"], t["b_qkv"], n, 3 * hidden, hidden, rg.ACT_NONE, rg.BF16, y)
        rg.regione_tune_gemm(ctx, 0, 0)
        return y[:, hidden:]

    same = torch.stack([(stored == projected(u)).all(1) for u in _wave_layernorm(h, t["shift1"], t["scale1"])])
    wide = torch.zeros((n, hidden), dtype=torch.bfloat16, device="cuda")
    rg.regione_layernorm(ctx, h, h_dtype, n, hidden, t["shift1"], t["scale1"], wide)
    other = (stored == projected(wide)).all(1)
    torch.cuda.synchronize()
    ctx.close()
    print("rows that are the wave's:", same.sum(1).tolist(), "several waves':", int(other.sum()), "of", n)
    assert bool(same.any(0).all())
    assert not bool(other.all())
