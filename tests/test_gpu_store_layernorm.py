"""LayerNorms of forwards that store K and V: one wave per row whatever its length, in kernels for as many rounds of 512 values as the row has.  The stored rows against float64."""
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
