"""The small launches of a float32 context: key ranges that several workgroups share (one and more queries, whole and partly filled query tiles and key groups, fresh rows, cache rows
and index lists, both head dimensions), and LayerNorms that the product behind them takes along, around the edges of where it does.  The reference is float64."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,d", [(4, 64), (2, 128), (24, 64)])
@pytest.mark.parametrize("n_q,n_fresh,n_cache,listed", [(1, 0, 97, False), (16, 16, 180, False), (17, 17, 544, True), (36, 0, 544, False), (128, 100, 700, True), (65, 0, 191, False)])
def test_attention_in_key_ranges(heads, d, n_q, n_fresh, n_cache, listed):
    g = torch.Generator(device="cuda")
    g.manual_seed(n_q + n_cache + d)
    rnd = lambda n: torch.empty((n, heads, d), device="cuda").normal_(generator=g)
    ctx = rg.Context(heads * d, heads, d, 256, 160, 16, compute_dtype=rg.FP32)
    q, kf, vf, k, v = rnd(n_q), rnd(n_fresh), rnd(n_fresh), rnd(n_cache), rnd(n_cache)
    index = torch.randperm(n_cache, device="cuda", generator=g)[:n_cache - 30].to(torch.int32).contiguous() if listed else None
    outs = []
    for _ in range(3):                       # the arrival counters are zero again after each call
        out = torch.zeros_like(q)
        rg.regione_attn_kvcache(ctx, q, n_q, kf if n_fresh else None, vf if n_fresh else None, n_fresh, k, v, n_cache, index, 0 if index is None else index.numel(), heads, d, 0.0, out)
        outs.append(out)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    rows = slice(None) if index is None else index.long()
    kk, vv = torch.cat([kf, k[rows]]).double(), torch.cat([vf, v[rows]]).double()
    s = torch.einsum("qhd,khd->hqk", q.double().cpu(), kk.cpu()) / d ** 0.5
    p = torch.softmax(s, -1)
    want = torch.einsum("hqk,khd->qhd", p, vv.cpu())
    # scores carry 2^-24 of the sum of their products' magnitudes (below 2 d here), weights that as a relative error, twice; sums of weights and products a few roundings more
    size = torch.einsum("hqk,khd->qhd", p, vv.abs().cpu())
    assert torch.all((outs[0].double().cpu() - want).abs() <= size * (4 * d ** 0.5 + 16) * 2.0 ** -23)


@pytest.mark.parametrize("hidden,mlp,n", [(256, 128, 1), (256, 128, 17), (256, 1024, 36), (256, 1024, 64), (256, 1024, 130), (256, 1024, 420), (512, 128, 33), (576, 128, 33), (128, 64, 5)])
def test_block_with_layernorms_in_its_products(hidden, mlp, n):
    heads = hidden // 64
    g = torch.Generator(device="cuda")
    g.manual_seed(hidden + n)
    rnd = lambda *s, k=1.0: torch.empty(s, device="cuda").normal_(generator=g) * k
    ctx = rg.Context(hidden, heads, 64, mlp, n, 16, compute_dtype=rg.FP32)
    t = {"w_qkv": rnd(3 * hidden, hidden, k=0.05), "w_o": rnd(hidden, hidden, k=0.05), "w_1": rnd(mlp, hidden, k=0.05), "w_2": rnd(hidden, mlp, k=0.05),
         "b_qkv": rnd(3 * hidden), "b_o": rnd(hidden), "b_1": rnd(mlp), "b_2": rnd(hidden)}
    for i in (1, 2):
        t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = rnd(hidden, k=0.1), rnd(hidden, k=0.1), rnd(hidden)
    bw = rg.BlockWeights()
    packed = {k: (rg.pack_weight(ctx, v) if k.startswith("w_") else v) for k, v in t.items()}
    bw.img = rg.make_stream_weights(packed)
    h = rnd(n, hidden)
    out = torch.zeros_like(h)
    rg.regione_block_forward(ctx, bw, rg.BLOCK_DOUBLE, h, out, rg.FP32, n, 0, None, 0, None, None, 0, 0)
    torch.cuda.synchronize()
    ctx.close()
    w = {k: v.double().cpu() for k, v in t.items()}
    ln = lambda x, i: torch.nn.functional.layer_norm(x, (hidden,), eps=1e-6) * (1 + w[f"scale{i}"]) + w[f"shift{i}"]
    x = h.double().cpu()
    q, k, v = (y.view(n, heads, 64).transpose(0, 1) for y in (ln(x, 1) @ w["w_qkv"].T + w["b_qkv"]).split(hidden, 1))
    a = (torch.softmax(q @ k.transpose(1, 2) / 8.0, -1) @ v).transpose(0, 1).reshape(n, hidden)
    h1 = x + w["gate1"] * (a @ w["w_o"].T + w["b_o"])
    m = torch.nn.functional.gelu(ln(h1, 2) @ w["w_1"].T + w["b_1"], approximate="tanh")
    want = h1 + w["gate2"] * (m @ w["w_2"].T + w["b_2"])
    # float32 throughout: the tolerance of the float32 context (1e-4 absolute on values of this size), relative to the largest value
    assert (out.double().cpu() - want).abs().max() <= 1e-5 * want.abs().max()
