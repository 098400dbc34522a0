"""Double-stream blocks whose text and image rows run on two lanes.  The rule (no GPU needed), and the results: every output row of two blocks in a row, retrieved
and stored keys and values, against the same call on one lane (per-class timing on) and against float64."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

WIDTHS = {512: (4, 128, 2048), 1024: (8, 128, 4096), 3072: (24, 128, 12288)}


@pytest.mark.parametrize("n_txt,n_img,hidden,dtype,lanes", [
    (128, 900, 3072, rg.BF16, 2), (512, 8192, 3072, rg.BF16, 2),
    (512, 820, 3072, rg.BF16, 1), (32, 512, 3072, rg.BF16, 1), (0, 8192, 3072, rg.BF16, 1), (512, 0, 3072, rg.BF16, 1),   # many text rows, little work, one group
    (32, 256, 3072, rg.FP32, 2), (512, 820, 1024, rg.FP32, 2), (512, 2048, 512, rg.FP32, 2),
    (32, 256, 1024, rg.FP32, 1), (64, 512, 512, rg.FP32, 1), (0, 4096, 1024, rg.FP32, 1),
])
def test_rule(n_txt, n_img, hidden, dtype, lanes):
    assert rg.regione_block_lanes_host(n_txt, n_img, hidden, WIDTHS[hidden][2], dtype) == lanes


def test_rule_refuses():
    for bad in ((-1, 4, 256, 1024, rg.BF16), (1, 4, 0, 1024, rg.BF16), (1, 4, 256, 1024, 7)):
        with pytest.raises(rg.RegionEError):
            rg.regione_block_lanes_host(*bad)


def _stream(r, ctx, hidden, mlp):
    raw, t = {}, {}
    for name, (o, i) in {"w_qkv": (3 * hidden, hidden), "w_o": (hidden, hidden), "w_1": (mlp, hidden), "w_2": (hidden, mlp)}.items():
        raw[name] = (0.02 * r(o, i)).to(ctx.torch_dtype)
        t[name], t["b" + name[1:]] = rg.pack_weight(ctx, raw[name]), 0.02 * r(o)
    for j in (1, 2):
        t[f"shift{j}"], t[f"scale{j}"], t[f"gate{j}"] = 0.1 * r(hidden), 0.1 * r(hidden), 1.0 + 0.1 * r(hidden)
    return raw, t


def _block64(streams, x, n_txt, heads, d):
    """One double-stream block in float64 on rows [text | image]."""
    ln = lambda y: (y - y.mean(1, keepdim=True)) / torch.sqrt(y.var(1, unbiased=False, keepdim=True) + 1e-6)
    gelu = lambda y: 0.5 * y * (1 + torch.tanh(0.7978845608028654 * (y + 0.044715 * y ** 3)))
    mm = lambda y, s, name: y @ s[0][name].double().T.contiguous() + s[1]["b" + name[1:]].double()
    vec = lambda s, name: s[1][name].double()
    parts = [(s, y) for s, y in zip(streams, (x[:n_txt], x[n_txt:]))]
    qkv = torch.cat([mm(ln(y) * (1 + vec(s, "scale1")) + vec(s, "shift1"), s, "w_qkv") for s, y in parts])
    q, k, v = qkv.view(x.shape[0], 3, heads, d).unbind(1)
    a = torch.stack([torch.softmax(q[:, h] @ k[:, h].T.contiguous() / d ** 0.5, -1) @ v[:, h].contiguous() for h in range(heads)], 1).flatten(1)
    out = []
    for (s, y), att in zip(parts, (a[:n_txt], a[n_txt:])):
        h1 = y + vec(s, "gate1") * mm(att, s, "w_o")
        out.append(h1 + vec(s, "gate2") * mm(gelu(mm(ln(h1) * (1 + vec(s, "scale2")) + vec(s, "shift2"), s, "w_1")), s, "w_2"))
    return torch.cat(out)


@pytest.mark.gpu
@pytest.mark.parametrize("n_txt,n_img,hidden,dtype", [(128, 900, 3072, rg.BF16), (33, 1001, 3072, rg.BF16), (512, 820, 1024, rg.FP32), (500, 2048, 512, rg.FP32)])
def test_two_lanes(n_txt, n_img, hidden, dtype):
    heads, d, mlp = WIDTHS[hidden]
    n, f32 = n_txt + n_img, dtype == rg.FP32
    assert rg.regione_block_lanes_host(n_txt, n_img, hidden, mlp, dtype) == 2
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    r = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    ctx = rg.Context(hidden, heads, d, mlp, n, 16, compute_dtype=dtype)
    blocks = []
    for _ in range(2):
        streams = [_stream(r, ctx, hidden, mlp) for _ in range(2)]
        bw = rg.BlockWeights()
        bw.txt, bw.img = (rg.make_stream_weights(t) for _, t in streams)
        blocks.append((bw, streams))
    h = r(n, hidden).to(ctx.torch_dtype)
    slots = torch.arange(n, dtype=torch.int32, device="cuda")
    runs = []
    for profiled in (False, False, True):
        rg.regione_profile_enable(ctx, profiled)
        caches = [torch.zeros((n, heads, d), dtype=ctx.torch_dtype, device="cuda") for _ in range(4)]
        x, mid = torch.full_like(h, float("nan")), torch.full_like(h, float("nan"))
        # the second block reads what both lanes of the first one wrote, at once
        rg.regione_block_forward(ctx, blocks[0][0], rg.BLOCK_DOUBLE, h, mid, dtype, n, n_txt, slots, 0, caches[0], caches[1], n, rg.FLAG_STORE)
        rg.regione_block_forward(ctx, blocks[1][0], rg.BLOCK_DOUBLE, mid, x, dtype, n, n_txt, slots, 0, caches[2], caches[3], n, rg.FLAG_STORE)
        mid.fill_(float("nan"))                          # on the caller's stream: both lanes have to be done with it
        runs.append([x, *caches])
    torch.cuda.synchronize()
    ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(runs[0], runs[1]))
    want = h.double()
    for _, streams in blocks:
        want = _block64(streams, want, n_txt, heads, d)
    # two blocks of bf16 operands and stores: 2^-9 relative each, some ten roundings in a row that add up as a random walk; float32: sums of up to 4096 terms
    bound = 2e-6 if f32 else 2.0 ** -7
    for rows in (slice(0, n_txt), slice(n_txt, n)):
        assert float((runs[0][0][rows].double() - want[rows]).norm() / want[rows].norm()) <= bound
        # the worst single row too: rows that one lane left unfinished would be off by their own size
        assert float(((runs[0][0][rows].double() - want[rows]).norm(dim=1) / want[rows].norm(dim=1)).max()) <= 4 * bound
    for a, b in zip(runs[0], runs[2]):                   # one lane: other K splits at most, the same roundings elsewhere
        assert float((a.double() - b.double()).norm() / b.double().norm()) <= bound
