"""E4M3 blocks of one group of rows, whose attention result is quantised by the launch that merges its key ranges (head dimension 128) or by the quantiser: one query to more than a query
tile, few and many heads, few keys (one range), many, and even ranges by themselves and behind whole query tiles.  The merged rows against float64 attention on the block's own queries, keys
and values, also where keys are NaN or scores overflow; codes and scales are the quantiser's on these rows bit for bit, and the block gives the same bits whether or not the rows are handed
out."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu

BIG = 1e30      # two of them make a product beyond float32


def _attention(q, k, v):
    """float64: the result, and the sum of weight times magnitude of the values"""
    out, size = torch.empty(q.shape, dtype=torch.float64, device=q.device), torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for head in range(q.shape[1]):
        p = torch.softmax(q[:, head].double() @ k[:, head].double().T / q.shape[2] ** 0.5, -1)
        out[:, head], size[:, head] = p @ v[:, head].double(), p @ v[:, head].double().abs()
    return out, size


def _check(heads, d, n, n_all, kind="finite"):
    """kind: of the last head's scores: all finite; "nan": one key of it is NaN; "plus": one key's scores overflow; "minus": those of the first 5/8 of the keys overflow downwards."""
    hidden, mlp = heads * d, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(heads + n)
    rnd = lambda *s, k=1.0: torch.empty(s, device="cuda").normal_(generator=g) * k
    ctx = rg.Context(hidden, heads, d, mlp, n, 16)
    raw = {"w_qkv": rnd(3 * hidden, hidden, k=0.05), "w_o": rnd(hidden, hidden, k=0.05), "w_1": rnd(mlp, hidden, k=0.05), "w_2": rnd(hidden, mlp, k=0.05)}
    raw = {k: v.to(torch.bfloat16) for k, v in raw.items()}
    t = {"b_qkv": rnd(3 * hidden), "b_o": rnd(hidden), "b_1": rnd(mlp), "b_2": rnd(hidden)}
    for i in (1, 2):
        t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = rnd(hidden, k=0.1), rnd(hidden, k=0.1), rnd(hidden)
    k, v = (rnd(n_all, heads, d).to(torch.bfloat16) for _ in range(2))
    slots = torch.randperm(n_all, device="cuda", generator=g)[:n].sort().values.to(torch.int32).contiguous()
    cached = torch.ones(n_all, dtype=torch.bool, device="cuda")
    cached[slots.long()] = False
    if kind == "nan":
        k[cached.nonzero()[0, 0], -1, 5] = float("nan")
    elif kind in ("plus", "minus"):
        # the last head's queries are BIG in their first element, its fresh keys zero there, and its cached ones as wanted
        first = (heads - 1) * d
        raw["w_qkv"][first] = 0
        raw["w_qkv"][hidden + first] = 0
        t["b_qkv"][first], t["b_qkv"][hidden + first] = BIG, 0.0
        k[:, -1, 0] = 0.0
        if kind == "plus":
            k[cached.nonzero()[-1, 0], -1, 0] = BIG
        else:
            k[: n_all * 5 // 8, -1, 0] = -BIG
    bw, w8 = rg.BlockWeights(), rg.BlockWeightsFp8()
    bw.img = rg.make_stream_weights(t)
    w8.img, held = rg.make_stream_weights_fp8(ctx, raw)
    h = rnd(n, hidden).to(torch.bfloat16)
    attn, q = (torch.zeros((n, hidden), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    codes, want = (torch.full((n + 1, hidden), 0x55, dtype=torch.uint8, device="cuda") for _ in range(2))
    scale, want_scale = (torch.full((n + 1,), -1.0, device="cuda") for _ in range(2))
    taps = rg.Fp8Taps()
    taps.q, taps.attn, taps.a_codes, taps.a_scale = q.data_ptr(), attn.data_ptr(), codes.data_ptr(), scale.data_ptr()
    outs = []
    for tap in (taps, None, taps):
        out = torch.zeros_like(h)
        rg.regione_block_forward_fp8(ctx, bw, w8, rg.BLOCK_DOUBLE, h, out, rg.BF16, n, 0, slots, 0, k, v, n_all, rg.FLAG_RETRIEVE, tap)
        outs.append(out)
    rg.regione_quantize_rows_fp8(ctx, attn, n, hidden, want, want_scale)
    form = rg.regione_attention_workgroups(ctx, n, n_all, heads, d, rg.KEYS_WIDE_8BIT if hidden > 1024 else rg.KEYS_CONTIGUOUS)
    torch.cuda.synchronize()
    ctx.close()
    got = attn.view(n, heads, d)
    sound = heads if kind in ("finite", "minus") else heads - 1               # heads whose results are numbers
    result, size = _attention(q.view(n, heads, d)[:, :sound], k[:, :sound], v[:, :sound])
    error = (got[:, :sound].double() - result).abs()
    # the weights are rounded to bf16, and so is the result: at most 2^-8 of either (eight significant bits), and 2^-12 for the exponentials and the sums in float32
    bound = (size + result.abs()) * (2.0 ** -8 + 2.0 ** -12)
    print(f"{heads} heads of {d}, {n} of {n_all}, {kind}: form, ranges, range tiles {form}, error of bound {float((error / bound).max()):.2f}")
    assert bool((error <= bound).all())
    assert sound == heads or bool(got[:, -1].isnan().all())
    assert float(attn[:, : sound * d].float().abs().max()) > 0 and (kind != "finite" or bool(torch.isfinite(outs[0].float()).all()))
    same = lambda a, b: torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert same(outs[0], outs[1]) and same(outs[0], outs[2])
    assert torch.equal(codes, want) and torch.equal(scale, want_scale)


@pytest.mark.parametrize("heads,d", [(2, 128), (9, 128), (24, 128), (32, 128), (4, 64)])
@pytest.mark.parametrize("n,n_all", [(1, 700), (33, 64), (205, 4608), (300, 4608), (820, 4608), (4608, 4608)])
def test_codes(heads, d, n, n_all):
    _check(heads, d, n, n_all)


# heads of 128, rows, keys: one of each kernel that merges and quantises (tests/test_attention_codes_routes.py): equal ranges, even ones of 128 and of 256 queries
MERGES = {"<128, 128, false>": [(2, 820, 4608), (32, 400, 8704)], "<128, 128, true>": [(2, 8704, 8704), (12, 1600, 4608)], "<128, 256, true>": [(4, 4608, 8704), (5, 6000, 8704)]}


@pytest.mark.parametrize("heads,n,n_all", sorted({call for calls in MERGES.values() for call in calls}))
def test_every_merge(heads, n, n_all):
    _check(heads, 128, n, n_all)


@pytest.mark.parametrize("kind", ["nan", "plus", "minus"])
@pytest.mark.parametrize("heads,d,n,n_all", [(2, 128, 33, 700), (9, 128, 300, 4608), (24, 128, 820, 4608), (24, 128, 3000, 4608), (5, 128, 4608, 8704), (4, 64, 205, 4608)])
def test_nonfinite_scores(heads, d, n, n_all, kind):
    _check(heads, d, n, n_all, kind)
