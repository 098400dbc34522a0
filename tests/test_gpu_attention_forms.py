"""The forms of attention workgroups at the sizes where each can go wrong, forced so that every call shows the form it names: 32-query tiles that deal their keys to
the waves (none, one, two and more blocks per wave, in one key range and in several), 128-query tiles whose two wave groups take a range each or one in turns, and
256-query tiles, unsplit and in even ranges; query and key counts around the tiles' edges, the place where the cache rows begin inside a tile, every key
source.  The oracle is float32 attention on the same bf16 inputs."""
import numpy as np
import pytest
import torch

from gpu_util import block_to_device, dev
from paper_2510_25590_amd import binding as rg
from paper_2510_25590_amd import inputs
from test_gpu_attention_ranges import _reference

pytestmark = pytest.mark.gpu


KEYS = {"one": rg.KEYS_CONTIGUOUS, "two": rg.KEYS_TWO, "indexed": rg.KEYS_INDEXED}


def _call(heads, d, n_q, n_fresh, n_cached, source, splits=0, form=0, ranges=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * n_q + n_cached)
    r = lambda n: torch.empty((n, heads, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    rows = n_cached if source != "indexed" else n_cached + 77
    q, kf, vf, kc, vc = r(n_q) * 2.0, r(n_fresh), r(n_fresh), r(max(rows, 1)), r(max(rows, 1))
    idx = torch.randperm(rows, generator=g, device="cuda")[:n_cached].int().contiguous() if source == "indexed" else None
    ctx = rg.Context(heads * d, heads, d, 256, max(n_q, 512), 16)
    rg.regione_tune_attention(ctx, splits)
    rg.regione_tune_attention_form(ctx, form, ranges)
    plan = rg.regione_attention_workgroups(ctx, n_q, n_fresh + n_cached, heads, d, KEYS[source])
    if form:
        assert plan[0] == form and (plan[2] > 0) == (ranges > rg.RANGES_EQUAL) and plan[1] == (splits or plan[1])
    outs = []
    for _ in range(2):
        out = torch.full((n_q + 1, heads, d), 7.0, dtype=torch.bfloat16, device="cuda")
        rg.regione_attn_kvcache(ctx, q, n_q, kf if n_fresh else None, vf if n_fresh else None, n_fresh, kc, vc, rows, idx, n_cached if source == "indexed" else 0,
                                heads, d, 0.0, out)
        torch.cuda.synchronize()
        outs.append(out)
    ctx.close()
    assert torch.equal(outs[0], outs[1])                 # no order that depends on timing
    used = (kc[idx.long()], vc[idx.long()]) if source == "indexed" else (kc[:n_cached], vc[:n_cached])
    k, v = torch.cat([kf, used[0]]), torch.cat([vf, used[1]])
    want, got = _reference(q, k, v, d), outs[0].float()
    assert torch.all(got[n_q] == 7.0)
    # weights and result in bf16: 2^-9 relative each, on rows whose weights add up to one
    assert float((got[:n_q] - want).norm() / want.norm()) <= 2.0 ** -8
    assert float((got[:n_q] - want).abs().max()) <= 2.0 ** -7 * float(v.float().abs().max())
    return plan


FEW = [(3, 128, 1, 1), (2, 64, 31, 32), (8, 128, 32, 33), (4, 64, 33, 65), (8, 128, 65, 257), (4, 64, 36, 544), (4, 64, 257, 575), (24, 128, 64, 513), (5, 128, 100, 1023),
       (24, 128, 17, 3500), (4, 64, 40, 4100)]


@pytest.mark.parametrize("source", ["one", "two", "indexed"])
@pytest.mark.parametrize("heads,d,n_q,n_keys,splits", [(*c, s) for c in FEW for s in (0, 3) if 64 * 2 * s <= c[3] + 63])     # a forced range has two key tiles at least
def test_few_queries(source, heads, d, n_q, n_keys, splits):
    n_fresh = 0 if source == "one" else min(n_q, n_keys // 2)
    _call(heads, d, n_q, n_fresh, n_keys - n_fresh, source, splits, rg.ATTN_DEALT)


@pytest.mark.parametrize("indexed", [False, True])
@pytest.mark.parametrize("heads,d", [(24, 128), (4, 64)])
def test_few_queries_weigh_their_largest_scores_exactly(heads, d, indexed):
    """Keys of a workgroup that deals them to its waves, 32 a wave: one key in every wave's block carries all the block's weight.  Each is its wave's reference, whose
    weight is exactly one; the waves are joined in float32, so that only the result's own rounding is left."""
    n_q, n_keys = 40, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    r = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda").normal_(generator=g)
    q, k, v = torch.zeros((n_q, heads, d), device="cuda"), torch.zeros((n_keys, heads, d), device="cuda"), r(n_keys, heads, d).to(torch.bfloat16)
    q[..., 0], q[..., 1] = 8.0, 1.0 + r(n_q, heads).abs()
    k[..., 0] = -100.0 * d ** 0.5 / 8.0                   # scores of -100 ...
    live = torch.arange(8, device="cuda") * 32 + torch.randint(0, 32, (8,), generator=g, device="cuda")
    k[live, :, 0], k[live, :, 1] = 0.0, r(8, heads) * d ** 0.5      # ... but for one key in 32, of about -5 to 5
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    out = torch.empty_like(q)
    ctx = rg.Context(heads * d, heads, d, 256, 512, 16)
    idx = torch.arange(n_keys, dtype=torch.int32, device="cuda") if indexed else None
    rg.regione_tune_attention_form(ctx, rg.ATTN_DEALT)
    assert rg.regione_attention_workgroups(ctx, n_q, n_keys, heads, d, KEYS["indexed" if indexed else "one"])[0] == rg.ATTN_DEALT
    rg.regione_attn_kvcache(ctx, q, n_q, None, None, 0, k, v, n_keys, idx, n_keys if indexed else 0, heads, d, 0.0, out)
    torch.cuda.synchronize()
    ctx.close()
    p = torch.softmax(torch.einsum("qhd,khd->hqk", q.cpu().double(), k.cpu().double()) / d ** 0.5, dim=-1)
    want = torch.einsum("hqk,khd->qhd", p, v.cpu().double())
    sizes = torch.einsum("hqk,khd->qhd", p, v.cpu().double().abs())
    # the nearest bf16 value, or where float32 scores (up to 20, scaled), exponentials and sums of eight terms (2^-17 of the terms' sizes) reach across a tie its neighbour
    assert torch.all((out.cpu().double() - want).abs() <= (want.to(torch.bfloat16).double() - want).abs() + 2.0 ** -16 * sizes)


@pytest.mark.parametrize("source", ["one", "two", "indexed"])
@pytest.mark.parametrize("heads,n_q,n_keys,splits,form,ranges", [
    (24, 257, 1500, 4, rg.ATTN_TILES_128, rg.RANGES_EQUAL), (24, 820, 4097, 2, rg.ATTN_TILES_128, rg.RANGES_EQUAL),       # ranges in pairs
    (24, 2500, 1217, 1, rg.ATTN_TILES_256, rg.RANGES_EQUAL), (8, 6500, 700, 1, rg.ATTN_TILES_256, rg.RANGES_EQUAL),       # unsplit; the last tile with a few rows
    (24, 300, 2300, 3, rg.ATTN_TILES_256, rg.RANGES_EQUAL), (24, 100, 600, 4, rg.ATTN_TILES_256, rg.RANGES_EQUAL),        # equal ranges; the last ones short or empty
    (24, 820, 513, 1, rg.ATTN_FREE, rg.RANGES_EQUAL), (24, 100, 600, 4, rg.ATTN_FREE, rg.RANGES_EQUAL), (24, 1400, 5001, 0, rg.ATTN_FREE, rg.RANGES_EVEN),      # free waves
    (24, 1400, 5001, 0, rg.ATTN_TILES_256, rg.RANGES_EVEN), (24, 1400, 5001, 0, rg.ATTN_TILES_128, rg.RANGES_EVEN),       # even ranges, alone ...
    (24, 3100, 2050, 0, rg.ATTN_TILES_256, rg.RANGES_EVEN_BEHIND), (24, 3100, 2050, 0, rg.ATTN_TILES_128, rg.RANGES_EVEN_BEHIND),      # ... and behind whole passes
])
def test_many_queries(source, heads, n_q, n_keys, splits, form, ranges):
    n_fresh = 0 if source == "one" else 333
    _call(heads, 128, n_q, n_fresh, n_keys - n_fresh, source, splits, form, ranges)


@pytest.mark.parametrize("source", ["one", "two", "indexed"])
@pytest.mark.parametrize("heads,d,n_q,n_keys", [(24, 128, 257, 1500), (24, 128, 1400, 5001), (24, 128, 3100, 2050), (4, 64, 36, 544), (4, 64, 1500, 3000), (8, 128, 100, 3000)])
def test_own_choice(source, heads, d, n_q, n_keys):
    """What the library takes by itself, and again after a form was forced and given back."""
    n_fresh = 0 if source == "one" else 33
    plan = _call(heads, d, n_q, n_fresh, n_keys - n_fresh, source)
    ctx = rg.Context(heads * d, heads, d, 256, max(n_q, 512), 16)
    for form, ranges in ((rg.ATTN_DEALT, 0), (rg.ATTN_TILES_256, rg.RANGES_EVEN), (rg.ATTN_FREE, rg.RANGES_EQUAL), (0, 0)):
        rg.regione_tune_attention_form(ctx, form, ranges)
        got = rg.regione_attention_workgroups(ctx, n_q, n_keys, heads, d, KEYS[source])
    assert got == plan
    for bad in ((-1, 0), (5, 0), (0, -1), (0, 4)):
        with pytest.raises(rg.RegionEError):
            rg.regione_tune_attention_form(ctx, *bad)
    with pytest.raises(rg.RegionEError):
        rg.regione_attention_workgroups(ctx, n_q, n_keys, heads, d, 4)
    ctx.close()


@pytest.mark.parametrize("splits", [1, 2, 3, 4, 7])
def test_forced_ranges(splits):
    """One range and odd numbers are taken by the wave groups in turns, even numbers a range to each group; the last ones are short or empty."""
    for n_keys in (128 * splits + 1, 128 * splits + 129, 2000):
        _call(2, 128, 150, 50, n_keys - 50, "indexed", splits, rg.ATTN_TILES_128)


@pytest.mark.parametrize("n_txt,n_img,n_all,plan", [
    (528, 400, 928, (rg.ATTN_TILES_128, 1, 0)), (17, 240, 257, (rg.ATTN_FREE, 1, 0)), (300, 1717, 2017, (rg.ATTN_TILES_256, 1, 0)),      # one range
    (20, 80, 1000, (rg.ATTN_FREE, 4, 0)), (0, 300, 3000, (rg.ATTN_TILES_128, 3, 0)),                     # equal ranges
    (60, 1272, 3000, (rg.ATTN_FREE, 1, 25)), (500, 1000, 1500, (rg.ATTN_FREE, 1, 14)), (100, 2600, 2700, (rg.ATTN_FREE, 1, 7)),      # even ranges, the last behind whole passes
])
def test_wide_8bit_block(n_txt, n_img, n_all, plan):
    """A double-stream E4M3 block above width 1024 keeps its key ranges, equal and even ones, in whatever form is the fastest for them."""
    heads, d, mlp, n = 24, 128, 256, n_txt + n_img
    hidden = heads * d
    rng = np.random.default_rng(n)
    streams = [inputs.stream_weights(rng, hidden, mlp, "double", "bf16", std=0.02) for _ in range(2)]
    ctx = rg.Context(hidden, heads, d, mlp, n, 16)
    assert rg.regione_attention_workgroups(ctx, n, n_all, heads, d, rg.KEYS_WIDE_8BIT) == plan
    bw, keep = block_to_device(streams, "double", ctx)
    w8 = rg.BlockWeightsFp8()
    held = []
    for name, s in (("txt", streams[0]), ("img", streams[1])):
        w, k = rg.make_stream_weights_fp8(ctx, {key: dev(v, "bf16") for key, v in s.items() if key.startswith("w_")})
        setattr(w8, name, w)
        held.append(k)
    h = dev(inputs.bf16_round(rng.standard_normal((n, hidden)).astype(np.float32)), "bf16")
    slots = torch.arange(n, dtype=torch.int32, device="cuda")
    kc, vc = (torch.randn((n_all, heads, d), device="cuda").to(torch.bfloat16) for _ in range(2))
    taps = {"q": torch.zeros((n, hidden), dtype=torch.bfloat16, device="cuda"), "attn": torch.zeros((n, hidden), dtype=torch.bfloat16, device="cuda")}
    out = torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda")
    rg.regione_block_forward_fp8(ctx, bw, w8, rg.BLOCK_DOUBLE, h, out, rg.BF16, n, n_txt, slots, 0, kc, vc, n_all, rg.FLAG_STORE if n == n_all else rg.FLAG_RETRIEVE,
                                 rg.make_fp8_taps(taps))
    torch.cuda.synchronize()
    ctx.close()
    want, got = _reference(taps["q"].view(n, heads, d), kc, vc, d), taps["attn"].view(n, heads, d).float()
    assert float((got - want).norm() / want.norm()) <= 2.0 ** -8
    assert float((got - want).abs().max()) <= 2.0 ** -7 * float(vc.float().abs().max())
