"""Keys that are NaN and scores that overflow, in unsplit calls, equal key ranges (some of them without keys) and even ranges: a
row of the result is NaN exactly where softmax makes it NaN, whatever the split, and scores of minus infinity only take a
key's weight away, also where they fill a range's first keys or a whole range.  The oracle is float32 attention on the same bf16 inputs."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg
from test_gpu_attention_ranges import _reference

pytestmark = pytest.mark.gpu

BIG = 1e30      # two of them make a product beyond float32


@pytest.mark.parametrize("heads,d,n_q,n_keys,splits,form", [
    (2, 128, 130, 1000, 1, rg.ATTN_TILES_128), (2, 128, 130, 1000, 4, rg.ATTN_TILES_128), (2, 64, 130, 1000, 1, rg.ATTN_FREE), (2, 64, 130, 1000, 4, rg.ATTN_FREE),
    (3, 128, 40, 2111, 16, rg.ATTN_TILES_128), (2, 128, 300, 1000, 1, rg.ATTN_TILES_256), (2, 128, 300, 1000, 4, rg.ATTN_TILES_256),
    (2, 128, 130, 1000, 1, rg.ATTN_DEALT), (2, 128, 130, 1000, 4, rg.ATTN_DEALT), (2, 64, 130, 1000, 1, rg.ATTN_DEALT), (2, 64, 130, 1000, 4, rg.ATTN_DEALT),
    (2, 128, 40, 200, 1, rg.ATTN_DEALT),                                                         # a block per wave, or none
    (2, 128, 300, 1000, 1, rg.ATTN_FREE), (2, 128, 300, 1000, 4, rg.ATTN_FREE), (24, 128, 3000, 3000, 0, rg.ATTN_FREE),
    (24, 128, 3000, 3000, 0, rg.ATTN_TILES_128), (24, 128, 3000, 3000, 0, rg.ATTN_TILES_256),    # whole passes of query tiles, even ranges behind them
])
@pytest.mark.parametrize("kind", ["nan", "plus", "minus"])
def test_nonfinite_scores(kind, heads, d, n_q, n_keys, splits, form):
    g = torch.Generator(device="cuda")
    g.manual_seed(n_q + d)
    r = lambda n: torch.empty((n, heads, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q, k, v = r(n_q), r(n_keys), r(n_keys)
    hit = torch.zeros((n_q, heads), dtype=torch.bool, device="cuda")      # rows that softmax makes NaN
    if kind == "nan":
        k[n_keys // 2, -1, 5] = float("nan")
        hit[:, -1] = True
    else:
        q[:, -1, 0] = 0.0
        q[::3, -1, 0] = BIG
        k[:, -1, 0] = 0.0
        if kind == "plus":
            k[n_keys // 2 + 3, -1, 0] = BIG
            hit[::3, -1] = True
        else:
            k[: n_keys * 5 // 8, -1, 0] = -BIG
    want = _reference(q, k, v, d)
    assert torch.equal(want.isnan().any(-1), hit) and torch.equal(want.isnan().all(-1), hit)
    ctx = rg.Context(heads * d, heads, d, 256, max(n_q, 2048), 16)
    rg.regione_tune_attention(ctx, splits)
    rg.regione_tune_attention_form(ctx, form, 0 if splits else rg.RANGES_EVEN_BEHIND)
    assert rg.regione_attention_workgroups(ctx, n_q, n_keys, heads, d)[0] == form
    plan = rg.regione_attention_plan(ctx, n_q, n_keys, heads, d)
    assert plan[0] == splits if splits else plan[1] > 0 and plan[2] > 0
    out = torch.full((n_q + 1, heads, d), 7.0, dtype=torch.bfloat16, device="cuda")
    rg.regione_attn_kvcache(ctx, q, n_q, None, None, 0, k, v, n_keys, None, 0, heads, d, 0.0, out)
    torch.cuda.synchronize()
    ctx.close()
    got = out.float()
    assert torch.all(got[n_q] == 7.0)
    assert torch.equal(got[:n_q].isnan().all(-1), hit)
    live = ~hit[..., None].expand_as(want)
    # weights and result in bf16: 2^-9 relative each, on rows whose weights add up to one
    assert float((got[:n_q][live] - want[live]).abs().max()) <= 2.0 ** -7 * float(v.float().abs().max())
