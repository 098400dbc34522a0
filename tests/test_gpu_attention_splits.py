"""Few queries on many keys: more than eight key ranges per query tile (the chosen count and forced ones), the last
range shorter than the others, ranges that end up without keys, the last query tile not full; the oracle is float32 attention."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg
from test_gpu_attention_ranges import _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,d,n_q,n_keys", [
    (24, 128, 1, 8704), (24, 128, 129, 4097), (8, 128, 33, 19450), (3, 128, 300, 2111), (4, 64, 1, 2050), (4, 64, 257, 16384), (5, 64, 1000, 2500),
])
def test_many_key_ranges(heads, d, n_q, n_keys):
    g = torch.Generator(device="cuda")
    g.manual_seed(n_q)
    r = lambda n: torch.empty((n, heads, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q, k, v = r(n_q), r(n_keys), r(n_keys)
    q *= 2.0                                             # a softmax with some contrast
    want = _reference(q, k, v, d)
    # a workspace for these queries only; it holds 8192 rows of partial results, or eight per query
    ctx = rg.Context(heads * d, heads, d, 256, n_q if 16 * n_q <= 8192 else 2 * n_q, 16)
    for splits in (0, 8, 9, 15, 16):
        rg.regione_tune_attention(ctx, splits)
        if splits:                                       # no forced count may end up as another for want of workspace or key tiles
            assert rg.regione_attention_plan(ctx, n_q, n_keys, heads, d) == (splits, 0, (n_q + 127) // 128)
        out = torch.full((n_q + 1, heads, d), 7.0, dtype=torch.bfloat16, device="cuda")
        rg.regione_attn_kvcache(ctx, q, n_q, None, None, 0, k, v, n_keys, None, 0, heads, d, 0.0, out)
        torch.cuda.synchronize()
        got = out.float()
        assert torch.all(got[n_q] == 7.0)
        # weights and result in bf16: 2^-9 relative each, on rows whose weights add up to one
        assert float((got[:n_q] - want).norm() / want.norm()) <= 2.0 ** -8, splits
        assert float((got[:n_q] - want).abs().max()) <= 2.0 ** -7 * float(v.float().abs().max()), splits
    ctx.close()
