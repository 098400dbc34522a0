"""Attention whose workgroups take even ranges of the list (head, query tile, key tile): ranges shorter and longer than a
query tile's keys, behind whole passes of unsplit query tiles or alone, with a last query tile and key tile that are not
full, for every key source; the oracle is float32 attention on the same bf16 inputs."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


def _reference(q, k, v, d):
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    for h in range(q.shape[1]):
        p = torch.softmax(q[:, h].float() @ k[:, h].float().T.contiguous() / d ** 0.5, dim=-1)
        out[:, h] = p @ v[:, h].float().contiguous()
    return out


FORMS = (rg.ATTN_TILES_128, rg.ATTN_TILES_256, rg.ATTN_FREE)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("source", ["contiguous", "two", "indexed"])
@pytest.mark.parametrize("heads,n_q,n_keys,whole,short", [
    (24, 1409, 3001, 0, (False, True, True)),     # no query tile in front; ranges longer than a tile of 128 queries' keys, shorter than one of 256
    (8, 1461, 3001, 0, (True, True, True)),       # 0.19 of a pass: many ranges meet in a query tile
    (12, 5450, 2499, 0, (False, False, False)),    # heads not a multiple of the XCDs; a range longer than a query tile's keys, no whole pass
    (8, 8700, 2497, 64, (True, True, True)),      # whole passes, the rest in ranges
    (24, 2900, 3001, 21, (True, True, True)),     # ... that the heads do not divide
])
def test_even_ranges(form, source, heads, n_q, n_keys, whole, short):
    d = 128
    g = torch.Generator(device="cuda")
    g.manual_seed(n_q)
    r = lambda n: torch.empty((n, heads, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q, k, v = r(n_q), r(n_keys), r(n_keys)
    q *= 2.0                                             # a softmax with some contrast
    n_fresh = 0 if source == "contiguous" else 333
    idx = torch.arange(n_keys - n_fresh, dtype=torch.int32, device="cuda").flip(0).contiguous() if source == "indexed" else None
    kc, vc = k[n_fresh:].contiguous(), v[n_fresh:].contiguous()
    ctx = rg.Context(heads * d, heads, d, 256, max(n_q, 2048), 16)
    keys = {"contiguous": rg.KEYS_CONTIGUOUS, "two": rg.KEYS_TWO, "indexed": rg.KEYS_INDEXED}[source]
    rg.regione_tune_attention_form(ctx, form, rg.RANGES_EVEN_BEHIND if whole else rg.RANGES_EVEN)
    splits, tiles, in_front = rg.regione_attention_plan(ctx, n_q, n_keys, heads, d, keys)
    assert rg.regione_attention_workgroups(ctx, n_q, n_keys, heads, d, keys) == (form, 1, tiles)
    # even ranges, of the case's kind; workgroups of 256 queries take the query tiles in front in pairs
    assert (splits, in_front) == (1, whole // 2 * 2 if form == rg.ATTN_TILES_256 else whole) and tiles > 0 and (tiles < (n_keys + 63) // 64) == short[FORMS.index(form)]
    outs = []
    for splits in (0, 0, 1):
        rg.regione_tune_attention(ctx, splits)
        out = torch.full((n_q + 1, heads, d), 7.0, dtype=torch.bfloat16, device="cuda")
        rg.regione_attn_kvcache(ctx, q, n_q, k[:n_fresh].contiguous() if n_fresh else None, v[:n_fresh].contiguous() if n_fresh else None, n_fresh, kc, vc, n_keys - n_fresh,
                                idx, n_keys - n_fresh if source == "indexed" else 0, heads, d, 0.0, out)
        torch.cuda.synchronize()
        outs.append(out)
    ctx.close()
    assert torch.equal(outs[0], outs[1])                 # no order that depends on timing
    want = _reference(q, k, v, d)
    for out in outs[1:]:
        got = out.float()
        assert torch.all(got[n_q] == 7.0)
        # weights and result in bf16: 2^-9 relative each, on rows whose weights add up to one
        assert float((got[:n_q] - want).norm() / want.norm()) <= 2.0 ** -8
        assert float((got[:n_q] - want).abs().max()) <= 2.0 ** -7 * float(v.float().abs().max())
