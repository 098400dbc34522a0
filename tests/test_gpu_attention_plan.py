"""How attentions of few query tiles are dealt to key ranges: the choice knows that a key tile costs more where its rows lie apart.
With the costs of contiguous keys these calls by index list took 1.15 to 1.3 times as long as in the ranges asked for here."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,d,n_q,n_keys,least,most", [
    (8, 128, 1719, 5982, 4, 6), (8, 128, 3861, 6305, 2, 4), (24, 128, 595, 6591, 4, 6), (16, 128, 540, 6857, 5, 7),
])
def test_index_lists_get_enough_ranges(heads, d, n_q, n_keys, least, most):
    torch.zeros(1, device="cuda")
    ctx = rg.Context(heads * d, heads, d, 256, max(n_q, 2048), 16)
    try:
        splits, tiles, _ = rg.regione_attention_plan(ctx, n_q, n_keys, heads, d, rg.KEYS_INDEXED)
        assert tiles == 0 and least <= splits <= most
        # the source matters for these calls only in how many ranges pay
        assert 1 <= rg.regione_attention_plan(ctx, n_q, n_keys, heads, d, rg.KEYS_CONTIGUOUS)[0] <= most
        with pytest.raises(rg.RegionEError):
            rg.regione_attention_plan(ctx, n_q, n_keys, heads, d, 3)
    finally:
        ctx.close()
