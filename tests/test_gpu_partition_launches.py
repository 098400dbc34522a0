"""The partition around the sizes where its launches change: lists written by the last workgroup of the score's launch (up to 2560 tokens), by a second launch that adds up the counts
itself, and behind a scan; several calls in a row, since the counter of the first form has to be zero again after each."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1024, 2559, 2560, 2561, 70001, 262143, 4 * 1024 * 1024 + 70])
@pytest.mark.parametrize("share", [0.0, 0.2, 1.0])
def test_lists(n, share):
    c = 8
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    ref = torch.ones((n, c), device="cuda", dtype=torch.bfloat16)
    ctx = rg.Context(256, 4, 64, 256, 16, n)
    for call in range(3 if n < 100000 else 1):
        edited = torch.rand(n, device="cuda", generator=g) < share
        x = torch.where(edited[:, None], -ref, ref)             # cosine -1 or 1
        v = torch.zeros_like(x)
        mask = torch.full((n + 16,), 7, dtype=torch.uint8, device="cuda")
        e, u = (torch.full((n + 4,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        count = torch.zeros(1, dtype=torch.int32, device="cuda")
        got = rg.regione_partition(ctx, x, v, ref, n, c, rg.BF16, 0.5, 0.9, None, mask, e, u, count)
        want_e, want_u = torch.nonzero(edited).view(-1).to(torch.int32), torch.nonzero(~edited).view(-1).to(torch.int32)
        assert got == int(count) == want_e.numel()
        assert torch.equal(mask[:n].bool(), edited) and bool((mask[n:] == 7).all())
        assert torch.equal(e[:got], want_e) and torch.equal(u[:n - got], want_u)
        assert bool((e[got:] == -1).all()) and bool((u[n - got:] == -1).all())
    ctx.close()
