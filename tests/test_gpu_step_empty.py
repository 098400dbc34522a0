"""A region step that finds nothing to edit ends behind its partition: the modulation matrices of its blocks, 0.9 GB here, are not read, whatever the call queued before it knew the count."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


def test_nothing_edited_reads_no_matrix():
    H, heads, M, n_img, c, n_blocks = 3072, 24, 64, 256, 64, 16
    ctx = rg.Context(H, heads, 128, M, n_img, n_img)
    z = lambda *s, dt=torch.float32: torch.zeros(s, dtype=dt, device="cuda")
    bf = torch.bfloat16
    w = {"w_1": rg.pack_weight(ctx, z(3 * H + M, H, dt=bf)), "w_2": rg.pack_weight(ctx, z(H, H + M, dt=bf)), "b_1": z(3 * H + M), "b_2": z(H), "b_mod": z(3 * H)}
    cond, matrices, blocks = z(H), [z(3 * H, H, dt=bf) for _ in range(n_blocks)], []
    for m in matrices:
        b = rg.BlockWeights()
        b.img, b.cond = rg.make_stream_weights({**w, "w_mod": m}), cond.data_ptr()
        blocks.append(b)
    k, v = (z(2 * n_img, heads, 128, dt=bf) for _ in range(2))
    x = torch.ones((n_img, c), dtype=bf, device="cuda")                     # the estimate is the reference: cosine 1
    h, rows, rows_out = (z(n_img, H, dt=bf) for _ in range(3))
    lists = [torch.full((n_img,), -1, dtype=torch.int32, device="cuda") for _ in range(2)]
    mask, count = torch.full((n_img,), 7, dtype=torch.uint8, device="cuda"), torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ca, xe = z(n_img, c, dt=bf), z(n_img, c, dt=bf)
    args = rg.make_region_step_args(x_t=x, v=torch.zeros_like(x), x_ref=x, n_tokens=n_img, c=c, dtype=rg.BF16, sigma_t=0.5, eta=0.9, score=None, mask=mask, e_index=lists[0], u_index=lists[1],
                                    n_edited_dev=count, h_full=h, h_dtype=rg.BF16, n_txt_fresh=0, h_rows=rows, h_rows_out=rows_out, slots=None, blocks=blocks,
                                    block_types=[rg.BLOCK_SINGLE] * n_blocks, k_caches=[k] * n_blocks, v_caches=[v] * n_blocks, n_all=2 * n_img, slot_offset=0,
                                    w_head=rg.pack_weight(ctx, z(c, H, dt=bf)), b_head=z(c), dt=0.04, v_out=None, c_a=ca, x_e=xe, x_next_full=x.clone(), h_next_full=h)
    times = []
    for _ in range(4):
        rg.regione_profile_enable(ctx, 1)
        assert rg.regione_region_step(ctx, args) == 0
        times.append(rg.regione_profile_read(ctx)["gemm"][0])
        rg.regione_profile_enable(ctx, 0)
    torch.cuda.synchronize()
    ctx.close()
    assert int(count) == 0 and int(mask.sum()) == 0 and torch.equal(lists[1], torch.arange(n_img, dtype=torch.int32, device="cuda"))
    print("modulation launch of an empty step, us:", [round(1e3 * t, 1) for t in times])
    # no card of this kind reads faster than 8 TB/s: half of the time that the matrices would take at least
    assert min(times) * 1e-3 < 0.5 * sum(m.numel() * 2 for m in matrices) / 8e12
