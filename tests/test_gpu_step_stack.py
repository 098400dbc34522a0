"""regione_region_step over stacks of blocks against the same step made of the separate calls, bit for bit: more modulation vectors than are formed at a time, blocks
with and without a conditioning vector, rows that the gather normalises on the way (more than 1024 values) and rows that it does not, a single-stream block first,
latent rows and tensors off the 16-byte grid, float32 and bf16 contexts, a head with more than 64 channels."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


def _block(g, ctx, H, M, kind, cond, keep):
    norm = lambda *s, k=1.0, dt=torch.float32: (torch.empty(s, device="cuda").normal_(generator=g) * k).to(dt)
    bw = rg.BlockWeights()
    for name in ("txt", "img") if kind == "double" else ("img",):
        shapes = {"w_qkv": (3 * H, H), "w_o": (H, H), "w_1": (M, H), "w_2": (H, M)} if kind == "double" else {"w_1": (3 * H + M, H), "w_2": (H, H + M)}
        t = {}
        for k, (n, c) in shapes.items():
            t[k], t["b" + k[1:]] = rg.pack_weight(ctx, norm(n, c, k=0.02, dt=ctx.torch_dtype)), norm(n, k=0.02)
        for i in (1, 2) if kind == "double" else (1,):
            t[f"shift{i}"], t[f"scale{i}"], t[f"gate{i}"] = norm(H, k=0.1), norm(H, k=0.1), norm(H, k=0.1)
        if cond is not None:
            n_mod = (6 if kind == "double" else 3) * H
            t["w_mod"], t["b_mod"] = norm(n_mod, H, k=0.02, dt=torch.bfloat16), norm(n_mod, k=0.02)
        keep.append(t)
        setattr(bw, name, rg.make_stream_weights(t))
    if cond is not None:
        bw.cond = cond.data_ptr()
    return bw, rg.BLOCK_DOUBLE if kind == "double" else rg.BLOCK_SINGLE


@pytest.mark.parametrize("H,heads,M,kinds,conds,n_txt_fresh,f32,channels,shifted", [
    (256, 4, 128, "d" * 18, "1" * 18, 24, False, 64, 0),           # 36 sets of vectors
    (256, 4, 128, "dsd", "101", 24, False, 64, 0),
    (1152, 9, 128, "ds", "10", 24, False, 64, 0),
    (1152, 9, 128, "sd", "00", 0, False, 64, 0),
    (1152, 9, 128, "sd", "00", 24, False, 64, 0),                  # a single-stream block first: text and image rows are one group
    (1152, 9, 128, "d", "0", 0, True, 64, 0),
    (256, 4, 128, "d", "0", 24, True, 64, 0),
    (256, 4, 128, "d", "0", 0, True, 12, 0),                        # latent rows of 48 bytes, no groups of eight
    (1152, 9, 128, "d", "1", 0, False, 64, 2),                     # hidden rows off the 16-byte grid on their way out
    (1152, 9, 128, "d", "1", 0, False, 136, 0),                    # a head of the tile kernels
])
def test_stack_equals_separate_calls(H, heads, M, kinds, conds, n_txt_fresh, f32, channels, shifted):
    g = torch.Generator(device="cuda")
    g.manual_seed(H + len(kinds) + n_txt_fresh)
    norm = lambda *s, k=1.0, dt=torch.float32: (torch.empty(s, device="cuda").normal_(generator=g) * k).to(dt)
    n_txt, n_img = 24, 300
    n_all = n_txt + 2 * n_img
    ctx = rg.Context(H, heads, H // heads, M, n_all, n_img, compute_dtype=rg.FP32 if f32 else rg.BF16)
    rdt, rows_dt = xdt, lat_dt = (rg.FP32, torch.float32) if f32 else (rg.BF16, torch.bfloat16)
    cond, keep = norm(H), []
    blocks = [_block(g, ctx, H, M, "double" if k == "d" else "single", cond if c == "1" else None, keep) for k, c in zip(kinds, conds)]
    kc = [norm(n_all, heads, H // heads, dt=ctx.torch_dtype) for _ in blocks]
    vc = [norm(n_all, heads, H // heads, dt=ctx.torch_dtype) for _ in blocks]
    want = torch.rand(n_img, device="cuda", generator=g) < 0.3
    ref = norm(n_img, channels)
    x_t = (ref + norm(n_img, channels) * want[:, None]).to(lat_dt)
    v = norm(n_img, channels, k=1e-3).to(lat_dt)
    w_head, b_head = rg.pack_weight(ctx, norm(channels, H, k=0.02, dt=ctx.torch_dtype)), norm(channels)
    h_full = norm(n_img, H, dt=rows_dt)
    txt = norm(n_txt_fresh, H, dt=rows_dt)
    x_ref = ref.to(lat_dt)

    def state():
        z = lambda *s, dt=torch.float32: torch.zeros(s, dtype=dt, device="cuda")
        flat = torch.zeros(n_img * H + 8, dtype=rows_dt, device="cuda")
        s = {"mask": z(n_img, dt=torch.uint8), "e": z(n_img, dt=torch.int32), "u": z(n_img, dt=torch.int32), "n": z(1, dt=torch.int32), "score": z(n_img),
             "rows": z(n_txt_fresh + n_img, H, dt=rows_dt), "rows_out": z(n_txt_fresh + n_img, H, dt=rows_dt), "slots": z(n_txt_fresh + n_img, dt=torch.int32),
             "v": z(n_img, channels, dt=lat_dt), "ca": z(n_img, channels, dt=lat_dt), "xe": z(n_img, channels, dt=lat_dt), "x": x_t.clone(),
             "h": flat[shifted:shifted + n_img * H].view(n_img, H), "k": [t.clone() for t in kc], "vv": [t.clone() for t in vc]}
        s["h"].copy_(h_full)
        s["rows"][:n_txt_fresh].copy_(txt)
        return s

    a = state()
    args = rg.make_region_step_args(x_t=x_t, v=v, x_ref=x_ref, n_tokens=n_img, c=channels, dtype=xdt, sigma_t=0.7, eta=0.9, score=a["score"], mask=a["mask"], e_index=a["e"],
                                    u_index=a["u"], n_edited_dev=a["n"], h_full=h_full, h_dtype=rdt, n_txt_fresh=n_txt_fresh, h_rows=a["rows"], h_rows_out=a["rows_out"],
                                    slots=a["slots"] if n_txt_fresh else None, blocks=[b for b, _ in blocks], block_types=[t for _, t in blocks], k_caches=a["k"], v_caches=a["vv"],
                                    n_all=n_all, slot_offset=n_txt, w_head=w_head, b_head=b_head, dt=0.04, v_out=a["v"], c_a=a["ca"], x_e=a["xe"], x_next_full=a["x"],
                                    h_next_full=a["h"])
    n = rg.regione_region_step(ctx, args)
    b = state()
    assert rg.regione_partition(ctx, x_t, v, x_ref, n_img, channels, xdt, 0.7, 0.9, b["score"], b["mask"], b["e"], b["u"], b["n"]) == n > 16
    rg.regione_gather_pair(ctx, h_full, H, rdt, b["rows"][n_txt_fresh:], x_t, channels, xdt, b["xe"], b["e"], b["n"], n)
    if n_txt_fresh:
        rg.regione_fresh_slots(ctx, b["e"], b["n"], n, n_txt_fresh, b["slots"])
    src = b["rows"]
    for (w, kind), k, vv in zip(blocks, b["k"], b["vv"]):
        rg.regione_block_forward(ctx, w, kind, src, b["rows_out"], rdt, n_txt_fresh + n, n_txt_fresh, b["slots"] if n_txt_fresh else b["e"], 0 if n_txt_fresh else n_txt,
                                 k, vv, n_all, rg.FLAG_RETRIEVE)
        src = b["rows_out"]
    rows_out = b["rows_out"][n_txt_fresh:]
    rg.regione_velocity_head(ctx, rows_out, w_head, b_head, n, channels, H, 0.04, b["v"], b["ca"], b["xe"], b["x"], b["e"], xdt)
    rg.regione_scatter(ctx, b["h"], H, rdt, b["e"], b["n"], n, rows_out)
    torch.cuda.synchronize()
    for key in a:
        for p, q in zip(a[key], b[key]) if isinstance(a[key], list) else [(a[key], b[key])]:
            assert torch.equal(p, q), key
    ctx.close()
