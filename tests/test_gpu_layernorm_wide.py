"""Rows that several waves share: every number of waves with whole and partly filled last ones, and more rows than the launch has workgroups, so that one goes through
several; bf16 and float32 in and out (the oracle and the bound of test_gpu_layernorm_rows.py), and the E4M3 form at the same widths."""
import pytest
import torch

from paper_2510_25590_amd import binding as rg
from oracle import fp8_reference as f8
import test_gpu_layernorm_rows as rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f32_ctx,f32_in", [(False, False), (False, True), (True, True), (True, False)])
@pytest.mark.parametrize("n,hidden", [(3, 1536), (2, 1544), (3, 2048), (1, 2056), (2, 2560), (2, 2568), (3, 3072), (2, 3080), (2, 3584), (1, 3592), (2, 4088), (2570, 1032), (1300, 3072), (1030, 4096)])
def test_rows_of_several_waves(f32_ctx, f32_in, n, hidden):
    rows.test_rows(f32_ctx, f32_in, n, hidden, 0)


@pytest.mark.parametrize("h_dtype", [rg.BF16, rg.FP32])
@pytest.mark.parametrize("n,hidden", [(3, 1152), (2, 1536), (2, 2048), (3, 2560), (1285, 3072), (2, 4096)])
def test_codes_of_wide_rows(n, hidden, h_dtype):
    """Through a block's first stage: the codes and scales of LayerNorm + modulation against the reference quantiser on the float64 result."""
    heads, mlp = hidden // 128, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(hidden)
    norm = lambda *s, dt=torch.float32, k=1.0: (torch.empty(s, device="cuda").normal_(generator=g) * k).to(dt)
    ctx = rg.Context(hidden, heads, 128, mlp, n, 16)
    t = {}
    for name, (a, b) in {"w_1": (3 * hidden + mlp, hidden), "w_2": (hidden, hidden + mlp)}.items():
        t[name], t["b" + name[1:]] = norm(a, b, dt=torch.bfloat16, k=0.02), norm(a)
    t["shift1"], t["scale1"], t["gate1"] = norm(hidden, k=0.1), norm(hidden, k=0.1), norm(hidden)
    w8, held = rg.make_stream_weights_fp8(ctx, t)
    bw, bw8 = rg.BlockWeights(), rg.BlockWeightsFp8()
    packed = {k: (rg.pack_weight(ctx, v) if k.startswith("w_") else v) for k, v in t.items()}
    bw.img, bw8.img = rg.make_stream_weights(packed), w8
    h = norm(n, hidden, dt=torch.bfloat16 if h_dtype == rg.BF16 else torch.float32)
    out = torch.zeros_like(h)
    taps = rg.Fp8Taps()
    codes, scale = torch.zeros((n, hidden), dtype=torch.uint8, device="cuda"), torch.zeros(n, device="cuda")
    taps.u1_codes, taps.u1_scale = codes.data_ptr(), scale.data_ptr()
    rg.regione_block_forward_fp8(ctx, bw, bw8, rg.BLOCK_SINGLE, h, out, h_dtype, n, 0, None, 0, None, None, 0, 0, taps)
    torch.cuda.synchronize()
    x = h.double()
    u = (x - x.mean(1, keepdim=True)) / torch.sqrt(x.var(1, unbiased=False, keepdim=True) + 1e-6) * (1 + t["scale1"].double()) + t["shift1"].double()
    want_codes, want_scale = f8.quantize_rows(u.float().cpu().numpy())
    # as in test_gpu_block_fp8.py: float32 against float64 moves the scale by a few 2^-24 and a value on a rounding boundary by one code
    got = codes.cpu().numpy()
    assert abs(scale.cpu().numpy() / want_scale - 1).max() <= 2e-5
    differ = got != want_codes
    a, b = f8.e4m3_decode(got[differ]), f8.e4m3_decode(want_codes[differ])
    assert differ.mean() < 1e-3 and (abs(a - b) <= 2.0 * f8.e4m3_half_step(b)).all()
    ctx.close()
