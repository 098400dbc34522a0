"""The activation in the products' epilogues, by the few-row kernel and by a tile kernel, on values handed in through the bias: the whole range, where the exponential
overflows, infinities and NaN."""
import numpy as np
import pytest
import torch

from paper_2510_25590_amd import binding as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [0, 222])
def test_activation_over_the_whole_range(tile):
    special = [0.0, -0.0, np.inf, np.nan, 1e-30, -1e-30, 1e19, -1e19, 3e38, -3e38, 13.0, -13.0, -14.5]
    special += [1.5e-38, -1.5e-38, 1e-40, -3e-45]
    near = np.linspace(-13.05, -12.9, 64)              # the divisor's reciprocal is below the smallest normal number, or the divisor infinite
    b = np.concatenate([np.array(special, np.float32), near, np.linspace(-16, 16, 512 - len(special) - len(near))]).astype(np.float32)
    n, k, m = len(b), 64, 3
    ctx = rg.Context(256, 4, 64, 1024, 16, 16)
    x = torch.zeros((m, k), dtype=torch.bfloat16, device="cuda")
    w = rg.pack_weight(ctx, torch.ones((n, k), dtype=torch.bfloat16, device="cuda"))
    y = torch.zeros((m, n), dtype=torch.float32, device="cuda")
    rg.regione_tune_gemm(ctx, tile, 1 if tile else 0)
    rg.regione_linear(ctx, x, w, torch.from_numpy(b).cuda(), m, n, k, rg.ACT_GELU_TANH, rg.FP32, y)
    got = y.cpu().numpy().astype(np.float64)
    ctx.close()
    v = b.astype(np.float64)
    with np.errstate(over="ignore", invalid="ignore"):
        u = np.sqrt(2 / np.pi) * (v + 0.044715 * v ** 3)
        want = v / (1 + np.exp(-2 * u))
    want[np.isposinf(v)] = np.inf
    assert np.array_equal(got[0], got[1], equal_nan=True) and np.array_equal(got[0], got[2], equal_nan=True)
    assert np.array_equal(np.isnan(got[0]), np.isnan(v)) and np.array_equal(np.isposinf(got[0]), np.isposinf(v))
    ok = np.isfinite(v)
    # The exponent 2u carries a few roundings of 2^-24 each, the exponential and the quotient one more each; where the exponential overflows (2u log2(e) of -128, less its own roundings) the
    # result is zero, and a quarter of a denormal x may lose a bit.
    overflow = -2 * u[ok] * np.log2(np.e) >= 128 * (1 - 2.0 ** -20)
    bound = np.abs(want[ok]) * (8 * np.minimum(np.abs(u[ok]), 50) + 4) * 2.0 ** -24 + np.abs(want[ok]) * overflow + 2.0 ** -149
    assert np.all(np.abs(got[0][ok] - want[ok]) <= bound)
