"""The tile that a product gets by itself: a pure host function, checked without a GPU."""
import pytest

from paper_2510_25590_amd import binding as rg

# code: rows, columns, waves that read fragments in a step, 16-row and 16-column fragments of a wave
E4M3 = {42: (128, 128, 8, 4, 2), 62: (192, 128, 8, 6, 2), 82: (256, 128, 8, 8, 2), 44: (128, 256, 8, 4, 4),
        54: (160, 256, 8, 5, 4), 64: (192, 256, 8, 6, 4), 74: (224, 256, 8, 7, 4), 84: (256, 256, 8, 8, 4),
        222: (64, 64, 4, 2, 2), 224: (64, 128, 4, 2, 4), 274: (224, 128, 4, 7, 4), 426: (128, 96, 4, 2, 6), 446: (256, 96, 4, 4, 6)}


@pytest.mark.parametrize("m", [2924, 3000, 4096, 6000, 8704, 19456])
@pytest.mark.parametrize("n,k", [(9216, 3072), (3072, 3072), (12288, 3072), (3072, 12288), (21504, 3072), (4096, 4096)])
def test_many_e4m3_rows_do_not_wait_for_the_lds(m, n, k):
    """With tiles whose waves own 128 x 32 the LDS is busy for 1.6 times the MFMAs' cycles, and such products lost 13 %."""
    tile, splits = rg.regione_gemm_plan_host(m, n, k, rg.GEMM_E4M3)
    rows, cols, waves, rf, cf = E4M3[tile]
    mfma, lds = rows * cols / 32, waves * 16 * (rf + cf) + rows + cols      # cycles of a step; 128 bytes a cycle, rows of 128 bytes
    assert splits == 1 and lds <= 1.3 * mfma, tile


@pytest.mark.parametrize("m", [1, 12, 46, 64])
@pytest.mark.parametrize("n,k", [(9216, 3072), (2117, 5120), (4096, 1024), (1024, 4096)])
def test_few_e4m3_rows_get_the_smallest_tile(m, n, k):
    """A tile of 128 rows leaves half the CUs without work and copies twice the latency chain: 13.2 us became 16.3 at 12 x 9216 x 3072."""
    assert rg.regione_gemm_plan_host(m, n, k, rg.GEMM_E4M3)[0] == 222


@pytest.mark.parametrize("m,n,k,good", [
    # us of the best plan, of 242/2 and of 242/3: 13.2, 15.5, - and 10.5, -, 12.9
    (1458, 512, 2560, [(222, 1)]), (1209, 512, 2048, [(222, 1)]),
    # 224/1 13.7 and 11.0, 242/1 15.3 and 11.2
    (2256, 512, 2048, [(224, 1)]), (6277, 256, 1280, [(224, 1), (242, 1)]),
    # 64/1 against 276/1: 12.3 / 13.8, 20.8 / 24.2, 12.2 / 13.6, 27.7 / 31.0, 27.8 / 31.1, 15.8 / 16.8, 15.3 / 16.8
    (9358, 1024, 256, [(64, 1)]), (10085, 1792, 256, [(64, 1)]), (12625, 768, 256, [(64, 1)]), (13106, 1536, 512, [(64, 1)]), (9960, 2048, 512, [(64, 1)]),
    (2860, 3584, 512, [(64, 1)]), (18356, 512, 512, [(64, 1)])])
def test_short_and_narrow_bf16_products(m, n, k, good):
    """Below 1024 columns or K, plans within 3 % of the best of all that were timed: constants fitted to larger products alone were up to 22 % behind here."""
    assert rg.regione_gemm_plan_host(m, n, k, rg.GEMM_BF16) in good


def test_plan_arguments():
    for bad in ((0, 8, 64, 0), (8, 0, 64, 0), (8, 8, 0, 0), (8, 8, 64, 7), (8, 8, 96, 0), (8, 8, 64, 1)):
        with pytest.raises(rg.RegionEError):
            rg.regione_gemm_plan_host(*bad)
    assert rg.regione_gemm_plan_host(820, 64, 3072, rg.GEMM_BF16)[0] == 0      # the kernel of narrow results
    # a split never needs more than the workspace it is told of
    for m in (5, 100, 820):
        assert rg.regione_gemm_plan_host(m, 3072, 12288, rg.GEMM_BF16, 0)[1] == 1
