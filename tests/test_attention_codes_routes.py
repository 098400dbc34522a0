"""The calls of test_gpu_fp8_attention_codes.py that are meant to reach each kernel that merges key ranges and forms the E4M3 codes of the rows do so, seen in the launches underneath a
stand-in for the HIP runtime."""
import pytest

from paper_2510_25590_amd import binding as rg
import launch_recorder
from test_gpu_fp8_attention_codes import MERGES


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


@pytest.mark.parametrize("arguments", sorted(MERGES))
def test_route(run, arguments):
    for heads, n, n_all in MERGES[arguments]:
        _, (_, launches) = run([f"context {128 * heads} {heads} 128 256 {n} 16 {rg.BF16}", f"block {rg.BLOCK_DOUBLE} 0 {n} {rg.BF16} {rg.FLAG_RETRIEVE} {n_all} 1"])
        names = [name for _, _, name in launches]
        assert sum(f"attn_combine_codes_kernel{arguments}" in name for name in names) == 1 and not any("quantize" in name for name in names[:4]), names
