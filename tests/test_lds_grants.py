"""No launch asks for more than 64 KiB of LDS, its own and what it gets at run time together, that was not granted for its kernel before (hipFuncAttributeMaxDynamicSharedMemorySize): the
runtime may refuse such a launch.  Blocks of every kind at sizes that take every form of product and attention."""
import pytest

from paper_2510_25590_amd import binding as rg
import launch_recorder


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


def own_lds(kernel):
    """LDS that a kernel has beside what its launch asks for: partial sums [8 waves][rows][columns + 4] of the float32 products."""
    for name in ("gemm_f32_kernel", "gemm_f32_pair_kernel"):
        if f"{name}<" in kernel:
            rb, cb = (int(x) for x in kernel.split("<", 1)[1].split(",")[1:3])
            return 8 * 16 * rb * (16 * cb + 4) * 4
    return 0


@pytest.mark.parametrize("hidden,heads,mlp,dtype,fp8", [(256, 4, 1024, rg.FP32, 0), (512, 8, 2048, rg.FP32, 0), (448, 7, 1280, rg.FP32, 0), (1024, 8, 4096, rg.FP32, 0), (256, 4, 1024, rg.BF16, 0),
                                                        (1024, 8, 4096, rg.BF16, 0), (3072, 24, 12288, rg.BF16, 0), (3072, 24, 12288, rg.BF16, 1), (256, 4, 1024, rg.BF16, 1)])
def test_launches_are_granted_their_lds(run, hidden, heads, mlp, dtype, fp8):
    commands = [f"context {hidden} {heads} {hidden // heads} {mlp} 9000 16 {dtype}"]
    for n_txt, n_img in [(0, 1), (0, 36), (0, 100), (0, 150), (0, 205), (0, 820), (0, 2048), (0, 8704), (16, 36), (33, 100), (64, 130), (128, 300), (128, 820), (512, 2048)]:
        for kind in (rg.BLOCK_DOUBLE, rg.BLOCK_SINGLE):
            commands += [f"block {kind} {n_txt} {n_img} {dtype} {rg.FLAG_RETRIEVE} {n_txt + n_img + 700} {fp8}", f"block {kind} {n_txt} {n_img} {dtype} {rg.FLAG_STORE} {n_txt + n_img} {fp8}"]
    granted, most = {}, 0
    for command, (grants, launches) in zip(commands, run(commands)):
        for n, kernel in grants:
            granted[kernel] = max(n, granted.get(kernel, 0))
        assert launches or not command.startswith("block")
        for _, lds, kernel in launches:
            total = lds + own_lds(kernel)
            most = max(most, total)
            assert total <= 65536 or granted.get(kernel, 0) >= lds, (command, total, kernel)
    assert (most > 65536) == (dtype == rg.BF16 or hidden <= 512)        # float32 rows of more than 512 values have a launch of their own
