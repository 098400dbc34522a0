"""Which kernels a storing forward's K and V come from, seen in the launches underneath a stand-in for the HIP runtime: the LayerNorm of a wave per row and the tile and K splits that
regione_gemm_plan_host names for REGIONE_GEMM_BF16_STORED; other forwards of the same rows, and the block's other products, take the general choice."""
import os
import re

import pytest

from paper_2510_25590_amd import binding as rg
import launch_recorder

CSRC = os.path.join(launch_recorder.ROOT, "paper_2510_25590_amd", "csrc")
TILES = {int(c): (k, tuple(int(x) for x in args.split(","))) for f in os.listdir(CSRC) if re.fullmatch(r"gemm_tiles_(128|96|kg|wide)\.hip", f)
         for c, k, args in re.findall(r"RG_TILE\((\d+), launch_(kg|pp), ([\d, ]+)\)", open(os.path.join(CSRC, f)).read())}
QKV = 1


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


def launch_of(m, n, k, plan, kind):
    """(workgroups, beginning of the kernel's name) of a product's launch"""
    tile, splits = plan
    family, args = TILES[tile]
    rows, cols = (32 * args[0], 64 * args[1]) if family == "pp" else (args[0] * 16 * args[2], args[1] * 16 * (4 // args[2]))
    units = -(-m // rows) * -(-n // cols) * splits
    return (units + 7) // 8 * 8, f"gemm_{family}_kernel<{', '.join(map(str, args + (kind,)))}"


@pytest.mark.parametrize("hidden,n", [(1024, 2500), (1152, 4000), (2048, 1300), (3072, 820), (3072, 1640), (3072, 2048), (3072, 4608), (3072, 8704), (4096, 1382)])
@pytest.mark.parametrize("kind", [rg.BLOCK_DOUBLE, rg.BLOCK_SINGLE])
def test_storing_forward(run, hidden, n, kind):
    mlp = 1024
    columns = 3 * hidden + (mlp if kind == rg.BLOCK_SINGLE else 0)
    kept, general = (rg.regione_gemm_plan_host(n, columns, hidden, k) for k in (rg.GEMM_BF16_STORED, rg.GEMM_BF16))
    out = run([f"context {hidden} {hidden // 128} 128 {mlp} {n} 16 {rg.BF16}"] + [f"block {kind} 0 {n} {rg.BF16} {flag} {n_all} 0" for flag, n_all in ((rg.FLAG_STORE, n), (rg.FLAG_RETRIEVE, n + 64))])
    for (_, launches), plan, rounds in ((out[1], kept, 4 if hidden <= 2048 else 6 if hidden <= 3072 else 8), (out[2], general, 0)):
        (_, _, norm), (grid, _, product) = launches[:2]
        if hidden <= 1024:
            assert "layernorm_mod_vec_kernel" in norm and ", 2>(" in norm
        elif rounds:
            assert "layernorm_mod_vec_kernel" in norm and f", {rounds}>(" in norm
        else:
            assert "layernorm_mod_wide_kernel" in norm
        workgroups, name = launch_of(n, columns, hidden, plan, QKV)
        assert name in product and grid[0] == workgroups, (plan, product, grid)
        later = [name for _, _, name in launches[2:] if "layernorm" in name]
        assert len(later) == (kind == rg.BLOCK_DOUBLE) and all(("layernorm_mod_wide_kernel" in name) == (hidden > 1024) for name in later)


def test_the_two_choices_differ_somewhere():
    """8704 rows of a 3072-wide model among them; below a tile's worth of rows both are the kernel of few rows."""
    plans = [tuple(rg.regione_gemm_plan_host(m, 9216, 3072, k) for k in (rg.GEMM_BF16_STORED, rg.GEMM_BF16)) for m in (12, 2048, 8704)]
    assert plans[0][0] == plans[0][1] == (0, 1) or plans[0][0][0] in TILES
    assert any(a != b for a, b in plans[1:])
