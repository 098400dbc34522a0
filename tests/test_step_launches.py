"""The launches of a region step underneath a stand-in for the HIP runtime: what is queued before the count of edited tokens is known, and what a step that is refused has launched."""
import re

import pytest

from paper_2510_25590_amd import binding as rg
import launch_recorder

D, S = rg.BLOCK_DOUBLE, rg.BLOCK_SINGLE


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


def names(launches):
    return [re.match(r"(?:void )?\(anonymous namespace\)::(\w+)", name).group(1) for _, _, name in launches]


@pytest.mark.parametrize("types", [[D], [S] * 16, [D] * 19 + [S] * 13])
@pytest.mark.parametrize("n_txt", [0, 24])
def test_modulation_launches(run, types, n_txt):
    sets = sum(2 if t == D and n_txt else 1 for t in types)
    head = f"context 3072 24 128 256 4200 4096 {rg.BF16}"
    tail = f"4096 64 {n_txt} {rg.BF16} {' '.join(map(str, types))}"
    (_, empty), (_, full) = run([head, f"step 0 {tail}", f"step 820 {tail}"])[1:]
    assert names(empty) == ["score_bits_kernel", "write_index_kernel", "vec_linear_batch_kernel"]
    assert "(VecBatch, int, int const*)" in full[2][2] and full[2][0][0] <= 16 * 6 * 3072 // 16
    assert sets / 16 <= names(full).count("vec_linear_batch_kernel") <= sets / 15 + 1 and "vec_linear_kernel" not in names(full)


@pytest.mark.parametrize("types", [[5], [S, 7]])
def test_unknown_block_types_read_no_matrix(run, types):
    """Whether a modulation matrix has 3 or 6 rows of vectors is not known for a block of no type."""
    _, (_, launches, answer) = run([f"context 256 4 64 256 300 256 {rg.BF16}", f"step 40 256 64 0 {rg.BF16} {' '.join(map(str, types))}"], refused=True)
    assert answer.startswith("-") and "bad block type" in answer
    known = types.count(S)
    batches = [grid for (grid, _, name) in launches if "vec_linear_batch_kernel" in name]
    assert [grid[0] for grid in batches] == [3 * 256 // 16] * known
