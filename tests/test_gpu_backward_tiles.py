"""Backward where its kernels' tiles, lists and workgroup order can go wrong, every element against the fp64 oracle: a last
row tile of 1, 31, 32, 33 and 63 rows (half tiles with no row, one row, all but one), one, three and nine heads (fewer and
more than the eight dies the grid is dealt over), more query blocks than one word of the turned-around selection holds,
blocks that every row, few rows and no row selected, and either side of the lines at which the launch is set up differently.
Bounds: those of test_gpu_parity_grad.py, derived there."""
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import rnd  # noqa: E402
from tests.test_gpu_parity_fine_mass import small_pair  # noqa: E402
from tests.test_gpu_parity_grad import backward_both, gpu  # noqa: E402,F401

pytestmark = pytest.mark.gpu

CASES = [
    # name,        H, d,   B,   Nq,   w, C, k, n_sink, causal, p_lens
    ("rows1",      1, 128, 64,  65,   1, 2, 2, 0, 1, [64, 33]),
    ("rows31",     3, 64,  64,  159,  1, 1, 2, 0, 0, [31]),
    ("rows32",     3, 128, 128, 160,  1, 2, 1, 0, 1, [128, 97]),
    ("rows33",     9, 64,  64,  97,   1, 2, 3, 0, 1, [1, 64]),
    ("rows63",     9, 128, 64,  127,  0, 1, 1, 0, 1, [32]),
    ("two_words",  1, 64,  64,  2113, 0, 1, 3, 0, 0, [64]),
    ("three_words", 2, 128, 64, 4100, 0, 1, 2, 0, 1, [64]),
    # up to 256 row tiles in all and fewer than eight per head, two waves share a row tile's walk: a walk of one tile leaves
    # one of them nothing
    ("one_tile",   1, 128, 64,  70,   0, 1, 1, 0, 1, [0]),
    ("three_tiles", 2, 64, 64,  130,  0, 2, 1, 0, 0, [64, 3]),
    # up to 448 workgroups of row tiles and key tiles, eight row tiles or more per head: four waves share a walk, of one tile,
    # of a few, of many, the last one ragged; just above, two share it again
    ("four_one",   1, 64,  64,  520,  0, 1, 1, 0, 1, [0]),
    ("four_few",   2, 128, 128, 1100, 0, 2, 1, 0, 0, [128, 5]),
    ("four_many",  1, 128, 64,  650,  1, 3, 9, 0, 1, [64, 1, 0]),
    ("two_above",  9, 64,  64,  1600, 0, 1, 1, 0, 1, [64]),
    # more than 256: a row tile per wave, an odd number of them per head
    ("pairs_128",  9, 128, 64,  1800, 0, 1, 2, 0, 1, [64]),
    ("pairs_64",   9, 64,  128, 1830, 0, 1, 1, 0, 0, [70]),
    # d = 64, at least 820 row tiles and 64 tiles to walk (most slots empty): dq and dkv as a launch each
    ("two_launches", 13, 64, 64, 4100, 0, 62, 1, 0, 1, [64] + [0] * 60 + [7]),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_backward_tile_edges(gpu, case):  # noqa: F811
    st, c = small_pair(gpu, case)
    name, H, d, B, Nq, w = case[:6]
    for g in range(w + 1):
        Q, K, V = rnd(140 + 3 * g, H, Nq, d), rnd(141 + 3 * g, H, Nq, d, scale=1.5), rnd(142 + 3 * g, H, Nq, d)
        backward_both(gpu, c, st, Q, K, V, g, f"bwd tiles {name}")
        if g < w:                            # nothing is evicted yet: both sides only close the chunk
            st.update()
            c.update()
