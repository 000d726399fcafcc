"""Backward on either side of the rule that gives a walk two waves or four: four with few row tiles (lists shorter and longer than
four tiles, a last tile of one row, a slot walk of one tile), two waves that share a row tile's walk and two with a
row tile each where workgroups are many.  Every element against the fp64 oracle, bounds of test_gpu_parity_grad.py."""
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import rnd  # noqa: E402
from tests.test_gpu_parity_fine_mass import small_pair  # noqa: E402
from tests.test_gpu_parity_grad import backward_both, gpu  # noqa: E402,F401

pytestmark = pytest.mark.gpu

CASES = [
    # name,          H, d,   B,   Nq,   w, C, k, n_sink, causal, p_lens
    ("four_1_row",   2, 64,  128, 1,    1, 2, 2, 0, 1, [128, 65]),
    ("four_5",       9, 64,  128, 305,  1, 5, 5, 0, 1, [128, 64, 1, 0, 65]),
    ("four_7",       3, 128, 128, 420,  1, 1, 3, 0, 0, [97]),
    ("four_long",    2, 128, 64,  200,  1, 30, 2, 0, 1, [64, 33] * 15),
    ("two_1_row",    16, 64, 64,  193,  2, 4, 2, 0, 1, [64, 7, 0, 64]),
    ("two_shared",   16, 128, 64, 320,  2, 5, 1, 0, 0, [64, 0, 31, 32, 33]),
    ("two_128",      16, 64, 128, 257,  2, 3, 1, 0, 1, [127, 64, 128]),
    ("two_pairs",    16, 128, 64, 1030, 1, 2, 1, 0, 1, [64, 9]),
    ("two_pairs_64", 16, 64, 128, 1090, 1, 1, 1, 0, 0, [70]),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_backward_two_waves_and_four(gpu, case):  # noqa: F811
    st, c = small_pair(gpu, case)
    name, H, d, B, Nq, w = case[:6]
    for g in range(w + 1):
        Q, K, V = rnd(160 + 3 * g, H, Nq, d), rnd(161 + 3 * g, H, Nq, d, scale=1.5), rnd(162 + 3 * g, H, Nq, d)
        heads = None if g == w and Nq < 500 else [0, H - 1]
        backward_both(gpu, c, st, Q, K, V, g, f"bwd waves {name}", heads)
        if g < w:                            # nothing is evicted yet: both sides only close the chunk
            st.update()
            c.update()


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_which_backward_runs(gpu, case):  # noqa: F811
    from tests.test_gpu_attention_team import kernels
    name, H, d, B, Nq, w, C, k = case[:8]
    print(f"[case] bwd route {name}", flush=True)
    c = gpu["cache"].PbsaCache(H, d, B, Nq, w, C, k, d ** -0.5, causal=case[9], device="cuda:0")
    for g in range(w + 1):
        c.adopt_chunk(g)
    Q = torch.zeros(H, Nq, d, dtype=torch.bfloat16, device="cuda:0")
    c.select(Q)
    lse = torch.zeros(H, Nq, device="cuda:0")
    O = c.attention(Q, lse=lse)
    names = kernels(lambda: c.attention_bwd(Q, O, Q, lse))
    assert f", {4 if name.startswith('four') else 2}>" in next(n for n in names if "bwd_walk_kernel" in n), names


LINES = [
    ("four_past",    12, 64, 128, 205,  1, 40, 2, 0, 1, [128, 64] * 20),   # few row tiles, though the places set the end
    ("four_24_rows", 9, 64,  64,  1500, 0, 4, 3, 0, 1, [64, 7, 0, 64]),
    ("two_25_rows",  9, 128, 64,  1549, 0, 3, 3, 0, 1, [64, 9, 33]),      # many, and the places set it
    ("two_512",      8, 64,  128, 970,  1, 7, 1, 0, 0, [70] * 7),
]


@pytest.mark.parametrize("case", LINES, ids=[c[0] for c in LINES])
def test_backward_at_the_models_lines(gpu, case):  # noqa: F811
    test_which_backward_runs(gpu, case)
    test_backward_two_waves_and_four(gpu, case)
