"""The attention's tile list on either side of what a workgroup fetches in one round: 384 local blocks, 128 slots, 256 selected
blocks of its one or two query blocks; an odd number of query blocks, so that the last workgroup has one."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from harness import synth  # noqa: E402
from oracle.rollout import OracleState  # noqa: E402
from tests.test_gpu_parity import DEV, gpu, rnd, run_both, sample_rows  # noqa: E402,F401

pytestmark = pytest.mark.gpu

CASES = [
    # d, B, query blocks, window chunks, C, k
    (64, 64, 48, 7, 127, 128),               # 384 blocks, 128 slots, 256 selected
    (64, 64, 43, 8, 128, 129),               # 387, 129, 258
    (128, 128, 35, 10, 129, 257),            # 385, 130, 257 by one query block
]


@pytest.mark.parametrize("case", CASES, ids=["%d_blocks_%d_slots_k%d" % (c[2] * (c[3] + 1), c[4] + 1, c[5]) for c in CASES])
def test_list_round_edges(gpu, case):  # noqa: F811
    d, B, nqb, w, C, k = case
    H, Nq, scale = 1, nqb * B - 17, np.float32(1.0 / math.sqrt(d))
    st = OracleState(H, d, B, Nq, w, C, k, scale, fold=False)
    c = gpu["cache"].PbsaCache(H, d, B, Nq, w, C, k, scale, fold=False, device=DEV)
    Kp, Vp = rnd(1, H, C, B, d), rnd(2, H, C, B, d)
    pl = np.full((H, C), B, np.int32)
    pl[:, 5], pl[:, 6], pl[:, -1] = 3, 0, B - 1
    ids = -100 - np.arange(C)[None, :].repeat(H, 0)
    st.set_persistent(Kp, Vp, pl, ids)
    c.set_persistent(gpu["wl"].bf16_tensor(Kp, DEV), gpu["wl"].bf16_tensor(Vp, DEV), torch.from_numpy(pl).to(DEV), torch.from_numpy(ids))
    lens = np.full(nqb, B, np.int32)
    lens[-1] = Nq - (nqb - 1) * B
    for g in range(w):
        Kw, Vw = rnd(700 + 2 * g, H, Nq, d, scale=1.5), rnd(701 + 2 * g, H, Nq, d)
        st.append_chunk(synth.to_blocks(Kw, B), synth.to_blocks(Vw, B), lens, g * nqb + np.arange(nqb))
        c.append_chunk(gpu["wl"].bf16_tensor(Kw, DEV), gpu["wl"].bf16_tensor(Vw, DEV), g)
    Q, K, V = rnd(790, H, Nq, d), rnd(791, H, Nq, d, scale=1.5), rnd(792, H, Nq, d)
    run_both(gpu, c, st, Q, K, V, w, sample_rows(H, Nq, B, per_head=24, seed=5), f"list edges {case}", update=False)
