"""Selection where its instances and its pooling can go wrong, bit for bit against the oracle: 1 to 672 local blocks (each of the
kernel's column counts, its smallest and its largest), the newest chunk's last block of 1 token to a whole one (at d = 64 two
blocks share a wave: a whole and a short one together), pooled by the selection and in its own launch, and values whose
logits overflow, are denormal or tie.  A logit is a chain of fused multiply-adds in one fixed order, so every bit is fixed."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from harness import synth  # noqa: E402
from oracle.rollout import OracleState  # noqa: E402
from tests.test_gpu_parity import DEV, compare_select, gpu, rnd  # noqa: E402,F401

pytestmark = pytest.mark.gpu

CASES = [
    # d, B, query blocks, tokens of the last one, window chunks, k
    (64, 64, 1, 1, 0, 1), (64, 64, 3, 63, 1, 2), (64, 128, 4, 64, 0, 4), (64, 128, 5, 65, 2, 3), (64, 128, 2, 127, 1, 9),
    (128, 64, 2, 33, 2, 3), (128, 128, 3, 1, 0, 2), (128, 128, 4, 104, 1, 5), (128, 128, 6, 128, 0, 6),
    (64, 64, 43, 64, 2, 17), (128, 64, 43, 7, 2, 40), (128, 64, 81, 64, 3, 12), (64, 64, 81, 31, 3, 324),
    (64, 64, 161, 50, 1, 9), (128, 64, 161, 64, 3, 33),
    (64, 64, 168, 50, 3, 9), (128, 64, 168, 1, 3, 40),
]


def logits_and_sets(gpu, d, B, nqb, tail, w, k, scale_qk, values):  # noqa: F811
    H, Nq, scale = 2, (nqb - 1) * B + tail, np.float32(1.0 / math.sqrt(d))
    C = 1 if (w + 1) * nqb <= gpu["pbsa"].PBSA_MAX_N_LOC_AUX else gpu["pbsa"].PBSA_MAX_C + 1      # beyond: no update's workspace
    st = OracleState(H, d, B, Nq, w, C, k, scale, fold=False)
    c = gpu["cache"].PbsaCache(H, d, B, Nq, w, C, k, scale, fold=False, device=DEV)
    lens = np.full(nqb, B, np.int32)
    lens[-1] = tail
    for g in range(w + 1):
        Q, K, V = values(500 + 3 * g, H, Nq, d, scale_qk), values(501 + 3 * g, H, Nq, d, scale_qk), rnd(502 + 3 * g, H, Nq, d)
        st.append_chunk(synth.to_blocks(K, B), synth.to_blocks(V, B), lens, g * nqb + np.arange(nqb))
        c.append_chunk(gpu["wl"].bf16_tensor(K, DEV), gpu["wl"].bf16_tensor(V, DEV), g)
    _, Z = st.select(Q, want_logits=True)
    c.select(gpu["wl"].bf16_tensor(Q, DEV))
    what = f"d{d} B{B} {nqb} blocks, last {tail}, window {w}, k {k}"
    compare_select(c, st, what)
    if c.Zl is not None:
        got = c.Zl.view(-1)[:Z.size].cpu().numpy().reshape(Z.shape)
        seen = np.arange(st.n_loc)[None] <= st.n_loc - nqb + np.arange(nqb)[:, None]     # the oracle leaves the others out
        assert np.array_equal(got.view(np.uint32)[:, seen], Z.view(np.uint32)[:, seen]), f"{what}: logits differ"


@pytest.mark.parametrize("case", CASES, ids=[f"d{c[0]}_B{c[1]}_{c[2]}x{c[4] + 1}_last{c[3]}_k{c[5]}" for c in CASES])
def test_selection_every_bit(gpu, case):  # noqa: F811
    logits_and_sets(gpu, *case, 1.0, lambda key, H, Nq, d, s: rnd(key, H, Nq, d, scale=s))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["denormal", "overflow", "ties", "infinite"])
def test_selection_of_unusual_values(gpu, d, kind):  # noqa: F811
    if kind == "infinite":                   # in one dimension, of one query block and of every third key block: no NaN arises
        def values(key, H, Nq, dd, s):
            x = rnd(key, H, Nq, dd)
            if key % 3 == 500 % 3:
                x[:, 2 * 64 + 5, 7] = 0x7F80
            else:
                x[:, 3::3 * 64, 7], x[:, 64 + 3::6 * 64, 7] = 0x7F80, 0xFF80
            return x
        logits_and_sets(gpu, d, 64, 9, 60, 2, 6, 1.0, values)
        logits_and_sets(gpu, d, 64, 45, 60, 2, 21, 1.0, values)
    elif kind == "ties":                       # few distinct values: many logits are equal, many are zero of either sign
        values = lambda key, H, Nq, dd, s: synth.to_bf16_bits(np.round(synth.normals(synth.stream_key(9, "misc", key), H * Nq * dd)).reshape(H, Nq, dd) * 0)  # noqa: E731
        logits_and_sets(gpu, d, 64, 7, 64, 1, 5, 1.0, values)
        values = lambda key, H, Nq, dd, s: synth.to_bf16_bits(np.repeat(np.sign(synth.normals(synth.stream_key(9, "misc", key), H * Nq)).reshape(H, Nq, 1), dd, 2))  # noqa: E731
        logits_and_sets(gpu, d, 64, 7, 64, 1, 5, 1.0, values)
    else:
        s = 2.0 ** -68 if kind == "denormal" else 2.0 ** 62      # products around the smallest normal; sums near the largest number
        logits_and_sets(gpu, d, 64, 9, 60, 2, 6, s, lambda key, H, Nq, dd, sc: rnd(key, H, Nq, dd, scale=sc))


@pytest.mark.parametrize("case", [(64, 64, 3, 1, 2), (64, 128, 5, 104, 1), (128, 64, 4, 64, 2), (128, 128, 3, 127, 1), (64, 64, 201, 9, 0)],
                         ids=lambda c: "d%d_B%d_%d_blocks_last%d" % c[:4])
def test_queries_pooled_with_the_append(gpu, case):  # noqa: F811
    """A step (queries pooled by the append where the launch is small: 2 heads of up to 200 blocks; strided as a model has them)
    against append and select by themselves: every bit of what the selection leaves."""
    d, B, nqb, tail, w = case
    H, Nq, scale = 2, (nqb - 1) * B + tail, np.float32(1.0 / math.sqrt(d))
    one, two = (gpu["cache"].PbsaCache(H, d, B, Nq, w, 3, 4, scale, device=DEV) for _ in range(2))
    for g in range(w + 2):
        Q, K, V = (gpu["wl"].bf16_tensor(rnd(900 + 3 * g + i, Nq, H, d), DEV).transpose(0, 1) for i in range(3))
        one.step(Q, K, V, g)
        two.append_chunk(K, V, g)
        two.select(Q)
        n = H * nqb * two.n_loc
        for name in ("Qc", "Kc_l", "sel"):
            a, b = (getattr(c, name).cpu().numpy() for c in (one, two))
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), f"chunk {g}: {name}"
        a, b = (c.Zl.view(-1)[:n].cpu().numpy().view(np.uint32) for c in (one, two))
        assert np.array_equal(a, b), f"chunk {g}: logits"
        two.attention(Q)
        two.update()
        assert np.array_equal(one.slot_src.cpu().numpy(), two.slot_src.cpu().numpy()), f"chunk {g}: slots"


@pytest.mark.parametrize("case", [(64, 64, 1, 1, 0), (64, 64, 12, 9, 4), (64, 64, 13, 64, 2), (64, 128, 5, 65, 3), (128, 64, 12, 64, 1),
                                  (128, 64, 5, 3, 31), (128, 128, 4, 127, 4), (128, 128, 5, 128, 1)],
                         ids=lambda c: "d%d_B%d_%d_blocks_last%d_w%d" % c)
def test_keys_pooled_by_the_selection(gpu, case):  # noqa: F811
    """A chunk whose stale keys the selection pools itself (up to 12 blocks and 256 KiB with the queries; 13 and more are pooled by
    a launch ahead), in a chained step with the update before it in the same launch, and after rewriting: every bit of what
    a step with everything pooled by its append leaves."""
    d, B, nqb, tail, w = case
    H, Nq, scale = 3, (nqb - 1) * B + tail, np.float32(1.0 / math.sqrt(d))
    one = gpu["cache"].PbsaCache(H, d, B, Nq, w, 3, 4, scale, device=DEV)
    two = gpu["cache"].PbsaCache(H, d, B, Nq, w, 3, 4, scale, device=DEV, ring_chunks=w + 2)
    for g in range(w + 3):
        Q, K, V = (gpu["wl"].bf16_tensor(rnd(950 + 3 * g + i, Nq, H, d), DEV).transpose(0, 1) for i in range(3))
        one.step(Q, K, V, g)
        two.append_chunk(V, K, g)            # as it was before a denoising pass
        if two._pending is None:
            two.select(K)
        two.rewrite_chunk(K, V)
        two.select(Q)
        two.attention_with_plan(Q)
        two.defer_apply()
        n = H * nqb * (len(one.chunk_pos) + (one.n_appended > w)) * nqb
        for name in ("Qc", "sel", "slot_src", "scores", "Kc_p", "S_cnt"):
            a, b = (getattr(c, name).cpu().numpy() for c in (one, two))
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), f"chunk {g}: {name}"
        a, b = (c.Zl.view(-1)[:n].cpu().numpy().view(np.uint32) for c in (one, two))
        assert np.array_equal(a, b), f"chunk {g}: logits"
    two.flush()
    for name in ("Kp", "Vp", "p_len", "S_sum"):
        a, b = (getattr(c, name).cpu() for c in (one, two))
        assert torch.equal(a, b), name


@pytest.mark.parametrize("case", [(64, 128, 4, 1, 2, 3), (128, 64, 8, 64, 1, 3), (128, 64, 9, 64, 1, 3), (128, 128, 4, 128, 2, 3),
                                  (64, 64, 1, 64, 1, 51), (64, 64, 1, 64, 1, 52), (64, 64, 1, 5, 1, 128), (64, 64, 1, 5, 1, 129),
                                  (64, 64, 1, 5, 1, 256), (64, 64, 1, 5, 1, 257), (64, 128, 12, 128, 1, 21), (64, 128, 12, 128, 1, 22)],
                         ids=lambda c: "d%d_B%d_%d_blocks_last%d_w%d_%d_heads" % c)
def test_keys_pooled_on_either_side_of_a_line(gpu, case):  # noqa: F811
    """A chunk whose stale keys the selection pools itself or a launch ahead of it -- up to 12 blocks, 128 KiB and 256 workgroups
    (128 with an append) or, of whole blocks, 256 KiB and 64; with the fold of the update before it in the same launch, a
    chained step, 256 KiB and 256 workgroups with those of the fold -- on either side of each line, and after rewriting:
    every bit of what a step with everything pooled by its append leaves."""
    d, B, nqb, tail, w, H = case
    Nq, scale = (nqb - 1) * B + tail, np.float32(1.0 / math.sqrt(d))
    one = gpu["cache"].PbsaCache(H, d, B, Nq, w, 3, 4, scale, device=DEV)
    two = gpu["cache"].PbsaCache(H, d, B, Nq, w, 3, 4, scale, device=DEV, ring_chunks=w + 2)
    for g in range(w + 3):
        Q, K, V = (gpu["wl"].bf16_tensor(rnd(950 + 3 * g + i, Nq, H, d), DEV).transpose(0, 1) for i in range(3))
        one.step(Q, K, V, g)
        two.append_chunk(V, K, g)            # as it was before a denoising pass
        if two._pending is None:
            two.select(K)
        two.rewrite_chunk(K, V)
        two.select(Q)
        two.attention_with_plan(Q)
        two.defer_apply()
        n = H * nqb * (len(one.chunk_pos) + (one.n_appended > w)) * nqb
        for name in ("Qc", "sel", "slot_src", "scores", "Kc_p", "S_cnt"):
            a, b = (getattr(c, name).cpu().numpy() for c in (one, two))
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), f"chunk {g}: {name}"
        a, b = (c.Zl.view(-1)[:n].cpu().numpy().view(np.uint32) for c in (one, two))
        assert np.array_equal(a, b), f"chunk {g}: logits"
    two.flush()
    for name in ("Kp", "Vp", "p_len", "S_sum"):
        a, b = (getattr(c, name).cpu() for c in (one, two))
        assert torch.equal(a, b), name


@pytest.mark.parametrize("case", [(64, 64, 4), (64, 64, 12), (128, 64, 6), (128, 128, 4)], ids=lambda c: "d%d_B%d_%d_blocks" % c)
def test_a_place_named_twice(gpu, case):  # noqa: F811
    """Older blocks in the places of blocks that the selection pools itself: their columns have the new pooled keys too, as if
    those had been pooled before."""
    d, B, nqb = case
    H, cap, pbsa = 2, 3 * nqb, gpu["pbsa"]
    K, Q = gpu["wl"].bf16_tensor(rnd(971, H, cap * B, d), DEV).view(H, cap, B, d), gpu["wl"].bf16_tensor(rnd(972, H, nqb * B, d), DEV)
    l_map = torch.arange(cap, dtype=torch.int32, device=DEV)
    l_map[0], l_map[nqb], l_map[2 * nqb - 1] = 3 * nqb - 1, 2 * nqb, 3 * nqb - 1
    l_len = torch.full((cap,), B, dtype=torch.int32, device=DEV)
    new = lambda *s, t=torch.float32, x=5.0: torch.full(s, x, dtype=t, device=DEV)  # noqa: E731
    Kc, Qc, k = new(H, cap, d), new(H, nqb, d), 5
    sel, want = (new(H, nqb, k, t=torch.int32, x=-1) for _ in range(2))
    Zl, Zw = new(H, nqb, cap), new(H, nqb, cap)
    p = pbsa.make_params(H, d, B, nqb * B, cap, cap, 1, k, np.float32(d ** -0.5), pool_from=2 * nqb)
    pbsa.pbsa_select_blocks(p, Q, K, l_len, l_map, Kc, Qc, sel, Zl)
    pbsa.pbsa_select_blocks(p, Q, K, l_len, l_map, Kc, Qc, want, Zw, pooled=True)
    assert torch.equal(Kc[:, :2 * nqb], new(H, 2 * nqb, d)) and not bool((Kc[:, 2 * nqb:] == 5.0).any())
    assert torch.equal(Zl.view(torch.int32), Zw.view(torch.int32)) and torch.equal(sel, want)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nqb", [7, 45])
def test_selection_of_nan(gpu, d, nqb):  # noqa: F811
    """NaN of either sign in a few key blocks and in a query block: logits are NaN where the chain has one and every bit of the
    others is the oracle's; a NaN ranks by its bits, above everything or below, as the numbers' order continues."""
    H, B, w, k = 2, 64, 2, 5
    Nq, scale = nqb * B, np.float32(1.0 / math.sqrt(d))
    st = OracleState(H, d, B, Nq, w, 1, k, scale, fold=False)
    c = gpu["cache"].PbsaCache(H, d, B, Nq, w, 1, k, scale, fold=False, device=DEV)
    for g in range(w + 1):
        Q, K, V = rnd(600 + 3 * g, H, Nq, d), rnd(601 + 3 * g, H, Nq, d), rnd(602 + 3 * g, H, Nq, d)
        K[:, 2 * B + 9, 5], K[:, 5 * B, d - 1], Q[:, 3 * B + 1, 11] = 0x7FC1, 0xFFC0, 0x7FC0
        st.append_chunk(synth.to_blocks(K, B), synth.to_blocks(V, B), np.full(nqb, B, np.int32), g * nqb + np.arange(nqb))
        c.append_chunk(gpu["wl"].bf16_tensor(K, DEV), gpu["wl"].bf16_tensor(V, DEV), g)
    _, Z = st.select(Q, want_logits=True)
    c.select(gpu["wl"].bf16_tensor(Q, DEV))
    got = c.Zl.view(-1)[:Z.size].cpu().numpy().reshape(Z.shape)
    seen = np.arange(st.n_loc)[None] <= st.n_loc - nqb + np.arange(nqb)[:, None]
    assert np.isnan(Z[:, seen]).any() and np.array_equal(np.isnan(got[:, seen]), np.isnan(Z[:, seen]))
    number = seen[None] & ~np.isnan(Z)
    assert np.array_equal(got.view(np.uint32)[number], Z.view(np.uint32)[number])
    bits = (got + np.float32(0)).view(np.uint32).astype(np.int64)
    key = np.where(bits >> 31, 0xFFFFFFFF - bits, bits + (1 << 31))
    sel = c.sel.cpu().numpy()
    for h in range(H):
        for i in range(nqb):
            best = sorted(np.flatnonzero(seen[i]), key=lambda l: (-key[h, i, l], l))[:k]
            assert sel[h, i].tolist() == sorted(int(l) for l in best), (h, i)
