"""The attention by teams of waves: lists with fewer tiles than a team has waves, with one more, up to the longest that the limits
allow; units of one row; tiles of 1, 32, 33 and 63 keys; teams of four and of two, several teams to a unit.  Against fp64 with the
bound derived in test_gpu_attention_split.py."""
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_attention_split import exact_rows  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def filled(H, d, B, Nq, w, C, k, lens=None, seed=0):
    from paper_2604_21221_amd.cache import PbsaCache
    gen = torch.Generator(device=DEV).manual_seed(seed + H + d + Nq)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16)
    c = PbsaCache(H, d, B, Nq, w, C, k, d ** -0.5, fold=False, device=DEV)
    for g in range(w + 1):
        c.append_chunk(2.0 * rnd(H, Nq, d), rnd(H, Nq, d), g)
    if C:
        n = torch.tensor(lens or [B], dtype=torch.int32, device=DEV).repeat(C)[:C].expand(H, C).contiguous()
        c.set_persistent(2.0 * rnd(H, C, B, d), rnd(H, C, B, d), n, torch.arange(C)[None].repeat(H, 1))
    Q = rnd(H, Nq, d)
    c.select(Q)
    return c, Q


def off_by(c, Q, O, lse, heads, blocks):
    """The largest error of O and lse over its bound."""
    l_map, l_len, _ = c._device_maps()
    host = c.p_len.tolist(), c.sel.tolist(), l_map.tolist(), l_len.tolist()
    v_max = max(float(c.Vl.abs().max()), float(c.Vp.abs().max()))
    worst = 0.0
    for h in heads:
        for i in blocks:
            want, want_lse, sd, sd_lse, _ = exact_rows(c, Q, h, i, *host)
            at = slice(i * c.B, min((i + 1) * c.B, c.Nq))
            off = (O[h, at].double() - want).abs() / (8 * sd + 2.0 ** -8 * want.abs() + 1e-5 * v_max)
            off_lse = (lse[h, at].double() - want_lse).abs() / (8 * sd_lse + 2e-5 * (1 + want_lse.abs()))
            worst = max(worst, float(off.max()), float(off_lse.max()))
    return worst


@pytest.mark.parametrize("H,d,B,Nq,w,C,k,lens", [
    (2, 64, 64, 65, 0, 1, 2, [1]),           # two or three tiles for four waves; a unit and a block of one row
    (2, 128, 64, 65, 1, 2, 3, [33, 63]),
    (3, 64, 128, 321, 1, 2, 3, [32, 96]),    # blocks of two tiles, one of them short or missing
    (1, 128, 128, 130, 1, 3, 3, [97, 64, 0]),
    (2, 64, 64, 256, 3, 2, 4, None),         # seven tiles
    (4, 128, 64, 256, 1, 3, 5, [31, 64]),    # nine
    (16, 64, 64, 1090, 1, 4, 6, [64, 5]),    # 288 units: teams of two
    (10, 128, 128, 3201, 1, 1, 2, [127]),    # 510 units, the last of one row
    (1, 64, 64, 1000, 1, 64, 16, [64, 40]),  # several teams to a unit
    (1, 128, 128, 1990, 2, 16, 16, [128, 65]),
    (1, 64, 64, 10752, 3, 336, 672, [64, 63]),   # the longest list of blocks of 64, all of 672 blocks and 336 slots
    (1, 128, 128, 2688, 31, 336, 672, None),     # and of 128
])
def test_team_matches_fp64(H, d, B, Nq, w, C, k, lens):
    from paper_2604_21221_amd import pbsa
    print(f"[case] team H={H} d={d} B={B} Nq={Nq} C={C} k={k}", flush=True)
    c, Q = filled(H, d, B, Nq, w, C, k, lens)
    lse = torch.empty(H, Nq, device=DEV)
    O = c.attention(Q, lse=lse)
    blocks = sorted({0, 1, c.nqb // 2, c.nqb - 1} & set(range(c.nqb)))
    worst = off_by(c, Q, O, lse, sorted({0, H - 1}), blocks)
    print(f"[case] worst error over its bound: {worst}", flush=True)
    assert worst <= 1.0
    if C <= pbsa.PBSA_MAX_C_AUX:             # the variants that record the mass or take decisions: the same bits
        lse2 = torch.empty_like(lse)
        O2, Mt = c.attention_with_mass(Q, lse=lse2)
        assert torch.equal(O2.view(torch.int16), O.view(torch.int16)) and torch.equal(lse2, lse)
        from tests.test_gpu_parity_fine_mass import MASS_ATOL, MASS_RTOL
        ref = c.attention_mass(Q, lse, torch.zeros_like(Mt))[:, :, :c.nqb]
        # the pass that repeats the first product: sums of unrounded probabilities, so within a probability's 2^-8 of each other
        assert bool(((Mt[:, :, :c.nqb] - ref).abs() <= (MASS_RTOL + 2.0 ** -8) * ref + MASS_ATOL).all())
        if C <= pbsa.PBSA_MAX_C:
            O3 = c.attention_with_plan(Q, lse=lse2)
            assert torch.equal(O3.view(torch.int16), O.view(torch.int16)) and torch.equal(lse2, lse)


@pytest.mark.parametrize("d,B", [(64, 64), (128, 128)])
def test_what_lies_beyond_a_blocks_length(d, B):
    """Infinities and NaN in rows beyond a block's valid length change nothing."""
    print(f"[case] team, rows beyond the length d={d} B={B}", flush=True)
    c, Q = filled(2, d, B, 2 * B + 9, 1, 3, 5, [B, 5, 40])
    want = c.attention(Q)
    for t, x in ((c.Kp, float("nan")), (c.Vp, float("inf"))):
        t[:, 1, 5:], t[:, 2, 40:] = x, -x
    for t, x in ((c.Kl, float("inf")), (c.Vl, float("nan"))):
        t.view(2, 2, c.nqb, B, d)[:, :, -1, 9:] = x
    assert torch.equal(c.attention(Q).view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("d", [64, 128])
def test_infinities_and_nan_reach_their_rows(d):
    """Keys and values that are infinite or NaN: the outputs that are not finite are those of the rows that attend them, and
    the others are what they are without."""
    print(f"[case] team, infinities d={d}", flush=True)
    c, Q = filled(2, d, 64, 320, 1, 2, 3, [64])
    clean = c.attention(Q)
    sel = c.sel.tolist()
    l_map = c._device_maps()[0].tolist()
    c.Vl[0, l_map[2], 7, 3], c.Kl[1, l_map[4], 11, 5] = float("inf"), float("nan")
    O = c.attention(Q)
    for h, block, cols in ((0, 2, [3]), (1, 4, list(range(d)))):
        for i in range(c.nqb):
            at = slice(64 * i, min(64 * i + 64, 320))
            if block not in sel[h][i]:
                assert torch.equal(O[h, at], clean[h, at])
                continue
            bad = ~torch.isfinite(O[h, at].float())
            assert bool(bad[:, cols].all()) and int(bad.sum()) == bad[:, cols].numel()


def test_a_block_named_twice_counts_once():
    print("[case] team, duplicates in a selection", flush=True)
    c, Q = filled(2, 64, 64, 200, 1, 2, 4, [64])
    want = c.attention(Q)
    c.sel[:, :, 3] = c.sel[:, :, 0]
    c.sel[:, :, 0] = -1
    once = c.attention(Q)
    c.sel[:, :, 0] = c.sel[:, :, 3]
    assert torch.equal(c.attention(Q), once) and not torch.equal(once, want)


LONGEST = [                                  # 672 local blocks, one to a chunk, and 336 slots
    (300, 64, 64, 64, 671, 336, 672, [64, 63]),   # teams of two, 505 tiles of 1009 to a wave
    (257, 64, 128, 64, 671, 336, 672, [128, 65]),     # 1009 of 2018, all that a wave's list holds
    (260, 128, 128, 1, 671, 336, 672, None),
    (200, 64, 128, 40, 671, 336, 672, [128, 1]),  # teams of four, 505 of 2018
    (100, 128, 128, 64, 671, 336, 672, None),     # two teams to a unit, 253 each
    (10, 64, 128, 128, 671, 336, 672, [97]),      # twelve, 43
    (4, 64, 64, 300, 133, 336, 672, [64, 40]),    # twelve, five units a head, the last of 44 rows
    (1, 64, 64, 64, 671, 336, 672, None),         # sixteen, 16
    (270, 64, 128, 64, 511, 192, 512, [128, 70]),     # recording the mass: the longest that the later pass takes, 705 to a wave
]


@pytest.mark.parametrize("H,d,B,Nq,w,C,k,lens", LONGEST)
def test_team_with_the_longest_lists(H, d, B, Nq, w, C, k, lens):
    test_team_matches_fp64(H, d, B, Nq, w, C, k, lens)


def kernels(call):
    """Names of the library's kernels that the call launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in p.events() if "pbsa::" in e.name]
    if not names:
        pytest.skip("the profiler sees no kernels here")
    return names


@pytest.mark.parametrize("H,d,B,Nq,w,C,k,waves,parts", [
    (2, 64, 64, 65, 0, 1, 2, 4, 1), (3, 64, 128, 321, 1, 2, 3, 4, 1), (4, 128, 64, 256, 1, 3, 5, 4, 1),
    (16, 64, 64, 1090, 1, 4, 6, 2, 1), (10, 128, 128, 3201, 1, 1, 2, 2, 1),
    (1, 64, 64, 1000, 1, 64, 16, 4, 11), (1, 128, 128, 1990, 2, 16, 16, 4, 6),
    (1, 64, 64, 10752, 3, 336, 672, 0, 6),   # by query tiles of 128 rows, in parts
    (1, 128, 128, 2688, 31, 336, 672, 4, 6),
    (1, 64, 64, 64, 0, 1, 0, 0, 1),          # two tiles
    (9, 64, 64, 3700, 0, 2, 3, 0, 1),        # 522 units
    (28, 64, 128, 539, 0, 2, 2, 0, 1),       # 252 units and 28 workgroups that take decisions, short lists
    (25, 64, 128, 539, 0, 2, 2, 4, 1),       # 225 and 25
    (28, 64, 128, 539, 0, 30, 2, 4, 1),      # long lists
    (19, 64, 128, 781, 1, 2, 1, 0, 1),       # 7 x 16 pairs of a query block and a column
    (15, 64, 128, 1075, 3, 2, 2, 4, 1),      # 9 x 38
    (36, 128, 128, 846, 1, 3, 1, 0, 1),      # 504 units
    (458, 128, 128, 5, 0, 1, 1, 2, 1),       # where query tiles would find no places either
    *[(*c[:7], waves, parts) for c, waves, parts in zip(LONGEST, (2, 2, 2, 4, 4, 4, 4, 4, 2), (1, 1, 1, 1, 2, 12, 12, 16, 1))],
])
def test_which_kernel_runs(H, d, B, Nq, w, C, k, waves, parts):
    """What the cases of this file are for is what they reach: teams of so many waves, several to a unit or not, or none."""
    from paper_2604_21221_amd.cache import PbsaCache
    print(f"[case] route H={H} d={d} B={B} Nq={Nq} C={C} k={k}", flush=True)
    c = PbsaCache(H, d, B, Nq, w, C, k, d ** -0.5, fold=False, device=DEV)
    for g in range(w + 1):
        c.adopt_chunk(g)
    c._installed = C                         # as by set_persistent(): empty slots all the same
    Q = torch.zeros(H, Nq, d, dtype=torch.bfloat16, device=DEV)
    names = kernels(lambda: c.attention(Q))
    want = f"attention_team_kernel<{d}, {waves}, false, false>" if waves else f"attention_kernel<{d}, {B}, false, false, {str(parts > 1).lower()}>"
    assert want in names[0] and len(names) == 1 + (parts > 1), names
    assert parts == 1 or "combine_kernel" in names[1]


@pytest.mark.parametrize("H,d,B,Nq,w,C,k,lens", [(28, 64, 128, 539, 0, 2, 2, [128, 65]), (36, 128, 128, 846, 1, 3, 1, [127, 64, 0])])
def test_where_decisions_keep_teams_away(H, d, B, Nq, w, C, k, lens):
    test_team_matches_fp64(H, d, B, Nq, w, C, k, lens)
