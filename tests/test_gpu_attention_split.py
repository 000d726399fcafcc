"""The attention launch whose last round of workgroups is shared out over the keys, and the same call with every query tile
walked whole, against fp64: parts with no tile of a class, ragged and empty slots, rows without keys, whole rounds ahead of
the split one.

Bound, for both: a probability p_j is rounded to bf16 (8 bits of significand), (1 + e_j) p_j with |e_j| <= 2^-8 and, over many
keys, e_j independent with root mean square at most 2^-8 / sqrt(3); the normaliser is the sum of the rounded ones.  To first
order O is then off by sum_j p_j e_j (v_j - O), of standard deviation 2^-8 / sqrt(3) sqrt(sum_j p_j^2 (v_j - O)^2), and lse by
sum_j p_j e_j.  Eight standard deviations (|e_j| <= sqrt(3) of one, so a row of one key is inside too), 2^-8 |O| for O's own
rounding, and fp32: 1e-5 of the largest |v|, 2e-5 (1 + |lse|)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def exact_rows(c, Q, h, i, lens, sel, l_map, l_len):
    """Query block i of head h in fp64: O, lse, the standard deviations of both (see above), and (key block, mass) pairs."""
    rows, u = [], []
    for slot in range(c.C + 1):
        rows.append((c.Kp[h, slot, :lens[h][slot]], c.Vp[h, slot, :lens[h][slot]]))
        u.append(slot)
    for l in sel[h][i][:c.k]:
        if l >= 0:
            rows.append((c.Kl[h, l_map[l], :l_len[l]], c.Vl[h, l_map[l], :l_len[l]]))
            u.append(c.C + 1 + l)
    K, V = (torch.cat([r[n] for r in rows]).double() for n in (0, 1))
    q = Q[h, i * c.B:(i + 1) * c.B].double()
    if K.shape[0] == 0:
        zero = torch.zeros(q.shape[0], dtype=torch.float64, device=DEV)
        return torch.zeros_like(q), zero - float("inf"), torch.zeros_like(q), zero, []
    z = torch.mm(q, K.t().contiguous()) * c.scale
    lse = torch.logsumexp(z, 1)
    P = torch.exp(z - lse[:, None])
    O = torch.mm(P, V)
    P2 = P * P
    var = torch.mm(P2, V * V) - 2 * O * torch.mm(P2, V) + O * O * P2.sum(1, keepdim=True)
    e = 2.0 ** -8 / 3 ** 0.5
    at, mass = 0, []
    for n, (k_rows, _) in zip(u, rows):
        mass.append((n, float(P[:, at:at + k_rows.shape[0]].sum())))
        at += k_rows.shape[0]
    return O, lse, e * var.clamp_min(0).sqrt(), e * P2.sum(1).sqrt(), mass


@pytest.mark.parametrize("H,d,B,Nq,w,C,k,causal,empty", [
    (2, 64, 64, 256, 3, 2, 12, 1, False),  # more parts than most classes have tiles
    (1, 128, 128, 300, 0, 30, 1, 1, False),  # nearly everything persistent
    (3, 128, 64, 1000, 2, 5, 17, 1, False),  # two query blocks per workgroup: solo tiles
    (3, 64, 64, 999, 1, 0, 20, 0, False),  # no slots but the (empty) summary
    (5, 64, 128, 1000, 3, 5, 7, 0, False),
    (2, 64, 64, 640, 1, 40, 0, 1, True),   # nothing selected, and a head whose slots are empty: rows without keys
    (3, 128, 128, 300, 1, 40, 0, 1, True),
    (40, 64, 64, 1664, 1, 3, 9, 1, False),   # 520 query tiles: 512 whole, 8 split
])
def test_split_and_whole_match_fp64(H, d, B, Nq, w, C, k, causal, empty):
    from paper_2604_21221_amd import pbsa
    from paper_2604_21221_amd.cache import PbsaCache
    from tests.test_gpu_parity_fine_mass import MASS_ATOL, MASS_RTOL
    gen = torch.Generator(device=DEV).manual_seed(H + d + Nq)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16)
    c = PbsaCache(H, d, B, Nq, w, C, k, d ** -0.5, causal=causal, device=DEV)
    print(f"[case] split H={H} d={d} B={B} Nq={Nq} C={C} k={k}", flush=True)
    for g in range(w + 1):
        c.append_chunk(2.0 * rnd(H, Nq, d), rnd(H, Nq, d), g)
    if C:
        lens = torch.randint(0, B + 1, (H, C), generator=gen, device=DEV, dtype=torch.int32)
        if empty:
            lens[0] = 0
        c.set_persistent(2.0 * rnd(H, C, B, d), rnd(H, C, B, d), lens, torch.arange(C)[None].repeat(H, 1))
    Q = rnd(H, Nq, d)
    c.select(Q)
    assert c._attn_bytes > 0 and c._split_pays(), "this shape is meant to be split"
    l_map, l_len, _ = c._device_maps()
    lse, lse_w, lse_m, lse_mw = (torch.empty(H, Nq, device=DEV) for _ in range(4))
    O = c.attention(Q, lse=lse)
    O_w = torch.empty_like(Q)
    args = Q, c.Kp, c.Vp, c.p_len, c.Kl, c.Vl, l_len, l_map, c.sel
    pbsa.pbsa_attention_fwd(c.params(Q=Q, O=O_w), *args, O_w, lse_w)
    assert not torch.equal(O, O_w) or empty, "not split after all"
    # the variant that records the mass takes the same parts, or none
    O_m, Mt = c.attention_with_mass(Q, lse=lse_m)
    O_mw, Mt_w = torch.empty_like(Q), torch.empty_like(Mt)
    p = c.params(Q=Q, O=O_mw)
    pbsa.pbsa_attention_fwd_mass(p, *args, O_mw, lse_mw, Mt_w, (c._mass_ws.data_ptr(), pbsa.pbsa_mass_workspace_bytes(p)))
    for a, b in ((O, O_m), (O_w, O_mw)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert torch.equal(lse, lse_m) and torch.equal(lse_w, lse_mw)
    # and so does the one that takes the update's decisions
    lse_p = torch.empty_like(lse)
    O_p = c.attention_with_plan(Q, lse=lse_p)
    assert torch.equal(O_p.view(torch.int16), O.view(torch.int16)) and torch.equal(lse_p, lse)
    host = c.p_len.tolist(), c.sel.tolist(), l_map.tolist(), l_len.tolist()
    v_max = max(float(c.Vl.abs().max()), float(c.Vp.abs().max()))
    no_key, worst = 0, {}
    for h in sorted({0, 1, H // 2, H - 2, H - 1} & set(range(H))):
        for i in range(c.nqb):
            want, want_lse, sd, sd_lse, mass = exact_rows(c, Q, h, i, *host)
            at = slice(i * B, min((i + 1) * B, Nq))
            for name, o, l, M in (("split", O, lse, Mt), ("whole", O_w, lse_w, Mt_w)):
                if not mass:
                    assert not o[h, at].any() and bool((l[h, at] == float("-inf")).all())
                    no_key += 1
                    continue
                off = (o[h, at].double() - want).abs() / (8 * sd + 2.0 ** -8 * want.abs() + 1e-5 * v_max)
                off_lse = (l[h, at].double() - want_lse).abs() / (8 * sd_lse + 2e-5 * (1 + want_lse.abs()))
                worst[name] = max(worst.get(name, 0.0), float(off.max()), float(off_lse.max()))
                got = M[h, :, i].tolist()
                for u, m in mass:
                    assert abs(got[u] - m) <= MASS_RTOL * m + MASS_ATOL, (name, h, i, u)
    print(f"[case] worst error over its bound: {worst}", flush=True)
    assert all(v <= 1.0 for v in worst.values())
    assert (no_key > 0) == empty


def _cache_and_chunks(n, H=5, d=64, B=128, Nq=1000, w=1, C=5, k=7):
    """A cache of a shape that is split, and n chunks."""
    from paper_2604_21221_amd.cache import PbsaCache
    gen = torch.Generator(device=DEV).manual_seed(n + H)
    c = PbsaCache(H, d, B, Nq, w, C, k, d ** -0.5, device=DEV)
    assert c._attn_bytes > 0, "this shape is meant to be split"
    return c, [[torch.randn(H, Nq, d, generator=gen, device=DEV).to(torch.bfloat16) for _ in range(3)] for _ in range(n)]


def test_plain_attention_leaves_its_workspace_alone():
    """pbsa_attention_fwd takes a workspace and does not look at it: callers hand the same one to every call, with a plan
    still to be applied in it."""
    from paper_2604_21221_amd import pbsa
    c, [(Q, K, V)] = _cache_and_chunks(1)
    c.append_chunk(K, V, 0)
    c.select(Q)
    l_map, l_len, _ = c._device_maps()
    print("[case] plain attention with a workspace", flush=True)
    out = []
    for ws in (None, torch.full((c._attn_bytes + 256,), 0x5A, dtype=torch.uint8, device=DEV)):
        O = torch.empty_like(Q)
        pbsa.pbsa_attention_fwd(c.params(Q=Q, O=O), Q, c.Kp, c.Vp, c.p_len, c.Kl, c.Vl, l_len, l_map, c.sel, O, None, ws)
        out.append(O)
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
    assert bool((ws == 0x5A).all())


def test_plain_attention_between_plan_and_apply_on_one_workspace():
    """pbsa_memory_update_plan, pbsa_attention_fwd, pbsa_memory_update_apply, all with one workspace: the state of
    pbsa_memory_update, bit for bit."""
    from paper_2604_21221_amd import pbsa
    a, chunks = _cache_and_chunks(4)
    b, _ = _cache_and_chunks(4)
    for g, (Q, K, V) in enumerate(chunks):
        print(f"[case] one workspace, chunk {g}", flush=True)
        for c in (a, b):
            c.append_chunk(K, V, g)
            c.select(Q)
        a.update()
        b.update_plan()
        l_map, l_len, _ = b._device_maps()
        O = torch.empty_like(Q)
        pbsa.pbsa_attention_fwd(b.params(Q=Q, O=O), Q, b.Kp, b.Vp, b.p_len, b.Kl, b.Vl, l_len, l_map, b.sel, O, None, b.ws)
        b.update_apply()
        for name in ("Kp", "Vp", "Kc_p", "p_len", "p_id", "S_sum", "S_cnt", "slot_src"):
            assert torch.equal(getattr(a, name), getattr(b, name)), (name, g)


def test_room_in_a_workspace_changes_nothing():
    """pbsa_attention_fwd_plan and pbsa_attention_fwd_mass give pbsa_attention_fwd's output bit for bit however large their
    workspace is, and use no more of it than they say."""
    from paper_2604_21221_amd import pbsa
    c, [(Q, K, V)] = _cache_and_chunks(1)
    c.append_chunk(K, V, 0)
    c.select(Q)
    l_map, l_len, l_id = c._device_maps(want_ids=True)
    p = c.params(Q=Q, O=Q)
    need = pbsa.pbsa_workspace_bytes(p), pbsa.pbsa_mass_workspace_bytes(p)
    args = Q, c.Kp, c.Vp, c.p_len, c.Kl, c.Vl, l_len, l_map, c.sel
    O = torch.empty_like(Q)
    lse = torch.empty(c.H, c.Nq, device=DEV)
    pbsa.pbsa_attention_fwd(p, *args, O, lse)
    print("[case] large workspaces", flush=True)
    for n, call in zip(need, (
            lambda O, lse, ws: pbsa.pbsa_attention_fwd_plan(p, *args, O, lse, c.Qc, c.Kc_l, c.Zl, c.Kc_p, c.p_id, c.S_cnt, l_id,
                                                            c.scores, c.slot_src, ws),
            lambda O, lse, ws: pbsa.pbsa_attention_fwd_mass(p, *args, O, lse, c._mass_buffer(), ws))):
        ws = torch.full((n + 2 * c._attn_bytes,), 0x5A, dtype=torch.uint8, device=DEV)
        O2, lse2 = torch.empty_like(O), torch.empty_like(lse)
        call(O2, lse2, ws)
        assert torch.equal(O.view(torch.int16), O2.view(torch.int16)) and torch.equal(lse, lse2)
        assert bool((ws[n:] == 0x5A).all())


def test_attention_from_two_streams():
    """Attention calls on one cache from two streams, each with its own Q and O, in a shape that is split: each gives what
    it gives alone."""
    c, chunks = _cache_and_chunks(2, Nq=2000, C=30, k=16)
    for g, (_, K, V) in enumerate(chunks):
        c.append_chunk(K, V, g)
    Qs = [chunks[0][0], chunks[1][0]]
    c.select(Qs[0])
    assert c._split_pays()
    want = [c.attention(Q) for Q in Qs]
    O = [torch.empty_like(Q) for Q in Qs]
    streams = [torch.cuda.Stream() for _ in Qs]
    torch.cuda.synchronize()
    print("[case] attention from two streams", flush=True)
    for r in range(20):
        for Q, o, s in zip(Qs, O, streams):
            with torch.cuda.stream(s):
                for _ in range(3):
                    c.attention(Q, o)
        torch.cuda.synchronize()
        assert all(torch.equal(o, w) for o, w in zip(O, want)), r


def test_split_attention_in_a_graph():
    """Captured, with its scratch from the graph's own memory: every replay gives what the eager call gives, with eager calls
    on the same cache in between and two graphs of one capture stream."""
    c, chunks = _cache_and_chunks(2, C=30, k=16)
    for g, (_, K, V) in enumerate(chunks):
        c.append_chunk(K, V, g)
    Q, other = chunks[0][0].clone(), chunks[1][0]
    O = [torch.empty_like(Q) for _ in range(2)]
    c.select(Q)
    assert c._split_pays()
    c.attention(Q, O[0])
    torch.cuda.synchronize()
    print("[case] split attention in a graph", flush=True)
    graphs = [torch.cuda.CUDAGraph() for _ in O]
    for g, o in zip(graphs, O):
        with torch.cuda.graph(g):
            c.attention(Q, o)
    for r in range(4):
        Q.copy_(chunks[r % 2][r % 3])
        for g in graphs:
            g.replay()
        eager = c.attention(other)
        torch.cuda.synchronize()
        want = c.attention(Q)
        assert torch.equal(O[0], want) and torch.equal(O[1], want) and torch.equal(eager, c.attention(other)), r
