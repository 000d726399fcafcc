"""The attention launch whose last round of workgroups is shared out over the keys, against the same call without scratch
(every query tile walked whole): parts with no tile of a class, ragged and empty slots, rows without keys, whole rounds
ahead of the split one.

Bound: both sides round every probability to bf16 (2^-9 relative, in numerator and normaliser alike) relative to
references that differ, so an output differs by at most 2 (2^-9 + 2^-9) max|V| before it is rounded to bf16 itself
(2^-9 |O| <= 2^-9 max|V| on either side): 3 * 2^-8 max|V|; lse by twice -log(1 - 2^-9)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("H,d,B,Nq,w,C,k,causal", [
    (2, 64, 64, 256, 3, 2, 12, 1),         # more parts than most classes have tiles
    (1, 128, 128, 300, 0, 30, 1, 1),       # nearly everything persistent
    (3, 128, 64, 1000, 2, 5, 17, 1),       # two query blocks per workgroup: solo tiles
    (3, 64, 64, 999, 1, 0, 20, 0),         # no slots but the (empty) summary
    (5, 64, 128, 1000, 3, 5, 7, 0),
    (1, 64, 64, 640, 1, 40, 0, 1),         # nothing selected
    (40, 64, 64, 1664, 1, 3, 9, 1),        # 520 query tiles: 512 whole, 8 split
])
def test_split_matches_whole(H, d, B, Nq, w, C, k, causal):
    from paper_2604_21221_amd import pbsa
    from paper_2604_21221_amd.cache import PbsaCache
    gen = torch.Generator(device=DEV).manual_seed(H + d + Nq)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16)
    c = PbsaCache(H, d, B, Nq, w, C, k, d ** -0.5, causal=causal, device=DEV)
    print(f"[case] split H={H} d={d} B={B} Nq={Nq} C={C} k={k}", flush=True)
    for g in range(w + 1):
        c.append_chunk(2.0 * rnd(H, Nq, d), rnd(H, Nq, d), g)
    if C:
        lens = torch.randint(0, B + 1, (H, C), generator=gen, device=DEV, dtype=torch.int32)
        c.set_persistent(2.0 * rnd(H, C, B, d), rnd(H, C, B, d), lens, torch.arange(C)[None].repeat(H, 1))
    Q = rnd(H, Nq, d)
    c.select(Q)
    assert c._attn_bytes > 0 and c._split_pays(), "this shape is meant to be split"
    lse, lse_w = (torch.empty(H, Nq, device=DEV) for _ in range(2))
    O = c.attention(Q, lse=lse)
    l_map, l_len, _ = c._device_maps()
    O_w = torch.empty_like(Q)
    pbsa.pbsa_attention_fwd(c.params(Q=Q, O=O_w), Q, c.Kp, c.Vp, c.p_len, c.Kl, c.Vl, l_len, l_map, c.sel, O_w, lse_w)
    fin = torch.isfinite(lse_w)
    assert torch.equal(torch.isfinite(lse), fin) and torch.equal(lse[~fin], lse_w[~fin])
    assert float((lse - lse_w)[fin].abs().max() if fin.any() else 0.0) <= 2 * 1.96e-3
    v_max = max(float(c.Vl.abs().max()), float(c.Vp.abs().max()))
    assert float((O.float() - O_w.float()).abs().max()) <= 3 * 2.0 ** -8 * v_max
    # the variant that records the mass takes the same parts
    O_m, _ = c.attention_with_mass(Q)
    assert torch.equal(O_m.view(torch.int16), O.view(torch.int16))


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
