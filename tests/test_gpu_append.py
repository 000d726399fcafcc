"""pbsa_append_chunk against torch copies and pbsa_pool_blocks: every byte of the rings and every bit of the pooled keys
(the same pinned additions), at the edges of a block (one token, one short of full, full) and for strided sources."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,B,Nq", [(64, 64, 1), (64, 64, 256), (64, 128, 127), (128, 64, 129), (128, 128, 1000), (128, 64, 4680)])
@pytest.mark.parametrize("strided", [False, True], ids=["dense", "strided"])
def test_append_matches_copies_and_pooling(d, B, Nq, strided):
    from paper_2604_21221_amd import pbsa
    from paper_2604_21221_amd.cache import PbsaCache
    H, w = 3, 1
    gen = torch.Generator(device=DEV).manual_seed(Nq + d + B)
    def draw():
        if strided:                       # [Nq][H][3 d], one third of it, heads in the middle
            return torch.randn(Nq, H, 3 * d, generator=gen, device=DEV).to(torch.bfloat16)[:, :, d:2 * d].permute(1, 0, 2)
        return torch.randn(H, Nq, d, generator=gen, device=DEV).to(torch.bfloat16)
    c = PbsaCache(H, d, B, Nq, w, 2, 1, d ** -0.5, device=DEV)
    c.Kl.fill_(7.0), c.Vl.fill_(7.0), c.Kc_l.fill_(7.0)
    print(f"[case] append d={d} B={B} Nq={Nq} strided={strided}", flush=True)
    want_K, want_V = c.Kl.clone(), c.Vl.clone()
    def put(dst, pos, x, tail):
        rows = dst[:, pos * c.nqb:(pos + 1) * c.nqb].view(H, c.nqb * B, d)
        rows[:, :Nq] = x
        if tail:
            rows[:, Nq:] = 0
    def same(a, b):
        return torch.equal(a.view(torch.int16), b.view(torch.int16))
    def pooled(pos):
        lens = c._chunk_lens.repeat(H).to(DEV)
        X = want_K[:, pos * c.nqb:(pos + 1) * c.nqb].contiguous()
        out = torch.empty(H * c.nqb, d, device=DEV)
        pbsa.pbsa_pool_blocks(c.params(), X, lens, H * c.nqb, out)
        return out.view(H, c.nqb, d)
    for g in range(2):
        K, V = draw(), draw()
        c.append_chunk(K, V, g)
        put(want_K, g, K, True), put(want_V, g, V, True)
        assert same(c.Kl, want_K) and same(c.Vl, want_V)
        assert torch.all(c.Kc_l[:, g * c.nqb:] == 7.0), "pooled before the selection has seen the rows"
        pbsa.pbsa_append_chunk(c._full, K, V, g * c.nqb, True, c.Kl, c.Vl, c.Kc_l)
        assert same(c.Kl, want_K) and same(c.Vl, want_V)
        assert torch.equal(c.Kc_l[:, g * c.nqb:(g + 1) * c.nqb], pooled(g)), "pooled keys"
        if g == 0:
            assert torch.all(c.Kc_l[:, c.nqb:] == 7.0), "another chunk's pooled keys were touched"
    tail_K = c.Kl[:, -1, Nq - (c.nqb - 1) * B:].clone()
    K = draw()
    c.rewrite_chunk(K)                     # K alone, the rows past the chunk's end stay
    put(want_K, 1, K, False)
    assert same(c.Kl, want_K) and same(c.Vl, want_V) and same(c.Kl[:, -1, Nq - (c.nqb - 1) * B:], tail_K)
    Q = draw()
    c.select(Q)                            # the keys pooled on the way in and the selection's own pooling agree
    kept = c.Kc_l.clone(), c.sel.clone(), c.Qc.clone()
    c.stale_from = 0
    c.select(Q)
    assert all(torch.equal(a, b) for a, b in zip(kept, (c.Kc_l, c.sel, c.Qc)))


def test_selection_pools_the_rows_it_finds():
    """Rows of the newest chunk that are changed in the ring between the append and the first selection count as changed."""
    from paper_2604_21221_amd.cache import PbsaCache
    H, d, B, Nq = 2, 64, 64, 200
    gen = torch.Generator(device=DEV).manual_seed(3)
    rnd = lambda: torch.randn(H, Nq, d, generator=gen, device=DEV).to(torch.bfloat16)
    Q, K, V, K2 = rnd(), rnd(), rnd(), rnd()
    print("[case] rows changed before the first selection", flush=True)
    got = []
    for first in (K, K2):
        c = PbsaCache(H, d, B, Nq, 1, 2, 2, d ** -0.5, device=DEV)
        c.append_chunk(first, V, 0)
        c.Kl[:, :c.nqb].view(H, c.nqb * B, d)[:, :Nq] = K2
        c.select(Q)
        got.append((c.Kc_l, c.sel))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def test_an_append_while_another_device_is_current(monkeypatch):
    """The library launches on the current device's stream; a copy runs where its tensors are."""
    from paper_2604_21221_amd import pbsa
    from paper_2604_21221_amd.cache import PbsaCache
    c = PbsaCache(2, 64, 64, 200, 1, 2, 2, 0.125, device=DEV)
    K, V = (torch.randn(2, 200, 64, device=DEV).to(torch.bfloat16) for _ in range(2))
    calls = []
    with monkeypatch.context() as m:
        m.setattr(pbsa, "pbsa_append_chunk", lambda *a, **k: calls.append(a))
        m.setattr(torch._C, "_cuda_getDevice", lambda: 1)
        c.append_chunk(K, V, 0)
    rows = [t[:, :c.nqb].view(2, c.nqb * 64, 64)[:, :200] for t in (c.Kl, c.Vl)]
    assert not calls and torch.equal(rows[0], K) and torch.equal(rows[1], V)


def test_chunks_that_go_through_torch():
    """Tensors that the launch does not take as they are (fp32, rows at an odd address, spread over the heads) end as the same
    rows, pooled keys, selection and output as their dense bf16 copies; so does V rewritten alone."""
    from paper_2604_21221_amd.cache import PbsaCache
    H, d, B, Nq = 3, 128, 64, 333
    gen = torch.Generator(device=DEV).manual_seed(17)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16)
    odd = rnd(H * Nq * d + 1)[1:].view(H, Nq, d)
    forms = {"fp32": rnd(H, Nq, d).float(), "odd address": odd, "one head for all": rnd(1, Nq, d)}
    assert odd.data_ptr() % 16 == 2
    for name, x in forms.items():
        print(f"[case] append through torch: {name}", flush=True)
        dense = x.to(torch.bfloat16).expand(H, Nq, d).clone()
        V, V2, Q = rnd(H, Nq, d), rnd(H, Nq, d), rnd(H, Nq, d)
        got = []
        for K in (x, dense):
            c = PbsaCache(H, d, B, Nq, 1, 2, 3, d ** -0.5, device=DEV)
            O = c.step(Q, K, V, 0)
            c.append_chunk(V, K, 1)
            c.select(Q)
            first = c.Kc_l.clone()
            c.rewrite_chunk(V=V2)
            c.select(Q)
            assert torch.equal(first, c.Kc_l), "V alone changed the pooled keys"
            got.append((O, c.Kl, c.Vl, c.Kc_l, c.sel, c.attention(Q)))
        assert all(torch.equal(a, b) for a, b in zip(*got))
        rows = got[0][2][:, c.nqb:].view(H, c.nqb * B, d)
        assert torch.equal(rows[:, :Nq], V2) and not rows[:, Nq:].any()
