"""A step's append carried by its selection (one launch for a small chunk): what it leaves, and when it is not taken."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2604_21221_amd import pbsa  # noqa: E402
from paper_2604_21221_amd.cache import PbsaCache  # noqa: E402
from tests.test_cache_host import B, D, H, NQ, chunk, rows  # noqa: E402


@pytest.fixture
def cache():
    return PbsaCache(H, D, B, NQ, 1, 3, 12, D ** -0.5, device="cpu")


@pytest.mark.xfail(strict=True, reason="holds what was wrong: a step whose one call is refused has appended nothing, so the chunk does not count")
def test_an_append_whose_selection_fails_is_in_the_ring(cache, monkeypatch):
    def refuse(*a, append=None, **k):
        assert append is not None
        raise pbsa.PbsaError(pbsa.PBSA_EHIP)

    monkeypatch.setattr(pbsa, "pbsa_select_blocks", refuse)
    with torch.no_grad():
        cache.Kl.fill_(7.0)
        cache.Vl.fill_(7.0)
    k, v = chunk(1), chunk(2)
    with pytest.raises(pbsa.PbsaError):
        cache.step(chunk(0), k, v, 0)
    assert torch.equal(rows(cache, cache.Kl), k) and torch.equal(rows(cache, cache.Vl), v)
    tail = cache.Kl[:, :cache.nqb].reshape(H, -1, D)[:, NQ:]
    assert tail.numel() and not tail.any()
    assert cache.chunk_ids == [0] and cache.stale_from == 0


@pytest.mark.parametrize("why", ["older block stale", "deferred update", "queries followed by autograd", "values through torch"])
def test_when_an_append_is_not_carried(cache, monkeypatch, why):
    launched, carried = [], []
    monkeypatch.setattr(pbsa, "pbsa_append_chunk", lambda *a, carried=False, **k: launched.append(carried) or (a if carried else None))
    for name in ("pbsa_select_blocks", "pbsa_select_blocks_apply"):
        monkeypatch.setattr(pbsa, name, lambda *a, append=None, **k: carried.append(append is not None))
    cache.adopt_chunk(0)
    cache.stale_from = cache.n_loc
    q, v = chunk(0), chunk(2)
    if why == "older block stale":
        cache.stale_from = 1
    elif why == "deferred update":
        cache._pending = cache.params(n_evict=0)
    elif why == "queries followed by autograd":
        q.requires_grad_()
    else:
        v = v.float()
    cache._select(q, cache._append(chunk(1), v, 1, True, q))
    assert not any(launched) and carried == [False]


@pytest.mark.gpu
@pytest.mark.parametrize("d,b,nqb,tail,w", [(64, 64, 1, 1, 0), (64, 64, 4, 33, 4), (64, 64, 12, 64, 2), (64, 64, 13, 5, 1), (64, 128, 5, 127, 1),
                                            (128, 64, 12, 9, 3), (128, 64, 3, 64, 41), (128, 64, 3, 2, 42), (128, 128, 4, 65, 2),
                                            (128, 128, 5, 128, 2)])
def test_a_carried_append_leaves_what_the_two_calls_do(d, b, nqb, tail, w):
    """On either side of what one launch takes (12 blocks, 256 KiB, 128 local blocks): every bit of the ring, the pooled keys and
    queries, the block sets and the logits; inputs token-major as a model has them."""
    dev, heads, nq = "cuda:0", 3, (nqb - 1) * b + tail
    print(f"[case] carried append d={d} B={b} {nqb} blocks, last {tail}, window {w}", flush=True)
    one, two = (PbsaCache(heads, d, b, nq, w, 1, 4, np.float32(1 / math.sqrt(d)), device=dev) for _ in range(2))
    gen = torch.Generator(device=dev).manual_seed(d + nq)
    for c in (one, two):
        c.Kl.fill_(3.0)
        c.Vl.fill_(3.0)
    for g in range(w + 3):
        q, k, v = (torch.randn(nq, heads, d, generator=gen, device=dev).to(torch.bfloat16).transpose(0, 1) for _ in range(3))
        pooled = one._append(k, v, g, True, q)
        assert isinstance(pooled, tuple)
        one._select(q, pooled)
        two.append_chunk(k, v, g)
        two.select(q)
        n = heads * nqb * two.n_loc
        for name in ("Kl", "Vl"):
            assert torch.equal(getattr(one, name).view(torch.int16), getattr(two, name).view(torch.int16)), (g, name)
        for name in ("Kc_l", "Qc", "sel"):
            assert torch.equal(getattr(one, name).view(torch.int32), getattr(two, name).view(torch.int32)), (g, name)
        assert torch.equal(one.Zl[:n].view(torch.int32), two.Zl[:n].view(torch.int32)), g
        if len(two.chunk_pos) == w + 1:
            for c in (one, two):
                c.chunk_pos.pop(0)
                c.chunk_ids.pop(0)
                c.stale_from = c.n_loc


def refuse(*a, **k):
    raise pbsa.PbsaError(pbsa.PBSA_EHIP)


def test_a_refused_call_is_made_as_two(cache, monkeypatch):
    """What the one call refuses the two calls decide: a chunk counts once its append went through, whatever the selection
    behind it says, and not before."""
    launched, ok = [], []
    monkeypatch.setattr(pbsa, "pbsa_append_select", refuse)
    monkeypatch.setattr(pbsa, "pbsa_append_chunk", lambda *a, **k: launched.append(a))
    with monkeypatch.context() as m:
        m.setattr(pbsa, "pbsa_select_blocks", refuse)
        with pytest.raises(pbsa.PbsaError):
            cache.step(chunk(0), chunk(1), chunk(2), 0)
    assert len(launched) == 1 and cache.chunk_ids == [0] and cache.n_appended == 1 and cache.stale_from == 0
    with monkeypatch.context() as m:
        m.setattr(pbsa, "pbsa_append_chunk", refuse)
        with pytest.raises(pbsa.PbsaError):
            cache.step(chunk(0), chunk(1), chunk(2), 1)
    assert cache.chunk_ids == [0] and cache.n_appended == 1 and cache.stale_from == 0
    for name in ("pbsa_select_blocks", "pbsa_attention_fwd_plan_split", "pbsa_attention_fwd_plan", "pbsa_memory_update_apply"):
        monkeypatch.setattr(pbsa, name, lambda *a, name=name, **k: ok.append(name))
    cache.step(chunk(0), chunk(1), chunk(2), 1)
    assert cache.chunk_ids == [1] and cache.chunk_pos == [1] and cache.n_appended == 2 and ok[0] == "pbsa_select_blocks"


def test_an_interrupted_call_declares_nothing(cache, monkeypatch):
    def interrupt(*a, **k):
        raise KeyboardInterrupt

    monkeypatch.setattr(pbsa, "pbsa_append_select", interrupt)
    with pytest.raises(KeyboardInterrupt):
        cache.step(chunk(0), chunk(1), chunk(2), 0)
    assert (cache.chunk_pos, cache.chunk_ids, cache.n_appended, cache.stale_from) == ([], [], 0, 0)


@pytest.mark.parametrize("call", ["step", "step_fine", "step_fused", "step_chained"])
def test_a_step_that_is_refused_declares_nothing(cache, monkeypatch, call):
    refused = []

    def refuse_as(name):
        def f(*a, **k):
            refused.append(name)
            raise pbsa.PbsaError(pbsa.PBSA_EINVAL)
        return f

    for name in ("pbsa_append_chunk", "pbsa_append_select"):
        monkeypatch.setattr(pbsa, name, refuse_as(name))
    with pytest.raises(pbsa.PbsaError):
        getattr(cache, call)(chunk(0), chunk(1), chunk(2), 0)
    assert refused == ["pbsa_append_select", "pbsa_append_chunk"]
    assert (cache.chunk_pos, cache.chunk_ids, cache.n_appended, cache.stale_from) == ([], [], 0, 0)


def test_a_step_begins_with_one_call(cache, monkeypatch):
    calls = []
    for name in ("pbsa_append_select", "pbsa_attention_fwd_plan", "pbsa_attention_fwd_plan_split", "pbsa_memory_update_apply"):
        monkeypatch.setattr(pbsa, name, lambda *a, name=name, **k: calls.append((name, a)))
    for name in ("pbsa_append_chunk", "pbsa_select_blocks"):
        monkeypatch.setattr(pbsa, name, lambda *a, **k: pytest.fail("a call of its own"))
    for g in range(4):
        cache.step(chunk(0), chunk(1), chunk(2), g)
        p, at = calls[-3][1][0], calls[-3][1][3]
        assert calls[-3][0] == "pbsa_append_select" and p.pool_from == p.n_loc == min(g + 1, 2) * cache.nqb
        assert at == g % 2 * cache.nqb and cache.n_appended == g + 1
    assert len(calls) == 12


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(64, 64, 12, 64, 2, 3), (64, 64, 1, 1, 0, 128), (64, 64, 1, 1, 0, 129), (64, 128, 12, 128, 1, 21),
                                  (64, 128, 12, 128, 1, 22)])
def test_a_carried_append_on_either_side_of_a_line(case):
    """On either side of what one launch takes (12 blocks, 128 local blocks, 128 KiB and 128 workgroups, with whole blocks 256 KiB and
    64): every bit of the ring, the pooled keys and queries, the block sets and the logits; inputs token-major as a model
    has them."""
    d, b, nqb, tail, w, heads = case
    dev, nq = "cuda:0", (nqb - 1) * b + tail
    print(f"[case] carried append H={heads} d={d} B={b} {nqb} blocks, last {tail}, window {w}", flush=True)
    one, two = (PbsaCache(heads, d, b, nq, w, 1, 4, np.float32(1 / math.sqrt(d)), device=dev) for _ in range(2))
    gen = torch.Generator(device=dev).manual_seed(d + nq)
    for c in (one, two):
        c.Kl.fill_(3.0)
        c.Vl.fill_(3.0)
    for g in range(w + 3):
        q, k, v = (torch.randn(nq, heads, d, generator=gen, device=dev).to(torch.bfloat16).transpose(0, 1) for _ in range(3))
        with pytest.MonkeyPatch.context() as m:
            m.setattr(pbsa, "pbsa_append_chunk", refuse)         # it is the one call
            one._select(q, one._append(k, v, g, True, q))
        two.append_chunk(k, v, g)
        two.select(q)
        n = heads * nqb * two.n_loc
        for name in ("Kl", "Vl"):
            assert torch.equal(getattr(one, name).view(torch.int16), getattr(two, name).view(torch.int16)), (g, name)
        for name in ("Kc_l", "Qc", "sel"):
            assert torch.equal(getattr(one, name).view(torch.int32), getattr(two, name).view(torch.int32)), (g, name)
        assert torch.equal(one.Zl[:n].view(torch.int32), two.Zl[:n].view(torch.int32)), g
        if len(two.chunk_pos) == w + 1:
            for c in (one, two):
                c.chunk_pos.pop(0)
                c.chunk_ids.pop(0)
                c.stale_from = c.n_loc
