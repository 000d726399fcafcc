"""Host side of PbsaCache without a GPU: a cache of CPU tensors whose library calls are replaced by recorders."""
import pytest

torch = pytest.importorskip("torch")

from paper_2604_21221_amd import pbsa  # noqa: E402
from paper_2604_21221_amd.cache import PbsaCache  # noqa: E402

H, D, B, NQ, W = 2, 64, 64, 200, 1


@pytest.fixture
def cache():
    return PbsaCache(H, D, B, NQ, W, 3, 12, D ** -0.5, device="cpu")


def chunk(seed=0):
    gen = torch.Generator().manual_seed(seed)
    return torch.randn(H, NQ, D, generator=gen).to(torch.bfloat16)


def overlap(a, b):
    return a.untyped_storage().data_ptr() == b.untyped_storage().data_ptr()


def test_attention_shares_no_scratch(cache, monkeypatch):
    """Two attention calls (of two streams, say) may be in flight at a time: what each is given to write is its own, and
    nothing that the cache keeps."""
    calls = []
    monkeypatch.setattr(pbsa, "pbsa_attention_fwd_split", lambda *a, **k: calls.append(a))
    cache.adopt_chunk(0)
    for _ in range(2):
        cache.attention(chunk())
    ws = [a[12] for a in calls]
    assert all(w.numel() == cache._attn_bytes > 0 for w in ws)
    assert not overlap(*ws) and not overlap(calls[0][10], calls[1][10])
    for name, t in vars(cache).items():
        if isinstance(t, torch.Tensor):
            assert not any(overlap(w, t) for w in ws), name


CALLS = ("pbsa_append_chunk", "pbsa_select_blocks", "pbsa_attention_fwd_split", "pbsa_attention_fwd_plan",
         "pbsa_attention_fwd_mass", "pbsa_memory_update", "pbsa_memory_update_apply", "pbsa_memory_update_fine")


def record(monkeypatch):
    calls = []
    for name in CALLS:
        monkeypatch.setattr(pbsa, name, lambda *a, name=name, **k: calls.append((name, a)))
    return calls


def books(c):
    return list(c.chunk_pos), list(c.chunk_ids), c.n_appended, c.stale_from


@pytest.mark.parametrize("call", ["append_chunk", "step", "step_fine", "step_fused", "step_chained"])
@pytest.mark.parametrize("missing", ["K", "V", "KV"])
def test_append_refuses_a_missing_tensor(cache, monkeypatch, call, missing):
    """None for K or V is no chunk: refused, with nothing launched and nothing declared.  (step_fused and step_chained take
    K = V = None for a chunk that has been adopted.)"""
    if call in ("step_fused", "step_chained") and "K" in missing:
        return
    calls = record(monkeypatch)
    kv = [None if n in missing else chunk() for n in "KV"]
    before = books(cache)
    with pytest.raises(TypeError):
        getattr(cache, call)(*([] if call == "append_chunk" else [chunk()]), *kv, 0)
    assert not calls and books(cache) == before


def test_step_is_append_select_attention_update(cache, monkeypatch):
    calls = record(monkeypatch)
    cache.step(chunk(0), chunk(1), chunk(2), 0)
    assert [n for n, _ in calls] == ["pbsa_append_chunk", "pbsa_select_blocks", "pbsa_attention_fwd_plan", "pbsa_memory_update_apply"]
    cache.Zl = None                          # without the logits the decisions are taken behind the attention
    del calls[:]
    cache.step(chunk(0), chunk(1), chunk(2), 1)
    assert [n for n, _ in calls] == ["pbsa_append_chunk", "pbsa_select_blocks", "pbsa_attention_fwd_split", "pbsa_memory_update"]


@pytest.mark.parametrize("call", ["append_chunk", "step", "step_fine", "step_fused", "step_chained"])
@pytest.mark.parametrize("why", ["K", "V", "library"])
def test_a_failed_append_declares_nothing(cache, monkeypatch, call, why):
    """K or V of a shape that fits nowhere, or an error of the library: the cache stands where it stood, and the same call
    with a good chunk goes through."""
    calls = record(monkeypatch)
    cache.append_chunk(chunk(0), chunk(1), 0)
    cache.stale_from = cache.n_loc
    before = books(cache)
    bad = torch.zeros(H, NQ + 1, D, dtype=torch.bfloat16)
    args = [] if call == "append_chunk" else [chunk(5)]

    def refuse(*a):
        raise pbsa.PbsaError(pbsa.PBSA_EINVAL)

    with monkeypatch.context() as m:
        if why == "library":
            m.setattr(pbsa, "pbsa_append_chunk", refuse)
        with pytest.raises(Exception):
            getattr(cache, call)(*args, bad if why == "K" else chunk(2), bad if why == "V" else chunk(3), 1)
    assert books(cache) == before
    del calls[:]
    cache.append_chunk(chunk(2), chunk(3), 1)
    assert cache.chunk_ids == [0, 1] and cache.n_appended == 2 and cache.chunk_pos == [0, 1]
    assert calls[0][1][0].n_loc >= calls[0][1][0].nqb          # which the library checks


def test_who_pools_the_newest_chunk(cache, monkeypatch):
    """A program that appends and selects by itself may change the rows in the ring in between: the selection pools what is
    there.  A step takes the pooled keys with the append and its selection starts behind them -- unless the chunk went
    through torch, or something older is stale as well."""
    calls = record(monkeypatch)
    nqb = cache.nqb

    def pooling():                           # by the append; from which block by the selection; of how many
        kc = [a[7] is not None for n, a in calls if n == "pbsa_append_chunk"]
        sel = [(a[0].pool_from, a[0].n_loc) for n, a in calls if n == "pbsa_select_blocks"]
        del calls[:]
        return kc, sel

    cache.append_chunk(chunk(0), chunk(1), 0)
    cache.select(chunk(2))
    assert pooling() == ([False], [(0, nqb)])
    cache.rewrite_chunk(chunk(3), chunk(4))
    cache.select(chunk(2))
    assert pooling() == ([False], [(0, nqb)])
    cache.step(chunk(0), chunk(1), chunk(2), 1)
    assert pooling() == ([True], [(2 * nqb, 2 * nqb)])
    for call in (cache.step_fused, cache.step_fine, cache.step):
        call(chunk(0), chunk(1), chunk(2), 2)
        assert pooling() == ([True], [(2 * nqb, 2 * nqb)])
    cache.step(chunk(0), chunk(1).float(), chunk(2), 3)          # converted by torch
    assert pooling() == ([], [(nqb, 2 * nqb)])
    cache.stale_from = 0
    cache.step(chunk(0), chunk(1), chunk(2), 4)
    assert pooling() == ([True], [(0, 2 * nqb)])
    # a step that ends between the two leaves nothing behind for the selection that follows
    with monkeypatch.context() as m:
        m.setattr(pbsa, "pbsa_select_blocks", lambda *a, **k: 1 / 0)
        with pytest.raises(ZeroDivisionError):
            cache.step(chunk(0), chunk(1), chunk(2), 5)
    cache.select(chunk(2))
    assert pooling() == ([True], [(nqb, 2 * nqb)])
