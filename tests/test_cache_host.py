"""Host side of PbsaCache without a GPU: a cache of CPU tensors whose library calls are replaced by recorders."""
import pytest

torch = pytest.importorskip("torch")

from paper_2604_21221_amd import pbsa  # noqa: E402
from paper_2604_21221_amd.cache import PbsaCache  # noqa: E402

H, D, B, NQ, W = 2, 64, 64, 200, 1


@pytest.fixture
def cache():
    c = PbsaCache(H, D, B, NQ, W, 3, 12, D ** -0.5, device="cpu")
    c._installed = 3                         # as by set_persistent()
    return c


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
    cache.adopt_chunk(1)
    for _ in range(2):
        cache.attention(chunk())
    ws = [a[12] for a in calls]
    assert all(w.numel() == cache._attn_bytes > 0 for w in ws)
    assert not overlap(*ws) and not overlap(calls[0][10], calls[1][10])
    for name, t in vars(cache).items():
        if isinstance(t, torch.Tensor):
            assert not any(overlap(w, t) for w in ws), name


CALLS = ("pbsa_append_chunk", "pbsa_select_blocks", "pbsa_pool_blocks", "pbsa_attention_fwd", "pbsa_attention_fwd_split",
         "pbsa_attention_fwd_plan_split", "pbsa_attention_fwd_mass_split", "pbsa_attention_fwd_plan",
         "pbsa_attention_fwd_mass", "pbsa_attention_bwd", "pbsa_memory_update", "pbsa_memory_update_apply",
         "pbsa_memory_update_fine")


def record(monkeypatch):
    """The library's calls from here on (but for the one by which a new cache asks what its geometry can do)."""
    calls = []
    for name in CALLS:
        monkeypatch.setattr(pbsa, name, lambda *a, name=name, **k: a[1:3] == (None, None) or calls.append((name, a)))
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


def rows(cache, t, pos=0):
    return t[:, pos * cache.nqb:(pos + 1) * cache.nqb].view(H, cache.nqb * B, D)[:, :NQ]


@pytest.mark.parametrize("which", ["K", "V"])
def test_gradients_reach_an_appended_tensor(cache, monkeypatch, which):
    """A copy into the ring is part of the graph: the gradient of the ring reaches K and V, and stops at rows that are
    written over."""
    calls = record(monkeypatch)
    x, w = chunk(0).requires_grad_(), chunk(1).float()
    cache.append_chunk(*((x, chunk(2)) if which == "K" else (chunk(2), x)), 0)
    ring = cache.Kl if which == "K" else cache.Vl
    assert not calls and torch.equal(rows(cache, ring).detach(), x.detach())
    g, = torch.autograd.grad((rows(cache, ring).float() * w).sum(), x, retain_graph=True)
    assert torch.equal(g, w.to(torch.bfloat16))
    cache.rewrite_chunk(chunk(3), chunk(3))
    assert not calls                         # the ring has a graph: the copy that cuts it off belongs there too
    g, = torch.autograd.grad((rows(cache, cache.Kl if which == "K" else cache.Vl).float() * w).sum(), x)
    assert not g.any()


def test_no_graph_no_detour(cache, monkeypatch):
    calls = record(monkeypatch)
    with torch.no_grad():
        cache.append_chunk(chunk(0).requires_grad_(), chunk(1), 0)
    with torch.inference_mode():
        cache.append_chunk(chunk(0), chunk(1), 1)
    with torch.inference_mode():
        c = PbsaCache(H, D, B, NQ, W, 3, 12, D ** -0.5, device="cpu")
        c.append_chunk(chunk(0), chunk(1), 0)
    assert len(calls) == 3
    with pytest.raises(RuntimeError, match="inference tensor"):      # as of any change in place outside the mode
        c.append_chunk(chunk(0), chunk(1), 1)
    assert len(calls) == 3 and c.chunk_ids == [0]


def test_what_follows_a_copy_sees_the_append(cache, monkeypatch):
    """Forward mode, function transforms and dispatch modes are given a copy to look at."""
    from torch.autograd import forward_ad
    from torch.utils._python_dispatch import TorchDispatchMode
    calls = record(monkeypatch)
    with forward_ad.dual_level():
        t = chunk(1)
        cache.append_chunk(forward_ad.make_dual(chunk(0), t), chunk(2), 0)
        assert torch.equal(rows(cache, forward_ad.unpack_dual(cache.Kl).tangent), t)
    c2 = PbsaCache(H, D, B, NQ, W, 3, 12, D ** -0.5, device="cpu")
    try:
        torch.func.grad(lambda x: (c2.append_chunk(x, x, 0), x.float().sum())[1])(chunk(0))
    except RuntimeError:
        pass                                 # torch may refuse the copy; a launch would not

    class Log(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.seen += func is torch.ops.aten.copy_.default
            return func(*args, **(kwargs or {}))

    c3 = PbsaCache(H, D, B, NQ, W, 3, 12, D ** -0.5, device="cpu")
    with Log() as log:
        c3.append_chunk(chunk(0), chunk(1), 0)
    assert log.seen >= 2 and not calls


def test_a_launch_counts_as_a_change_in_place(cache, monkeypatch):
    record(monkeypatch)
    q = torch.randn(D, requires_grad=True)
    y = (cache.Kl.float() @ q).sum() + (cache.Vl * q.to(torch.bfloat16)).float().sum()
    before = cache.Kl._version, cache.Vl._version
    cache.append_chunk(chunk(0), chunk(1), 0)
    assert cache.Kl._version > before[0] and cache.Vl._version > before[1]
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        y.backward()
    v = cache.Vl._version
    cache.rewrite_chunk(chunk(0))
    assert cache.Vl._version == v


def test_what_a_copy_takes_is_taken(cache, monkeypatch):
    """Everything that can be assigned to the chunk's rows: other types, shapes that spread, numbers, lazily negated
    tensors, subclasses."""
    calls = record(monkeypatch)
    x = chunk(0)
    for src in (x.float(), x[:1], x[0], x.repeat(1, 1, 2)[:, :, 1:D + 1], torch._neg_view(x), torch.nn.Parameter(x, requires_grad=False)):
        cache.rewrite_chunk(src, src) if cache.chunk_pos else cache.append_chunk(src, src, 0)
        want = src.detach().to(torch.bfloat16).expand(H, NQ, D)
        assert torch.equal(rows(cache, cache.Kl), want) and torch.equal(rows(cache, cache.Vl), want)
    cache.rewrite_chunk(0.5, 2)
    assert bool((rows(cache, cache.Kl) == 0.5).all()) and bool((rows(cache, cache.Vl) == 2).all())
    assert not calls


def test_rows_of_the_ring_are_copied_in_order(cache, monkeypatch):
    """K from the rows of Vl that V is about to take: K is copied first, then V."""
    calls = record(monkeypatch)
    with torch.no_grad():
        cache.Vl[:, :cache.nqb] = torch.randn(H, cache.nqb, B, D).to(torch.bfloat16)
    old, v = rows(cache, cache.Vl).clone(), chunk(1)
    cache.append_chunk(rows(cache, cache.Vl), v, 0)
    assert torch.equal(rows(cache, cache.Kl), old) and torch.equal(rows(cache, cache.Vl), v)
    k = chunk(2)
    cache.rewrite_chunk(k, rows(cache, cache.Kl))
    assert torch.equal(rows(cache, cache.Kl), k) and torch.equal(rows(cache, cache.Vl), k) and not calls


@pytest.mark.parametrize("kw", [dict(d=32), dict(B=32), dict(n_sink=101), dict(causal=2), dict(scale=0.0), dict(H=65536, d=32)],
                         ids=lambda kw: next(iter(kw)))
def test_a_geometry_no_kernel_takes_can_be_stored(monkeypatch, kw):
    """With more slots than the update maintains nothing of the library is asked when a cache is made: whatever the kernels
    would refuse holds chunks all the same."""
    a = dict(H=2, d=64, B=64, Nq=3, window_chunks=1, C=100, k=2, scale=0.1)
    a.update(kw)
    if a["H"] > 1000:
        a.update(C=65, Nq=1, B=1, window_chunks=0, fold=False, pass_logits=False)
    c = PbsaCache(**a, device="cpu")
    k, v = (torch.randn(a["H"], a["Nq"], a["d"]).to(torch.bfloat16) for _ in range(2))
    c.append_chunk(k, v, 0)
    for t, x in ((c.Kl, k), (c.Vl, v)):
        assert torch.equal(t[:, :c.nqb].reshape(a["H"], -1, a["d"])[:, :a["Nq"]], x)


def test_a_saved_cache_goes_on(cache, monkeypatch):
    """Saved and loaded, with scratch of whatever size it had, and from a file that holds only what a cache was first made
    of."""
    import copy
    import pickle
    calls = record(monkeypatch)
    cache.append_chunk(chunk(0), chunk(1), 0)
    cache._bwd_ws = cache._mass_ws = torch.empty(16, dtype=torch.uint8)
    old = copy.copy(cache)
    old.__dict__ = {k: v for k, v in vars(cache).items() if k not in ("_full", "_by_launch", "_attn_bytes", "_installed", "_pays")}
    for c in (pickle.loads(pickle.dumps(cache)), copy.deepcopy(cache), pickle.loads(pickle.dumps(old))):
        assert c.chunk_ids == [0] and c._attn_bytes == cache._attn_bytes > 0
        assert not hasattr(c, "_bwd_ws") and not hasattr(c, "_mass_ws")
        del calls[:]
        c.append_chunk(chunk(0), chunk(1), 1)
        c.attention(chunk(3))
        c.attention_bwd(chunk(3), chunk(3), chunk(3), torch.zeros(H, NQ))
        assert [n for n, _ in calls] == ["pbsa_append_chunk", "pbsa_attention_fwd_split", "pbsa_attention_bwd"]
        need = pbsa.pbsa_bwd_workspace_bytes(c.params())
        assert calls[-1][1][-1].numel() == need and calls[1][1][-1].numel() == c._attn_bytes


def test_no_split_for_what_is_not_there_yet(monkeypatch):
    """64 slots and a selection of one block: nothing to share out until blocks have been installed in the slots or have left
    the window for them; attention, attention with decisions and attention with mass agree at every chunk."""
    calls = record(monkeypatch)
    make = lambda: PbsaCache(H, D, B, 512, 1, 64, 1, D ** -0.5, device="cpu")
    x = torch.zeros(H, 512, D, dtype=torch.bfloat16)

    def splits(c):
        del calls[:]
        c.select(x)
        c.attention(x)
        c.attention_with_mass(x)
        c.attention_with_plan(x)
        made = [(n, a) for n, a in calls if n.startswith("pbsa_attention")]
        split = made[0][0] == "pbsa_attention_fwd_split"
        assert [n for n, _ in made] == [f"pbsa_attention_fwd{n}{'_split' if split else ''}" for n in ("", "_mass", "_plan")]
        assert not split or all(a[-1].numel() == c._attn_bytes for _, a in made)
        c.update_apply()
        return split

    c = make()
    assert c._attn_bytes > 0
    seen = []
    for g in range(12):
        c.append_chunk(x, x, g)
        seen.append(splits(c))
    assert seen == sorted(seen) and not any(seen[:3]) and seen[-1]      # from some chunk on, once 8 blocks a chunk have left
    c = make()
    c.set_persistent(torch.zeros(H, 64, B, D, dtype=torch.bfloat16), torch.zeros(H, 64, B, D, dtype=torch.bfloat16),
                     torch.full((H, 64), B, dtype=torch.int32), torch.arange(64)[None].repeat(H, 1))
    c.append_chunk(x, x, 0)
    assert splits(c)


def test_who_pools_the_queries(cache, monkeypatch):
    """A step's append pools the queries along, and its selection starts from them, where it reads them as they are and nothing
    older is stale; a selection by itself pools its own."""
    asked = []
    for name in CALLS:
        monkeypatch.setattr(pbsa, name, lambda *a, name=name, **k: asked.append((name, len(a) > 9 and a[9] is not None, k.get("pooled", False))))

    def steps(Q):
        del asked[:]
        cache.step(Q, chunk(1), chunk(2), cache.n_appended)
        return asked[0][1], asked[1][2]

    assert steps(chunk(0)) == (True, True)
    assert steps(torch.zeros(H, NQ, D + 1, dtype=torch.bfloat16)[:, :, 1:]) == (False, False)       # rows that are not aligned
    assert steps(chunk(0).requires_grad_()) == (False, False)
    cache.stale_from = 0                     # an older block is stale: the selection pools, the queries too
    assert steps(chunk(0)) == (True, False)
    cache.append_chunk(chunk(1), chunk(2), cache.n_appended)
    del asked[:]
    cache.select(chunk(0))
    assert asked == [("pbsa_select_blocks", False, False)]


@pytest.mark.parametrize("kind", [int, "int64", "int32", "int16", "tensor", float])
def test_chunk_ids_of_any_integer_type(cache, kind):
    """Whatever type of number a program counts its chunks with, consecutive or not: the update is given the blocks' ids as
    64-bit integers, where they are consecutive by a plain address."""
    import ctypes
    import numpy as np
    make = kind if kind in (int, float) else torch.tensor if kind == "tensor" else getattr(np, kind)
    nqb = cache.nqb

    def ids(first, second):
        cache.chunk_pos, cache.chunk_ids = [], []
        for g in (first, second):
            cache.adopt_chunk(make(g))
        return cache._device_maps(want_ids=True)[2]

    if kind is float:                        # not a number of a chunk, but gaps have always been taken
        with pytest.raises(TypeError):
            ids(6, 7)
    else:
        at = ids(6, 7)
        assert type(at) is int and 0 <= at - cache._arange64.data_ptr() <= 8 * (cache._arange64.numel() - 2 * nqb)
        assert list((ctypes.c_int64 * (2 * nqb)).from_address(at)) == list(range(6 * nqb, 8 * nqb))
    for first, second in ((6, 8), (7, 6), (-1, 0)):
        got = ids(first, second)
        assert got.dtype == torch.int64 and got.tolist() == [g * nqb + i for g in (first, second) for i in range(nqb)]
