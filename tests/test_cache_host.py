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
