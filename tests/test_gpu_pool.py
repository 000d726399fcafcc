"""Pooling by tiles (up to 1024 blocks in a launch) and by threads (more), bit for bit against additions in the pinned order: the
largest launch of the one and the smallest of the other, lengths of none, one, around a sweep's rows, whole and beyond."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [1, 1024, 1025])
@pytest.mark.parametrize("d,B", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_pooling_every_bit(d, B, n):
    from paper_2604_21221_amd import pbsa
    print(f"[case] pooling d={d} B={B} blocks={n}", flush=True)
    gen = torch.Generator().manual_seed(n + d + B)
    X = (3.0 * torch.randn(n, B, d, generator=gen)).to(torch.bfloat16)
    X[0, 0, 0], X[0, 0, 1], X[-1, 1, 2] = float("-inf"), float("nan"), float("inf")
    lens = torch.tensor([B - 1, 0, 1, 15, 16, 17, 32, 33, B, B + 5, -3], dtype=torch.int32).repeat(n // 11 + 1)[:n]
    lens[-1] = B
    want, rows = torch.zeros(n, d), lens.clamp(0, B)
    for r in range(B):
        want = torch.where((r < rows)[:, None], want + X[:, r].float(), want)
    want = torch.where(rows[:, None] > 0, want / rows.clamp(min=1)[:, None].float(), torch.zeros(()))
    out = torch.full((n, d), 7.0, device=DEV)
    pbsa.pbsa_pool_blocks(pbsa.make_params(1, d, B, B, 1, 1, 1, 1, 1.0), X.to(DEV), lens.to(DEV), n, out)
    got = out.cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got.nan_to_num(0.5).view(torch.int32), want.nan_to_num(0.5).view(torch.int32))
