"""Pooling by tiles (up to 768 blocks in a launch at d = 64, 128 at d = 128) and by threads (more), bit for bit against additions in
the pinned order: the largest launch of the one and the smallest of the other, lengths of none, one, around a sweep's rows, whole and beyond."""
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


@pytest.mark.parametrize("d,B", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_pooling_at_the_lines(d, B):
    line = 768 if d == 64 else 128
    for n in (line, line + 1):
        test_pooling_every_bit(d, B, n)


@pytest.mark.parametrize("d,B,blocks,heads,tail", [
    (64, 64, 16, (24, 25), 64),              # whole blocks: 768 in the launch, 800
    (64, 128, 16, (32, 33), 77),             # a last one that is not: 1024, 1056
    (128, 64, 16, (4, 5), 64),               # 128, 160
    (128, 64, 16, (16, 17), 3),              # 512, 544
    (128, 128, 16, (32, 33), 1),             # 1024, 1056
])
def test_pooling_for_a_selection(d, B, blocks, heads, tail):
    """A chunk's keys and queries on either side of each line of the selection's pooling launch: as the append pools them."""
    import numpy as np
    from paper_2604_21221_amd.cache import PbsaCache
    for H in heads:
        print(f"[case] pooling launch d={d} B={B} {H} heads x {blocks}, last {tail}", flush=True)
        nq = (blocks - 1) * B + tail
        one, two = (PbsaCache(H, d, B, nq, 0, 1, 2, np.float32(d ** -0.5), device=DEV) for _ in range(2))
        gen = torch.Generator(device=DEV).manual_seed(d + nq)
        q, k, v = (torch.randn(nq, H, d, generator=gen, device=DEV).to(torch.bfloat16).transpose(0, 1) for _ in range(3))
        one.append_chunk(k, v, 0)
        one.select(q)
        two._write_chunk(0, k, v, True, True, q)
        two.append_chunk(k, v, 0)
        if H * blocks > 400:                 # its append leaves the queries to the selection
            two.stale_from = two.n_loc
            two.select(q)
        for name in ("Kc_l", "Qc"):
            assert torch.equal(getattr(one, name).view(torch.int32), getattr(two, name).view(torch.int32)), name
