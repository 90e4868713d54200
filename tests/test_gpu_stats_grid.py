"""Block statistics on either side of the size that chooses their workgroups: per-block values and counts must be those of the
rows taken a few at a time."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def whole_is_the_sum(B, K, rows, signed, part=16):
    import paper_2511_04214_amd as brq
    brq.lib()
    th = (0.5, 1.5, 3.0)
    g = torch.Generator(device="cuda").manual_seed(B + K)
    x = torch.randn((max(rows), K), generator=g, device="cuda").to(torch.bfloat16)
    signs = (torch.randint(0, 2, (K,), generator=g, device="cuda") * 2 - 1).to(torch.int8) if signed else None
    flipped = x * signs.to(x.dtype) if signed else x
    parts = [brq.block_stats(flipped[i:i + part], B, thresholds=th) for i in range(0, max(rows), part)]
    amax, loss = (torch.cat([p[k] for p in parts]) for k in (0, 2))
    for M in rows:
        print("case", B, K, M, signed, flush=True)
        got = brq.block_stats(x[:M], B, thresholds=th, signs=signs)
        assert torch.equal(got[0], amax[:M]) and torch.equal(got[2], loss[:M])
        full = M // part
        want = sum((p[1] for p in parts[:full]), torch.zeros_like(got[1]))
        if M % part:
            want = want + brq.block_stats(flipped[full * part:M], B, thresholds=th)[1]
        assert torch.equal(got[1], want)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B", [1, 32, 256, 1024, 2048])
def test_whole_is_the_sum_of_its_parts(B, dtype):
    import paper_2511_04214_amd as brq
    brq.lib()
    K, th = 8192, (0.5, 1.5, 3.0)
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn((2051, K), generator=g, device="cuda").to(dtype)
    for M in (1, 7, 2048, 2051):        # 2048 x 8192: the last of one workgroup a compute unit
        print("case", B, dtype, M, flush=True)
        amax, counts, loss = brq.block_stats(x[:M], B, thresholds=th)
        parts = [brq.block_stats(x[i:min(i + 100, M)], B, thresholds=th) for i in range(0, M, 100)]
        assert torch.equal(amax, torch.cat([p[0] for p in parts])) and torch.equal(loss, torch.cat([p[2] for p in parts]))
        assert torch.equal(counts, sum(p[1] for p in parts))
        if B == 1:
            assert counts.tolist() == [int((x[:M].float().abs() > t).sum()) for t in th]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("B,K,rows", [(32, 736, (1, 445, 446)), (32, 8192, (40, 41)), (512, 4096, (80, 81))])
def test_small_launches(B, K, rows, signed):
    """About 80 * 512 chunks of 8 values, where workgroups of 512 threads become workgroups of 1024."""
    whole_is_the_sum(B, K, rows, signed)


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("K,rows", [(8192, (99, 100, 101)), (1024, (800, 801, 3 << 14, (3 << 14) + 1))])
def test_blocks_of_1024(K, rows, signed):
    """800 and 3 * 2^14 blocks, between which workgroups have 1024 threads."""
    whole_is_the_sum(1024, K, rows, signed, part=max(rows) // 7)


@pytest.mark.parametrize("K,rows", [(736, (300, 1090, 1130)), (4128, (300, 1000, 1050))])
def test_signed_rows_that_do_not_divide_the_grid(K, rows):
    """Either side of the sizes where the grid is rounded to whole rows of columns, so that signs are read once, and where not."""
    whole_is_the_sum(32, K, rows, True, part=50)
