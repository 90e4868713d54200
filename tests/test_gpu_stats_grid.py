"""Block statistics on either side of the size that chooses their workgroups: per-block values and counts must be those of the
rows taken a few at a time."""
import pytest
import torch

pytestmark = pytest.mark.gpu


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
