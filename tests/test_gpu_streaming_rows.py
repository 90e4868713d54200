"""Up to 16 rows against row-major weights: a wavefront loads whole lines of 32 rows and turns them round in LDS.  Columns
around a wavefront's, a workgroup's and a chip's share, K of every number of superstages around the register rotation's length and
the longest that the one-launch call takes.  The general kernel sums in the same order and reads no LDS, and tiled weights go
another way: the results must be theirs, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def brq():
    import paper_2511_04214_amd as b
    b.lib()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return b


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def product(brq, route, a, w, M, N, K, la, lw):
    buf = torch.full((M + 1, N + 3), -7.0, device="cuda")
    brq.diag_mxfp4_gemm_on(route, *a, *w, buf[:M, :N], K, a_layout=la, w_layout=lw)
    y = buf[:M, :N].clone()
    buf[:M, :N] = -7.0
    assert (buf == -7.0).all(), "wrote outside the M x N block"
    return y


@pytest.mark.parametrize("columns", [1, 7, 31, 33, 130, "32", "32 + 1", "64 - 1", "64 + 1"])
def test_row_major_weights(brq, columns):
    N = columns if isinstance(columns, int) else (int(columns.split()[0]) * cus() + int("".join(columns.split()[1:]) or 0))
    g = torch.Generator(device="cuda").manual_seed(N)
    for nss in (1, 2, 3, 4, 5, 6, 7, 8, 14, 32) if N <= 130 else (1, 4, 5):
        K = 512 * nss
        ww = torch.randn((N, K), generator=g, device="cuda")
        w = {l: brq.rotate_quantize_fused(ww, 32, layout=l) for l in ("rowmajor", "tiled")}
        for M in (1, 7, 16):
            print("case", N, K, M, flush=True)
            x = torch.randn((M, K), generator=g, device="cuda")
            a = {l: brq.rotate_quantize_fused(x, 32, layout=l) for l in ("rowmajor", "tiled")}
            want = product(brq, "general", a["rowmajor"], w["rowmajor"], M, N, K, "rowmajor", "rowmajor")
            for la, lw in (("rowmajor", "rowmajor"), ("tiled", "rowmajor"), ("rowmajor", "tiled")):
                assert torch.equal(product(brq, "stream", a[la], w[lw], M, N, K, la, lw), want)
            assert torch.equal(brq.mxfp4_gemm(*a["rowmajor"], *w["rowmajor"]), want)
            for out in (torch.float32, torch.bfloat16):
                y = brq.rotate_quantize_gemm_fused(x, 32, *w["rowmajor"], N, out_dtype=out)
                assert torch.equal(y, want.to(out))
