"""The weight-streaming kernel and the one-launch decode call, whose workgroups own 32, 64 or 128 columns by how many there
are: one column past and short of the numbers where that changes, ragged columns, K of every number of superstages
around the register rotation's length, 1 to 16 rows.  The one-tile kernel sums in the same order: the results must be its,
bit for bit."""
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


@pytest.mark.parametrize("columns", [1, 31, 33, 300, "32", "32 + 1", "64 - 1", "64 + 1"])
def test_streaming_kernel_is_the_one_tile_kernel(brq, columns):
    N = columns if isinstance(columns, int) else (int(columns.split()[0]) * cus() + int("".join(columns.split()[1:]) or 0))
    g = torch.Generator(device="cuda").manual_seed(N)
    for nss in (1, 2, 4, 5, 6, 7, 8, 9, 10, 14) if N <= 300 else (3, 4, 5, 8):
        K = 512 * nss - (96 if nss % 3 == 0 else 0)             # (tiled operands are padded to whole superstages)
        w = brq.rotate_quantize_fused(torch.randn((N, K), generator=g, device="cuda"), 32, layout="tiled")
        for M in (1, 7, 16):
            print("case", N, K, M, flush=True)
            x = torch.randn((M, K), generator=g, device="cuda")
            a = brq.rotate_quantize_fused(x, 32, layout="tiled")
            out = []
            for route in ("stream", "64x128"):
                buf = torch.full((M + 1, N + 3), -7.0, device="cuda")
                brq.diag_mxfp4_gemm_on(route, *a, *w, buf[:M, :N], K, a_layout="tiled", w_layout="tiled")
                out.append(buf[:M, :N].clone())
                buf[:M, :N] = -7.0
                assert (buf == -7.0).all(), "wrote outside the M x N block"
            assert torch.equal(out[0], out[1])
            if K % 512 == 0:
                for xs in (x, x.to(torch.bfloat16)):
                    two = brq.mxfp4_gemm(*brq.rotate_quantize_fused(xs, 32, layout="tiled"), *w, a_layout="tiled", w_layout="tiled", M=M, N=N, K=K)
                    assert torch.equal(brq.rotate_quantize_gemm_fused(xs, 32, *w, N, w_layout="tiled"), two)
