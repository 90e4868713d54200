"""The product's LDS-staged kernel for what the others do not take: row-major K of any 32 elements, mixed layouts with K of no whole
superstages.  Tiles short of full and past it, a last pair of stages of every number of groups, output rows anywhere.  Tiled
operands of the same values go to another kernel, which sums in the same order: the results must be its, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def brq():
    import paper_2511_04214_amd as b
    b.lib()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return b


@pytest.mark.parametrize("M,N,Ks", [
    (17, 1, (2080, 4000)), (64, 130, (2112, 2144)), (65, 257, (4128, 4160, 4192, 4256)), (128, 385, (4320, 4896)), (300, 129, (8160,)),
    (1000, 4100, (288, 416, 480, 544)), (2100, 4096, (256, 384, 800)), (640, 8191, (352,))])
def test_any_k(brq, M, N, Ks):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    for K in Ks:
        x, w = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
        q = {(n, l): brq.rotate_quantize_fused(t, 32, layout=l) for n, t in (("a", x), ("w", w)) for l in ("rowmajor", "tiled")}
        want = brq.mxfp4_gemm(*q["a", "tiled"], *q["w", "tiled"], a_layout="tiled", w_layout="tiled", M=M, N=N, K=K)
        for la, lw in (("rowmajor", "rowmajor"), ("tiled", "rowmajor"), ("rowmajor", "tiled")):
            for dt, pad in ((torch.float32, 0), (torch.bfloat16, 3), (torch.bfloat16, 32)):
                print("case", M, N, K, la, lw, dt, pad, flush=True)
                assert la != lw or brq.diag_mxfp4_gemm_route(M, N, K, la, lw, dt, ldy=N + pad) == "general"
                buf = torch.full((M + 1, N + pad), -7.0, dtype=dt, device="cuda")
                brq.mxfp4_gemm(*q["a", la], *q["w", lw], out=buf[:M, :N], a_layout=la, w_layout=lw, M=M, N=N, K=K)
                assert torch.equal(buf[:M, :N], want.to(dt))
                buf[:M, :N] = -7.0
                assert (buf == -7.0).all(), "wrote outside the M x N block"
