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
                assert la != lw or brq.diag_mxfp4_gemm_route(M, N, K, la, lw, dt, ldy=N + pad) == "any_k"
                buf = torch.full((M + 1, N + pad), -7.0, dtype=dt, device="cuda")
                brq.mxfp4_gemm(*q["a", la], *q["w", lw], out=buf[:M, :N], a_layout=la, w_layout=lw, M=M, N=N, K=K)
                assert torch.equal(buf[:M, :N], want.to(dt))
                buf[:M, :N] = -7.0
                assert (buf == -7.0).all(), "wrote outside the M x N block"


def test_scales_past_2_gib(brq):
    """K = 2^30 + 512: the weights' scales of the last superstage lie 2^31 bytes behind their row's first (tiled, one slab of 36 GB).  Codes
    1 in 32 groups at either end of K and around that place, 0 elsewhere; all sums are exact."""
    M, N, K = 17, 15, 2 ** 30 + 512
    ac, as_ = torch.zeros((M, K // 2), dtype=torch.uint8, device="cuda"), torch.full((M, K // 32), 127, dtype=torch.uint8, device="cuda")
    wc, ws = (torch.full((n,), v, dtype=torch.uint8, device="cuda") for n, v in zip(brq.operand_bytes(N, K, "tiled"), (0, 127)))
    g = torch.Generator(device="cuda").manual_seed(3)
    want = torch.zeros((M, N), dtype=torch.float64)
    for at in (0, 2 ** 25 - 48, 2 ** 25 - 16):              # first of 32 groups, two superstages of the weights
        ea, ew = (torch.randint(0, 5, (n, 32), generator=g, device="cuda") for n in (M, N))
        ac[:, 16 * at:16 * at + 512] = 0x22
        as_[:, at:at + 32] = (125 + ea).to(torch.uint8)
        wc.view(K // 128, 64, 64)[at // 4:at // 4 + 8, :N] = 0x22
        ws.view(K // 512, 64, 16)[at // 16:at // 16 + 2, :N] = (125 + ew).to(torch.uint8).view(N, 2, 16).transpose(0, 1)
        want += 32 * torch.exp2(ea.cpu().double() - 2) @ torch.exp2(ew.cpu().double() - 2).t()
    assert torch.equal(brq.mxfp4_gemm(ac, as_, wc, ws, w_layout="tiled", N=N).cpu().double(), want)
