"""Outputs that leave by more than one kind of store: the product's rows on and off 128-byte lines, and codes that go
through the L2 or past it.  Either kind must give the same bytes, and write nothing outside its block."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def brq():
    import paper_2511_04214_amd as b
    b.lib()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return b


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("route", ["256x256", "128x256", "64x128", "128x128", "192x128", "192x256", "320x128", "256x128"])
def test_product_rows_on_and_off_lines(brq, route, dtype):
    """N of whole 128-byte lines, 16-byte chunks, and (one-tile kernels) anything; rows that begin on a line (pitch 512,
    column 0), on a 16-byte chunk (pitch 520, or column 8), on a half line (column 32 of bf16), and anywhere (pitch 517; an
    output that begins anywhere is refused)."""
    M, K = 133, 512
    g = torch.Generator(device="cuda").manual_seed(3)
    a = brq.rotate_quantize_fused(torch.randn((M, K), generator=g, device="cuda"), 32, layout="tiled")
    for N in (384, 296) + ((301, 293) if "256" not in route.split("x")[1] or route == "192x256" else ()):
        w = brq.rotate_quantize_fused(torch.randn((N, K), generator=g, device="cuda"), 32, layout="tiled")
        want = torch.empty((M, N), dtype=dtype, device="cuda")
        brq.diag_mxfp4_gemm_on("general", *a, *w, want, K, a_layout="tiled", w_layout="tiled")
        for pitch, col in ((512, 0), (512, 8), (520, 0), (544, 32)) + (((517, 0),) if N % 8 else ()):
            print("case", route, dtype, N, pitch, col, flush=True)
            buf = torch.full((M + 1, pitch), -7.0, dtype=dtype, device="cuda")
            brq.diag_mxfp4_gemm_on(route, *a, *w, buf[:M, col:col + N], K, a_layout="tiled", w_layout="tiled")
            assert torch.equal(buf[:M, col:col + N], want)
            buf[:M, col:col + N] = -7.0
            assert (buf == -7.0).all(), "wrote outside the block"


@pytest.mark.parametrize("B", [32, 512, 2048])
@pytest.mark.parametrize("layout,M,K", [("rowmajor", 256, 2048), ("tiled", 4096, 8192)])
def test_codes_on_either_side_of_the_size_that_chooses_their_store(brq, layout, M, K, B):
    """M rows are the first number whose codes go through the L2; the halves, quantized by themselves, go past it (tiled codes of
    B = 2048, a register rotation, all go through it: see below)."""
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    both = [brq.rotate_quantize_fused(x[i:i + M // 2], B, layout=layout) for i in (0, M // 2)]
    for rows in (M - 64, M):
        print("case", layout, rows, K, B, flush=True)
        codes, scales = brq.rotate_quantize_fused(x[:rows], B, layout=layout)
        for whole, parts in ((codes, [b[0] for b in both]), (scales, [b[1] for b in both])):
            assert torch.equal(whole.flatten(), torch.cat(parts).flatten()[:whole.numel()])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,K,first,gated", [
    (2048, 2048, 256, False), (8192, 8192, 64, False),                                      # register rotations (bf16): from 256 KB
    (32, 11008, 191, False), (256, 11008, 191, True), (32, 11008, 191, True),               # K above 8192: from 1 MB, K padding behind
    (32, 8224, 256, False), (8, 8224, 256, True), (1, 11008, 191, True)])
def test_tiled_codes_on_either_side_of_the_size_that_chooses_their_store(brq, B, K, first, gated, dtype):
    """`first` rows are the first number whose tiled codes go through the L2.  Rows by themselves, a few at a time, go past it."""
    g = torch.Generator(device="cuda").manual_seed(B + K)
    x, u = (torch.randn((first + 1, K), generator=g, device="cuda").to(dtype) for _ in range(2))

    def step(lo, hi):
        if gated:
            t = brq.swiglu_rotate_quantize_fused(x[lo:hi], u[lo:hi], B, layout="tiled")
        else:
            t = brq.rotate_quantize_fused(x[lo:hi], B, layout="tiled")
        return t, brq.to_rowmajor(*t, hi - lo, K)

    n = 40
    parts = [step(i, min(i + n, first + 1))[1] for i in range(0, first + 1, n)]
    codes, scales = (torch.cat([p[k] for p in parts]) for k in (0, 1))
    Kp = (K + 511) // 512 * 512
    for rows in (first - 1, first, first + 1):
        print("case", B, K, rows, gated, dtype, flush=True)
        tiled, (c, s) = step(0, rows)
        assert torch.equal(c, codes[:rows]) and torch.equal(s, scales[:rows])
        if Kp > K:                       # the K padding of the rows of whole slabs: zeros
            slabs = rows // 64
            pad = tiled[0][:slabs * 64 * (Kp // 2)].view(slabs, Kp // 128, 64, 64).transpose(1, 2).reshape(slabs * 64, Kp // 2)[:, K // 2:]
            assert not pad.any()
