"""The product's tiles of 256 x 128, which it takes in place of 320 x 128 and 192 x 256 where they go round the chip as often: rows
and columns around a tile's, K with and without an overlapping last window, mixed layouts, pitches on and off lines.  All product
kernels but one sum in the same order, so the result is that of the kernel it takes the place of, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def brq():
    import paper_2511_04214_amd as b
    b.lib()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return b


# rows left of a tile of 256 (64 of them a wavefront's two MFMA tiles), columns left, K over 512
SHAPES = [(0, 0, 2688), (250, 6, 2048), (63, 64, 4224), (140, 120, 1152), (255, 16, 3328), (128, 6, 2944), (129, 64, 1664), (192, 1, 2560)]


# (mixed layouts take whole superstages)
@pytest.mark.parametrize("rows,cols,K,layouts", [(*s, (a, w)) for s in SHAPES for a, w in (("rowmajor", "rowmajor"), ("tiled", "rowmajor"), ("rowmajor", "tiled"))
                                                 if a == w or s[2] % 512 == 0])
def test_tall_tile(brq, rows, cols, K, layouts):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device="cuda").manual_seed(rows * 7 + cols + K)
    found = 0
    for tm in (1, 2, 4, 7, 8):                                # tiles of 256 x 128 down; as many across as one round has room for
        M = 256 * (tm - (rows > 0)) + rows
        N = 128 * (cus // tm - (cols > 0)) + cols
        for out in (torch.bfloat16, torch.float32):
            if M <= 16 or brq.diag_mxfp4_gemm_route(M, N, K, *layouts, out, cus=cus) != "256x128":
                continue
            found += 1
            print("case", M, N, K, layouts, out, flush=True)
            x, w = (torch.randn((n, K), generator=g, device="cuda") for n in (M, N))
            a, b = brq.rotate_quantize_fused(x, 32, layout=layouts[0]), brq.rotate_quantize_fused(w, 32, layout=layouts[1])
            for pad in (0, 3):
                y, want = (torch.full((M + 1, N + pad), -7.0, dtype=out, device="cuda") for _ in range(2))
                brq.mxfp4_gemm(*a, *b, out=y[:M, :N], out_dtype=out, a_layout=layouts[0], w_layout=layouts[1], M=M, N=N, K=K)
                brq.diag_mxfp4_gemm_on("320x128", *a, *b, want[:M, :N], K, a_layout=layouts[0], w_layout=layouts[1])
                assert torch.equal(y, want)                   # (the cells beside the product too: untouched)
    assert found, "no such shape goes this way"


# tiled over 320 x 128 in one and in two rounds of 256 workgroups and over 192 x 256 in two, row-major over both in two; the route is bf16's
@pytest.mark.parametrize("M,N,K,layout", [(3913, 3746, 4224, "tiled"), (6046, 2568, 8192, "tiled"), (1194, 6374, 5504, "tiled"), (2840, 2623, 9344, "tiled"),
                                          (4078, 1876, 5248, "tiled"), (4642, 2744, 8064, "rowmajor"), (5924, 2584, 1536, "rowmajor"), (5063, 3200, 1536, "rowmajor")])
def test_tall_tile_by_name(brq, M, N, K, layout):
    assert brq.diag_mxfp4_gemm_route(M, N, K, layout, layout, torch.bfloat16) == "256x128"
    lay = dict(a_layout=layout, w_layout=layout)
    g = torch.Generator(device="cuda").manual_seed(M + K)
    a, b = (brq.rotate_quantize_fused(torch.randn((n, K), generator=g, device="cuda"), 32, layout=layout) for n in (M, N))
    for out in (torch.bfloat16, torch.float32):
        print("case", M, N, K, layout, out, flush=True)
        for pad in (0, 3):
            z, y, want = (torch.full((M + 1, N + pad), -7.0, dtype=out, device="cuda") for _ in range(3))
            brq.mxfp4_gemm(*a, *b, out=z[:M, :N], out_dtype=out, **lay, M=M, N=N, K=K)
            brq.diag_mxfp4_gemm_on("256x128", *a, *b, y[:M, :N], K, **lay)
            brq.diag_mxfp4_gemm_on("320x128", *a, *b, want[:M, :N], K, **lay)
            assert torch.equal(y, want) and torch.equal(z, want)
