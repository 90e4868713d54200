"""Parity of the one-tile-per-workgroup product kernel (64 x 128, 128 x 128, 192 x 128, 192 x 256 and 320 x 128 tiles) where it
can go wrong: one row or column past a tile, one short of it, one element per store (N or the pitch not a multiple
of a 16-byte chunk), K of a single superstage, and row-major K that is not a multiple of 512 (the last superstage is
then a window that overlaps the one before, its shared stages masked).  Bars as in test_gpu_gemm.py; every shape in
both layouts, both output types, with a guard right of column N - 1 and below row M - 1.  Each shape runs on the tile it is
listed for, and through the dispatcher, which may take another and must give the same bits."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev, to_host
from test_gpu_gemm import FLOOR, RTOL, bf16_rne
from test_gpu_layout import to_tiled

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def brq():
    import paper_2511_04214_amd as b
    b.lib()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return b


# the tile (rows x columns), then the shape
@pytest.mark.parametrize("tile,M,N,K", [
    ("64x128", 129, 77, 512), ("64x128", 129, 130, 640), ("64x128", 191, 136, 896), ("64x128", 193, 257, 1152),
    ("64x128", 129, 128, 2048), ("128x128", 193, 16390, 640), ("128x128", 577, 6150, 640), ("128x128", 383, 8200, 640),
    ("128x128", 500, 8200, 512), ("192x128", 129, 28672, 2048), ("192x128", 191, 16390, 4096),
    ("192x256", 1153, 28672, 640), ("192x256", 1153, 16390, 4096),
    # few rows (16 and more); rings deeper than K's stages and K of a few more stages than the ring
    ("64x128", 16, 300, 512), ("64x128", 17, 77, 512), ("64x128", 33, 130, 1024), ("64x128", 64, 520, 1536),
    ("64x128", 65, 264, 896), ("128x128", 128, 28672, 1024), ("320x128", 300, 28672, 2048), ("320x128", 600, 28674, 640)])
def test_tiles_of_the_mid_kernel(brq, orc, tile, M, N, K):
    from paper_2511_04214_amd import inputs
    aq, as_ = inputs.random_mxfp4(M, K, seed=M * 3 + K)
    wq, ws = inputs.random_mxfp4(N, K, seed=N * 7 + K)
    rows = sorted({M - 1, M - 2, M // 2} | {r for r in (0, 31, 32, 63, 64, 127, 128, 191, 192, 255, 256) if r < M})
    ref, bound = orc.mxfp4_gemm(aq, as_, wq, ws, rows=rows)
    ops = {"rowmajor": [to_dev(t) for t in (aq, as_, wq, ws)],
           "tiled": [to_dev(t) for t in to_tiled(aq, as_) + to_tiled(wq, ws)]}
    for layout, (a, sa, w, sw) in ops.items():
        for pad in (8, 3):
            print("case", tile, M, N, K, layout, pad, flush=True)
            out = {}
            for dt in (torch.float32, torch.bfloat16):
                buf = torch.full((M + 2, N + pad), -7.0, dtype=dt, device="cuda")
                brq.diag_mxfp4_gemm_on(tile, a, sa, w, sw, buf[:M, :N], K, a_layout=layout, w_layout=layout)
                y = brq.mxfp4_gemm(a, sa, w, sw, out_dtype=dt, a_layout=layout, w_layout=layout, M=M, N=N, K=K)
                assert torch.equal(y, buf[:M, :N]), "differs from the dispatcher's kernel"
                assert (buf[M:] == -7.0).all() and (buf[:, N:] == -7.0).all(), "wrote outside the M x N block"
                out[dt] = to_host(buf[:M, :N])
            got = out[torch.float32][np.asarray(rows)].astype(np.float64)
            err = np.abs(got - ref)
            assert (err <= RTOL * bound + FLOOR).all(), "max err/bound = %g" % float((err / (bound + FLOOR)).max())
            assert np.array_equal(out[torch.bfloat16], bf16_rne(out[torch.float32]))


def test_masked_stages_vanish_from_a_zero_sum(brq):
    """Row-major K = 640: the last window shares 384 elements with the superstage before it.  With every code 6 there
    and scale bytes 0 elsewhere, anything the masked stages leaked would be the only thing in the sum."""
    M, N, K = 200, 136, 640
    codes = torch.zeros((max(M, N), K // 2), dtype=torch.uint8, device="cuda")
    codes[:, 64:256] = 0x77                      # elements 128 .. 511: in both windows
    scales = torch.full((max(M, N), K // 32), 127, dtype=torch.uint8, device="cuda")
    y = brq.mxfp4_gemm(codes[:M], scales[:M], codes[:N], scales[:N])
    assert (y == 36.0 * 384).all(), "the shared stages were counted %s times" % float(y[0, 0] / (36.0 * 384))
    scales[:, 4:16] = 0                          # the shared groups' own scales: 2^-127 * 2^-127
    y = brq.mxfp4_gemm(codes[:M], scales[:M], codes[:N], scales[:N])
    assert (y == 0).all()
