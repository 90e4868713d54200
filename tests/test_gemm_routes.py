"""Which kernel the product takes for a shape, on the CPU (host arithmetic for a device of 256 compute units).  The
parity tests of test_gpu_gemm_routes.py run every kernel by its name; these say that the dispatcher uses them."""
import os
import subprocess

import pytest
import torch

import paper_2511_04214_amd as brq

BF16, F32 = torch.bfloat16, torch.float32


def route(M, N, K, layout="tiled", dtype=BF16, **kw):
    return brq.diag_mxfp4_gemm_route(M, N, K, layout, layout, dtype, **kw)


@pytest.mark.parametrize("shape,layout,want", [
    ((16, 256, 256), "rowmajor", "skinny"), ((16, 256, 256), "tiled", "stream"), ((1, 28672, 8192), "tiled", "stream"),
    ((16, 28672, 8192), "tiled", "stream"), ((100, 28672, 8192), "tiled", "128x128"), ((300, 28672, 8192), "tiled", "320x128"),
    ((300, 28672, 8192), "rowmajor", "320x128"), ((2048, 8192, 2048), "tiled", "256x256"), ((4096, 2048, 8192), "tiled", "128x256"),
    ((8192, 14336, 4096), "tiled", "256x256"), ((1000, 4096, 11008), "tiled", "128x128"), ((1000, 4096, 11008), "rowmajor", "192x128"),
    ((2000, 4096, 11008), "rowmajor", "256x128"), ((192, 256, 4096), "tiled", "64x128"),
    # ragged rows and columns, and K of one superstage, on the persistent kernel
    ((4100, 14344, 4096), "tiled", "256x256"), ((5000, 8200, 4096), "tiled", "256x256"), ((5000, 8200, 4096), "rowmajor", "256x256"),
    ((8192, 14336, 512), "rowmajor", "256x256"),
    # short K of row-major operands: single stages of 128 x 128, two workgroups a CU
    ((4000, 8192, 512), "rowmajor", "128x128"), ((787, 17600, 512), "rowmajor", "128x128"), ((1100, 1000, 512), "rowmajor", "64x128"),
    # N or K that no staged kernel takes, on either side of where LDS pays
    ((300, 520, 96), "rowmajor", "general"), ((40, 70, 256), "rowmajor", "general"), ((4, 70, 1056), "rowmajor", "skinny"),
    ((300, 2048, 1056), "rowmajor", "general"), ((1000, 8192, 544), "rowmajor", "any_k"), ((64, 1024, 2080), "rowmajor", "any_k"),
    ((15897, 2, 672), "rowmajor", "general"), ((4182, 5, 3872), "rowmajor", "general"), ((141, 5692, 1088), "rowmajor", "general"),
    ((2000, 520, 2080), "rowmajor", "any_k"), ((141, 28672, 1088), "rowmajor", "any_k"), ((300, 7, 4128), "rowmajor", "any_k")])
def test_route(shape, layout, want):
    assert route(*shape, layout=layout) == want


@pytest.mark.parametrize("shape,layout,dtype,want", [
    ((250, 28672, 8192), "rowmajor", BF16, "256x128"), ((1000, 8192, 4096), "rowmajor", BF16, "256x128"), ((3769, 2136, 1536), "rowmajor", BF16, "256x128"),
    ((5924, 2584, 1536), "rowmajor", BF16, "256x128"), ((4642, 2744, 8064), "rowmajor", F32, "256x128"), ((4642, 2744, 8064), "rowmajor", BF16, "256x128"),
    ((1194, 6374, 5504), "tiled", BF16, "256x128"), ((2840, 2623, 9344), "tiled", F32, "256x128"), ((4078, 1876, 5248), "tiled", BF16, "256x128"),
    ((3913, 3746, 4224), "tiled", BF16, "256x128"), ((6046, 2568, 8192), "tiled", BF16, "256x128"), ((6046, 2568, 8192), "tiled", F32, "256x128"),
    ((7459, 2176, 2560), "tiled", BF16, "256x128"),
    # a round more; tiled, 192 x 256 in one round
    ((834, 18856, 2048), "rowmajor", BF16, "320x128"), ((2300, 4096, 1536), "rowmajor", BF16, "192x256"), ((300, 28672, 8192), "tiled", BF16, "320x128"),
    ((3776, 2080, 4224), "tiled", F32, "192x256")])
def test_tall_tile(shape, layout, dtype, want):
    """256 x 128 in place of 320 x 128 and 192 x 256 where it goes round the chip as often, in one round and in two."""
    assert route(*shape, layout=layout, dtype=dtype) == want


def test_few_rows():
    """Up to 16 rows: weight streaming, whatever the layouts."""
    for M in (1, 16):
        for N, K in ((256, 512), (2048, 2048), (28672, 8192)):
            for la in ("rowmajor", "tiled"):
                for dt in (F32, BF16):
                    assert brq.diag_mxfp4_gemm_route(M, N, K, la, "tiled", dt) == "stream"
                    assert brq.diag_mxfp4_gemm_route(M, N, K, la, "rowmajor", dt) == "stream"


def test_every_kernel_is_taken_somewhere():
    seen = {}
    for layout in ("rowmajor", "tiled"):
        for M in (1, 16, 40, 130, 200, 300, 500, 600, 1000, 1100, 2048, 4096, 8192):
            for N in (128, 1024, 2048, 4096, 8192, 28672):
                for K in (96, 512, 2048, 2080, 4096, 8192, 11008):
                    seen.setdefault(route(M, N, K, layout=layout), set()).add(layout)
    assert set(seen) == set(brq.GEMM_ROUTES)


def test_arguments():
    for bad in (dict(ldy=127), dict(cus=0)):
        with pytest.raises(brq.BrqError) as e:
            route(4, 128, 512, **bad)
        assert e.value.status == 2
    for shape in ((0, 128, 512), (4, 0, 512), (4, 128, 40)):
        with pytest.raises(brq.BrqError) as e:
            route(*shape)
        assert e.value.status == 2
    # N or a pitch that is not whole 16-byte chunks keeps a call off the persistent kernel
    assert route(8192, 14338, 4096) not in ("256x256", "128x256")
    assert route(8192, 14336, 4096, ldy=14339) not in ("256x256", "128x256")


@pytest.mark.parametrize("layout", ["rowmajor", "tiled"])
def test_long_k_stays_on_a_staged_kernel(layout):
    # a lane's 32-bit offset inside a tile: 2 slabs of 64 rows up to K < 2^26, 4 up to 2^25
    for K in (2 ** 24 + 512, 2 ** 25, 2 ** 26 - 512):
        for M in (17, 100, 128):
            assert route(M, 130, K, layout=layout) in ("64x128", "128x128")
    assert route(17, 130, 2 ** 26, layout=layout) == "any_k"
    assert route(300, 130, 2 ** 25 + 512, layout=layout) in ("64x128", "128x128", "192x128")


@pytest.mark.parametrize("shape,on,off", [((6812, 3520, 2048), "192x256", "256x256"), ((4434, 4224, 2048), "192x256", "320x128")])
def test_an_output_that_begins_off_a_line_is_one_off_lines(shape, on, off, tmp_path):
    """The product's rows lie off 128-byte lines by their pitch or by where the output begins: the same choice of tile.
    (The public call has no address: the library's own is compiled against here.)"""
    M, N, K = shape
    assert route(M, N, K, "rowmajor") == on and route(M, N, K, "rowmajor", ldy=N + 8) == off
    csrc = os.path.join(os.path.dirname(brq.LIB_PATH), "csrc")
    src, exe = tmp_path / "at.cpp", str(tmp_path / "at")
    src.write_text('''#include <stdio.h>
#include "brq_launch.h"
int main() {
    for (int at : {0, 128, 16, 32, 64, 112}) printf("%%d ", brq::gemm_route(brq::GemmShape{%d, %d, %d, false, false, true, %d, (uintptr_t)at}, 256));
}''' % (M, N, K, N))
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-isystem/opt/rocm/include", "-I" + csrc, str(src), brq.LIB_PATH, "-o", exe,
                           "-Wl,-rpath," + os.path.dirname(brq.LIB_PATH), "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined"])
    got = [brq.GEMM_ROUTES[int(r)] for r in subprocess.check_output([exe], text=True).split()]
    assert got == [on, on, off, off, off, off]
