"""Parity of every product kernel, by its name, where it can go wrong: the dispatcher sends a shape to the kernel that is
the fastest there, so tests of small and ragged shapes through it reach two or three of the twelve.  Bars as in
test_gpu_gemm.py; every kernel in every layout and both output types, with a guard right of column N - 1 and below row
M - 1.  Kernels that take the K groups in the same order must agree bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev, to_host
from test_gpu_gemm import FLOOR, RTOL, bf16_rne
from test_gpu_layout import to_tiled

pytestmark = pytest.mark.gpu

LAYOUTS = [("rowmajor", "rowmajor"), ("tiled", "tiled"), ("tiled", "rowmajor"), ("rowmajor", "tiled")]
TILE = {r: tuple(int(d) for d in r.split("x")) for r in ("256x256", "128x256", "64x128", "128x128", "192x128", "192x256", "320x128", "256x128")}


@pytest.fixture(scope="module")
def brq():
    import paper_2511_04214_amd as b
    b.lib()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return b


def check_route(brq, orc, route, M, N, K, layouts, rows=None, pads=(8, 0)):
    from paper_2511_04214_amd import inputs
    a, w = inputs.random_mxfp4(M, K, seed=M * 3 + K), inputs.random_mxfp4(N, K, seed=N * 7 + K)
    ref, bound = orc.mxfp4_gemm(*a, *w, rows=rows)
    dev = {"rowmajor": [[to_dev(t) for t in o] for o in (a, w)]}
    if any("tiled" in l for l in layouts):
        dev["tiled"] = [[to_dev(t) for t in to_tiled(*o)] for o in (a, w)]
    first = None
    for la, lw in layouts:
        for pad in pads:
            print("case", route, M, N, K, la, lw, pad, flush=True)
            out = {}
            for dt in (torch.float32, torch.bfloat16):
                buf = torch.full((M + 2, N + pad), -7.0, dtype=dt, device="cuda")
                brq.diag_mxfp4_gemm_on(route, *dev[la][0], *dev[lw][1], buf[:M, :N], K, a_layout=la, w_layout=lw)
                assert (buf[M:] == -7.0).all() and (buf[:, N:] == -7.0).all(), "wrote outside the M x N block"
                out[dt] = to_host(buf[:M, :N])
            y = out[torch.float32]
            got = (y if rows is None else y[np.asarray(rows)]).astype(np.float64)
            err = np.abs(got - ref)
            assert (err <= RTOL * bound + FLOOR).all(), "max err/bound = %g" % float((err / (bound + FLOOR)).max())
            assert np.array_equal(out[torch.bfloat16], bf16_rne(y))
            first = y if first is None else first
            assert np.array_equal(y, first), "layouts or pitches differ"
    return first


# rows and columns relative to the tile's, K.  64, 128 .. : one superstage (4 stages; rings hold 4, 5 or 6), 2, 3, 5
# of them; one row alone; one past, one short of and several tiles
SHAPES = [(1, 3, 512), (-1, -1, 1024), (0, 5, 1536), (17, 128, 2560), (1, 1, 1024)]


@pytest.mark.parametrize("route", ["64x128", "128x128", "192x128", "192x256", "320x128", "256x128"])
def test_one_tile_kernels(brq, orc, route):
    tm, tn = TILE[route]
    for dm, dn, K in SHAPES:
        check_route(brq, orc, route, tm + dm, tn + dn, K, LAYOUTS, pads=(8, 3))
    for M in (1, 16):                                        # whole wavefronts' rows past M
        check_route(brq, orc, route, M, 2 * tn - 8, 3584, LAYOUTS, pads=(8,))
    check_route(brq, orc, route, 2 * tm + 33, 9 * tn + 2, 512, LAYOUTS[:2], pads=(1,))        # more than one tile on an XCD


@pytest.mark.parametrize("route", ["64x128", "128x128", "192x128", "192x256", "320x128", "256x128"])
@pytest.mark.parametrize("K", [640, 768, 896, 1152, 2688])   # the last window overlaps by 3, 2, 1, 3 and 3 stages
def test_one_tile_kernels_k_of_128s(brq, orc, route, K):
    tm, tn = TILE[route]
    check_route(brq, orc, route, tm + 5, tn + 9, K, LAYOUTS[:2], pads=(8, 3))


@pytest.mark.parametrize("route", ["256x256", "128x256"])
def test_persistent_kernel_ragged(brq, orc, route):
    tm, tn = TILE[route]
    for M, N, K in ((tm + 1, tn + 8, 512), (tm - 1, tn - 8, 1024), (1, 8, 1536), (2 * tm + 1, 2 * tn + 8, 2560), (33, 264, 512)):
        check_route(brq, orc, route, M, N, K, LAYOUTS)
    check_route(brq, orc, route, tm + 3, tn + 24, 544, LAYOUTS[1:2])                          # zero-padded K


# More tiles than compute units: some workgroups take two, the first one's output under the second's first stage, which
# for K of one, two and three superstages is also, precedes, or is two before the workgroup's last.  Ragged last row and column.
@pytest.mark.parametrize("K", [512, 1024, 1536])
@pytest.mark.parametrize("route,M,N", [("256x256", 4100, 4104), ("128x256", 4000, 2568)])
def test_persistent_kernel_two_tiles_a_workgroup(brq, orc, route, M, N, K):
    tm, tn = TILE[route]
    assert -(-M // tm) * -(-N // tn) > 256
    rng = np.random.default_rng(47)
    rows = sorted({r for t in range(0, M, tm) for r in (t, min(t + tm, M) - 1)} | {M - 2} | set(rng.integers(0, M, 6).tolist()))
    check_route(brq, orc, route, M, N, K, LAYOUTS[:2], rows=rows)


# three register sets up to four superstages (0 or 1 turns of the main loop), five with 7 and 16 (1 and 3 turns), and 0 to 2 superstages
# after it
@pytest.mark.parametrize("nss", [1, 2, 3, 4, 7, 16])
def test_streaming_kernel(brq, orc, nss):
    for M, N in ((1, 300), (7, 77), (16, 256)):
        y = check_route(brq, orc, "stream", M, N, 512 * nss, LAYOUTS, pads=(8, 3))
        assert np.array_equal(y, check_route(brq, orc, "64x128", M, N, 512 * nss, LAYOUTS[1:2], pads=(0,)))
    check_route(brq, orc, "stream", 5, 130, 512 * nss - 96, LAYOUTS[1:2])


def test_kernels_for_any_k(brq, orc):
    for K in (32, 96, 512, 1056):
        check_route(brq, orc, "general", 70, 67, K, LAYOUTS, pads=(3,))
        check_route(brq, orc, "skinny", 13, 67, K, LAYOUTS, pads=(3,))


# 64 and 128 rows a tile; one row or column past, one short of and several tiles; 8 down to 1 groups in the last pair of stages
@pytest.mark.parametrize("M,N", [(64, 129), (17, 70), (65, 127), (129, 131), (300, 260)])
def test_any_k_kernel(brq, orc, M, N):
    for K in (256, 288, 480, 512, 576, 672, 800, 864, 928, 1056):
        y = check_route(brq, orc, "any_k", M, N, K, LAYOUTS, pads=(8, 3))
        assert np.array_equal(y, check_route(brq, orc, "general", M, N, K, LAYOUTS[:1], pads=(0,)))


def test_staged_kernels_agree_bit_for_bit(brq, orc):
    """One shape on every kernel that sums in the order of the stages."""
    M, N, K = 330, 264, 1536
    ys = [check_route(brq, orc, r, M, N, K, LAYOUTS[:2], pads=(0,)) for r in ["general", "any_k"] + sorted(TILE)]
    for y in ys[1:]:
        assert np.array_equal(y, ys[0])


def test_a_kernel_refuses_what_it_does_not_take(brq):
    q = lambda r, K: (torch.zeros((r, K // 2), dtype=torch.uint8, device="cuda"), torch.zeros((r, K // 32), dtype=torch.uint8, device="cuda"))
    for route, M, N, K in (("skinny", 17, 64, 512), ("stream", 17, 64, 512), ("stream", 4, 64, 544), ("256x256", 300, 250, 512),
                           ("128x256", 300, 256, 544), ("64x128", 64, 64, 544), ("320x128", 64, 64, 256), ("any_k", 64, 64, 224)):
        out = torch.full((M, N), -7.0, dtype=torch.float32, device="cuda")
        with pytest.raises(brq.BrqError) as e:
            brq.diag_mxfp4_gemm_on(route, *q(M, K), *q(N, K), out, K)
        assert e.value.status == 2 and (out == -7.0).all()


@pytest.mark.parametrize("layout", ["rowmajor", "tiled"])
def test_longest_k(brq, layout):
    """K = 2^26 - 512: a lane's offset into the second 64-row slab of the weights passes 2^31, the last one's 2^32 - 2^15.
    All codes 1; every row's last group has a scale of its own, and so has its first.  All sums are exact."""
    M, N, K = 17, 130, 2 ** 26 - 512
    assert brq.diag_mxfp4_gemm_route(M, N, K, layout, layout) == "64x128"
    def operand(rows):
        slabs = -(-rows // 64)
        c = torch.full((slabs * 64 * (K // 2),), 0x22, dtype=torch.uint8, device="cuda")
        s = torch.full((slabs * 64 * (K // 32),), 127, dtype=torch.uint8, device="cuda")
        e = torch.arange(slabs * 64, device="cuda", dtype=torch.int64)
        if layout == "tiled":
            v = s.view(slabs, K // 512, 64, 16)
            v[:, -1, :, 15] = (127 + e % 5).to(torch.uint8).view(slabs, 64)
            v[:, 0, :, 0] = (127 + e % 3).to(torch.uint8).view(slabs, 64)
        else:
            c, s = c.view(-1, K // 2)[:rows], s.view(-1, K // 32)[:rows]
            s[:, -1] = (127 + e % 5).to(torch.uint8)[:rows]
            s[:, 0] = (127 + e % 3).to(torch.uint8)[:rows]
        return c, s, 2.0 ** (e % 5)[:rows].double(), 2.0 ** (e % 3)[:rows].double()
    ac, as_, al, af = operand(M)
    wc, ws, wl, wf = operand(N)
    y = brq.mxfp4_gemm(ac, as_, wc, ws, a_layout=layout, w_layout=layout, M=M, N=N, K=K)
    want = K - 64 + 32 * (al[:, None] * wl[None, :] + af[:, None] * wf[None, :])
    assert torch.equal(y.double(), want)
