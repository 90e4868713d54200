// What the two LDS-staged product kernels share: the block-scaled fp4 MFMA as an instruction that stays where
// it is written, waits, and the walk from workgroup ids to output tiles.
#pragma once
#include "brq_device.h"

namespace brq {

template <int V>
struct IC { static constexpr int value = V; };

// f(IC<S>), ..., f(IC<N - 1>)
template <class F, int N, int S = 0>
__device__ __forceinline__ void static_for(F&& f, IC<N> n, IC<S> = {}) {
    if constexpr (S < N) {
        f(IC<S>{});
        static_for(f, n, IC<S + 1>{});
    }
}

// Wait until at most N of this wavefront's vector-memory operations are outstanding and all
// its LDS reads have returned, then meet the other wavefronts.
template <int N>
__device__ __forceinline__ void wait_vm_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier\n\t" ::"n"(N) : "memory");
}
// The same without a wait for global memory: the caller has already seen its loads land.
__device__ __forceinline__ void lds_wait_and_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier\n\t" ::: "memory");
}

// Elements O .. O + 7 of an accumulator, copied to vector registers by instructions that stay where they
// are written (volatile, ordered with the MFMAs).
template <int O>
__device__ __forceinline__ void read_acc8(const v16f& a, IC<O>, float (&c)[16]) {
    asm volatile("v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\tv_accvgpr_read_b32 %2, %10\n\t"
                 "v_accvgpr_read_b32 %3, %11\n\tv_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\t"
                 "v_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15"
                 : "=v"(c[O]), "=v"(c[O + 1]), "=v"(c[O + 2]), "=v"(c[O + 3]), "=v"(c[O + 4]), "=v"(c[O + 5]), "=v"(c[O + 6]), "=v"(c[O + 7])
                 : "a"(a[O]), "a"(a[O + 1]), "a"(a[O + 2]), "a"(a[O + 3]), "a"(a[O + 4]), "a"(a[O + 5]), "a"(a[O + 6]), "a"(a[O + 7]));
}

// The MFMAs are issued through volatile inline assembly: the compiler treats pure intrinsic
// calls as freely movable and sinks all of a stage's MFMAs behind its memory operations,
// which is the opposite of the interleaving these kernels live on.  Volatile asm statements
// keep their source order relative to each other and to the LDS reads.  The accumulator is
// an AGPR tuple ("a"), the fragments are 4-register VGPR tuples; SEL picks scale byte 0 / 1.
__device__ __forceinline__ void mfma_fp4(v16f& acc, const v4i& wf, const v4i& af, IC<0>, int sw, int sa) {
    asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0] cbsz:4 blgp:4"
                 : "+a"(acc) : "v"(wf), "v"(af), "v"(sw), "v"(sa));
}
__device__ __forceinline__ void mfma_fp4(v16f& acc, const v4i& wf, const v4i& af, IC<1>, int sw, int sa) {
    asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel:[1,1,0] op_sel_hi:[0,0,0] cbsz:4 blgp:4"
                 : "+a"(acc) : "v"(wf), "v"(af), "v"(sw), "v"(sa));
}
// The same with C = 0: the first MFMA of a tile on its accumulator starts the sum, so that the accumulator
// registers are never cleared by separate instructions.
__device__ __forceinline__ void mfma_fp4_init(v16f& acc, const v4i& wf, const v4i& af, int sw, int sa) {
    asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, 0, %3, %4 op_sel_hi:[0,0,0] cbsz:4 blgp:4"
                 : "+a"(acc) : "v"(wf), "v"(af), "v"(sw), "v"(sa));     // (tied like the others; the old value is not read)
}

// Tiles of one workgroup.  Workgroup ids are dealt round-robin to the 8 XCDs, each with its
// own L2: XCD x takes the contiguous id range [x*per_xcd, (x+1)*per_xcd), and ids run down 8
// tile rows before moving to the next tile column, so the tiles an XCD works on at one
// time form a patch 8 tiles high and share operand panels in its L2.
struct TileWalk {
    int first, end, stride, tiles_m, tiles_n;
    __device__ __forceinline__ void tile(int i, int& tm, int& tn) const {
        int id = first + i * stride;
        int group = id / (8 * tiles_n), rem = id - group * 8 * tiles_n;
        int rows = min(8, tiles_m - group * 8);
        tm = group * 8 + rem % rows;
        tn = rem / rows;
    }
};

// Pair order of the accumulators of a wavefront with MB A tiles (the order in which the output path takes
// them): index X -> W tile 2 * ((X / 2) / MB) + X % 2, A tile (X / 2) % MB: the two W tiles of one 128-byte
// bf16 output block are neighbours.
template <int X, int MB>
struct PairA { static constexpr int value = 2 * ((X >> 1) / MB) + (X & 1); };
template <int X, int MB>
struct PairB { static constexpr int value = (X >> 1) % MB; };

}  // namespace brq
