// Device-side building blocks shared by the gfx950 kernels of the block-rotation MXFP4
// path: bf16 widening, wavefront lane exchange, the E8M0 scale rule and the packed E2M1
// encoder.  CDNA4 only (64-wide wavefronts, DPP, the scaled fp4 convert instruction).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace brq {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }

// A dword holds two bf16 values; bf16 is the upper half of an fp32, so widening is a
// shift (low element) or a mask (high element), both exact.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return as_f32(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return as_f32(w & 0xffff0000u); }

// fp32 -> bf16 bits, round to nearest even (finite input), integer form.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = as_u32(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// Two fp32 -> one dword of two bf16 (lo in the low half), round to nearest even:
// v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Value of `v` held by the neighbouring lane (lane ^ 1); folds into the consuming VALU instruction as a DPP modifier.
__device__ __forceinline__ float lane_xor1(float v) {
    int iv = __builtin_bit_cast(int, v);
    iv = __builtin_amdgcn_update_dpp(iv, iv, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, true);
    return __builtin_bit_cast(float, iv);
}

// Radix-8 butterfly on 8 consecutive elements held by one lane: stages h = 1, 2, 4 of
// the ascending-order Walsh-Hadamard transform, pair (i, i+h) -> (a+b, a-b).
__device__ __forceinline__ void wht8(float (&v)[8]) {
#pragma unroll
    for (int h = 1; h < 8; h *= 2) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if ((i & h) == 0) {
                float a = v[i], b = v[i + h];
                v[i] = a + b;
                v[i + h] = a - b;
            }
        }
    }
}

// Cross-lane stages.  The lane whose bit is clear owns a and needs a+b; the other owns b and needs a-b.  Both evaluate
// fma(partner, s, own) with s = +1 / -1: the lower lane gets a+b, the upper lane gets
// b-a, i.e. the NEGATED result (one rounding, so exactly -fl(a-b)).  The caller tracks
// the sign (it flips once per stage in which the lane is the upper one) and folds it into
// the final normalisation multiply; only the sign of exact zeros can differ, and the
// encoder stores every zero magnitude as code 0.
// This one: partner lane ^ 1 alone (B = 16).
__device__ __forceinline__ void wht_cross1(float (&v)[8], float s) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = __builtin_fmaf(lane_xor1(v[i]), s, v[i]);
}

// The two stages that stay inside a quad (partner lane ^ 1, then lane ^ 2), i.e. h = 8 and
// h = 16 at 8 elements per lane.  The compiler folds a DPP lane permute into v_add/v_sub
// but not into v_fmac, so the 16 fused multiply-adds are written out: v_fmac_f32_dpp
// computes D = dpp(S0) * S1 + D.  A VGPR written by a VALU instruction may be read through
// DPP only 2 wait states later: the leading s_nop covers the compiler's code in front, and
// inside the block 7 instructions separate every write from its DPP read.
#define BRQ_FMAC_DPP(r, s, perm) \
    "v_fmac_f32_dpp " r ", " r ", " s " quad_perm:" perm " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
__device__ __forceinline__ void wht_cross_quad(float (&v)[8], float s1, float s2) {
    asm volatile(
        "s_nop 1\n\t"
        BRQ_FMAC_DPP("%0", "%8", "[1,0,3,2]") BRQ_FMAC_DPP("%1", "%8", "[1,0,3,2]")
        BRQ_FMAC_DPP("%2", "%8", "[1,0,3,2]") BRQ_FMAC_DPP("%3", "%8", "[1,0,3,2]")
        BRQ_FMAC_DPP("%4", "%8", "[1,0,3,2]") BRQ_FMAC_DPP("%5", "%8", "[1,0,3,2]")
        BRQ_FMAC_DPP("%6", "%8", "[1,0,3,2]") BRQ_FMAC_DPP("%7", "%8", "[1,0,3,2]")
        BRQ_FMAC_DPP("%0", "%9", "[2,3,0,1]") BRQ_FMAC_DPP("%1", "%9", "[2,3,0,1]")
        BRQ_FMAC_DPP("%2", "%9", "[2,3,0,1]") BRQ_FMAC_DPP("%3", "%9", "[2,3,0,1]")
        BRQ_FMAC_DPP("%4", "%9", "[2,3,0,1]") BRQ_FMAC_DPP("%5", "%9", "[2,3,0,1]")
        BRQ_FMAC_DPP("%6", "%9", "[2,3,0,1]") BRQ_FMAC_DPP("%7", "%9", "[2,3,0,1]")
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])
        : "v"(s1), "v"(s2));
}
#undef BRQ_FMAC_DPP

// Blocks wider than a quad.  No DPP modifier reaches lane ^ 4 or lane ^ 8, but two reach the mirror image: lane ^ 7
// inside 8 lanes and lane ^ 15 inside 16.  So the chunks are dealt to the lanes in an order in which the mirror image
// IS the partner: lane L of a 16-lane row holds chunk M(L), M linear over the bits with M(1) = 1, M(2) = 2,
// M(7) = 4, M(15) = 8.  Quads still hold whole 32-element groups (in reverse order where bit 2 of the lane is
// set), 16 lanes still read 256 contiguous bytes, and the stages h = 32 and 64 cost one instruction per value
// like those inside a quad (through the LDS swizzle they cost that, an LDS operation and its latency).
__device__ __forceinline__ uint32_t chunk_of_lane(uint32_t lane) {
    return lane ^ ((lane & 4u) ? 3u : 0u) ^ ((lane & 8u) ? 4u : 0u);
}
#define BRQ_FMAC_MIRROR(r, how) "v_fmac_f32_dpp " r ", " r ", %8 " how " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define BRQ_CROSS_MIRROR(v, s, how)                                                                                \
    asm volatile("s_nop 1\n\t" BRQ_FMAC_MIRROR("%0", how) BRQ_FMAC_MIRROR("%1", how) BRQ_FMAC_MIRROR("%2", how)     \
                 BRQ_FMAC_MIRROR("%3", how) BRQ_FMAC_MIRROR("%4", how) BRQ_FMAC_MIRROR("%5", how)                  \
                 BRQ_FMAC_MIRROR("%6", how) BRQ_FMAC_MIRROR("%7", how)                                             \
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])    \
                 : "v"(s))
__device__ __forceinline__ void wht_cross_mirror8(float (&v)[8], float s) { BRQ_CROSS_MIRROR(v, s, "row_half_mirror"); }
__device__ __forceinline__ void wht_cross_mirror16(float (&v)[8], float s) { BRQ_CROSS_MIRROR(v, s, "row_mirror"); }
#undef BRQ_CROSS_MIRROR
#undef BRQ_FMAC_MIRROR

// The stages between 16-lane rows (h = 128) and between the halves of the wavefront (h = 256): two registers trade
// the part the stage pairs, the butterfly is then between the two registers of one lane, and trading again puts the
// values back: four instructions per two values and stage, no LDS, true signs.
template <bool HALVES>
__device__ __forceinline__ void trade(float& x, float& y) {
    if constexpr (HALVES) {
        const auto s = __builtin_amdgcn_permlane32_swap(as_u32(x), as_u32(y), false, false);
        x = as_f32(s[0]);
        y = as_f32(s[1]);
    } else {
        const auto s = __builtin_amdgcn_permlane16_swap(as_u32(x), as_u32(y), false, false);
        x = as_f32(s[0]);
        y = as_f32(s[1]);
    }
}
template <bool HALVES>
__device__ __forceinline__ void wht_cross_rows(float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        trade<HALVES>(v[i], v[i + 1]);
        const float a = v[i], b = v[i + 1];
        v[i] = a + b;
        v[i + 1] = a - b;
        trade<HALVES>(v[i], v[i + 1]);
    }
}

// A lane's chunk of 8 consecutive elements, read once with the streaming hint (16 bytes of bf16, 32 of fp32), as it
// comes from memory and as fp32 values.
template <bool BF16>
struct RawChunk { v4f a, b; };
template <>
struct RawChunk<true> { v4i w; };
template <bool BF16>
__device__ __forceinline__ RawChunk<BF16> load_raw(const void* p) {
    RawChunk<BF16> c;
    if constexpr (BF16) {
        c.w = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
    } else {
        c.a = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
        c.b = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p) + 1);
    }
    return c;
}
template <bool BF16>
__device__ __forceinline__ void widen(const RawChunk<BF16>& c, float (&v)[8]) {
    if constexpr (BF16) {
        const v4i w = c.w;
        v[0] = bf16_lo((uint32_t)w.x); v[1] = bf16_hi((uint32_t)w.x); v[2] = bf16_lo((uint32_t)w.y); v[3] = bf16_hi((uint32_t)w.y);
        v[4] = bf16_lo((uint32_t)w.z); v[5] = bf16_hi((uint32_t)w.z); v[6] = bf16_lo((uint32_t)w.w); v[7] = bf16_hi((uint32_t)w.w);
    } else {
        v[0] = c.a.x; v[1] = c.a.y; v[2] = c.a.z; v[3] = c.a.w; v[4] = c.b.x; v[5] = c.b.y; v[6] = c.b.z; v[7] = c.b.w;
    }
}
template <bool BF16>
__device__ __forceinline__ void load_chunk(const void* p, float (&v)[8]) {
    widen<BF16>(load_raw<BF16>(p), v);
}

// The random sign diagonal of a randomized Hadamard rotation, applied on load: `signs` points at the 8 sign
// bytes of this chunk (8-byte aligned); element i is negated where its byte is negative.
__device__ __forceinline__ void apply_signs(float (&v)[8], const int8_t* signs) {
    const uint2 sg = *reinterpret_cast<const uint2*>(signs);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t word = (i < 4) ? sg.x : sg.y;
        v[i] = as_f32(as_u32(v[i]) ^ ((word << (24 - 8 * (i & 3))) & 0x80000000u));
    }
}

// Stages of the order-2^LOG2B transform (at most a wavefront's 512 elements) for the chunk in `v`.  `chunk`: which
// chunk of the wavefront the lane holds: the lane's own number up to B = 32, chunk_of_lane beyond.  The DPP stages
// track signs: afterwards v holds wht_sign<LOG2B>(chunk) * (x H).
constexpr bool wht_mirrored(int log2b) { return log2b >= 6; }
template <int LOG2B>
__device__ __forceinline__ float wht_sign(uint32_t chunk) {
    constexpr uint32_t bits = LOG2B < 3 ? 0u : LOG2B >= 7 ? 15u : (1u << (LOG2B - 3)) - 1u;
    return (__builtin_popcount(chunk & bits) & 1) ? -1.0f : 1.0f;
}
template <int LOG2B>
__device__ __forceinline__ void wht_inwave(float (&v)[8], uint32_t chunk) {
    static_assert(LOG2B >= 3 && LOG2B <= 9, "a lane holds 8 elements, a wavefront 512");
    wht8(v);
    if constexpr (LOG2B == 4) wht_cross1(v, (chunk & 1) ? -1.0f : 1.0f);
    if constexpr (LOG2B >= 5) wht_cross_quad(v, (chunk & 1) ? -1.0f : 1.0f, (chunk & 2) ? -1.0f : 1.0f);
    if constexpr (LOG2B >= 6) wht_cross_mirror8(v, (chunk & 4) ? -1.0f : 1.0f);
    if constexpr (LOG2B >= 7) wht_cross_mirror16(v, (chunk & 8) ? -1.0f : 1.0f);
    if constexpr (LOG2B >= 8) wht_cross_rows<false>(v);
    if constexpr (LOG2B >= 9) wht_cross_rows<true>(v);
}

// silu(g) * u = g / (1 + exp(-g)) * u, the gated activation that produces the input of the rotated
// layer (Sec. 4.3: the online rotation sits in front of down_proj).  The paper fixes no arithmetic
// for it, so the kernel takes the cheapest one that stays within a stated bound of the definition:
// exp(-g) = 2^(g * -log2(e)) on v_exp_f32, the reciprocal of 1 + exp(-g) on v_rcp_f32 (1 ulp each),
// three multiplies and one add, each rounded once.  Error against the exact value:
//   z = g * -log2(e) carries half an ulp of its own size plus the rounding of log2(e), which the
//   exponential turns into 1.5 |g| 2^-24 relative; exp and rcp 2^-23 each; 1 + e, g * y and s * u
//   2^-24 each: together below (8 + 2 |g|) 2^-24 relative (brq.h states that bound, the tests
//   measure it).  Far below zero (g < -87) 1 + exp(-g) leaves the range whose reciprocal is a
//   normal number and the result may be flushed to zero: an absolute error below 2^-119 |u|.
// With this the SwiGLU-fused step costs 6 instructions per element for the activation instead of
// 22 for a correctly rounded sequence, and is bound by HBM like the plain step.
__device__ __forceinline__ float swiglu_f32(float g, float u) {
    const float z = g * -as_f32(0x3FB8AA3Bu);
    const float e = __builtin_amdgcn_exp2f(z);
    const float d = 1.0f + e;
    const float y = __builtin_amdgcn_rcpf(d);
    const float s = g * y;
    return s * u;
}

// The lane's 8 gate values in v become h = swiglu(v, w); with `to_bf16` (uniform) h passes
// through bf16 (round to nearest even) as if a separate activation kernel had stored it.
__device__ __forceinline__ void swiglu8(float (&v)[8], const float (&w)[8], bool to_bf16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = swiglu_f32(v[i], w[i]);
    if (to_bf16) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            const uint32_t pk = pack_bf16x2(v[i], v[i + 1]);
            v[i] = bf16_lo(pk);
            v[i + 1] = bf16_hi(pk);
        }
    }
}

// Maximum magnitude of the lane's 8 values.
__device__ __forceinline__ float absmax8(const float (&y)[8]) {
    float m = fmaxf(fmaxf(fabsf(y[0]), fabsf(y[1])), fabsf(y[2]));
    m = fmaxf(fmaxf(m, fabsf(y[3])), fabsf(y[4]));
    m = fmaxf(fmaxf(m, fabsf(y[5])), fabsf(y[6]));
    return fmaxf(m, fabsf(y[7]));
}

// Maximum over the 4 lanes of a quad (= one 32-element MXFP4 group at 8 per lane).  The
// argument is non-negative, so comparing the bit patterns as unsigned integers orders
// them like the floats.  Same DPP read-after-write spacing rule as above.
__device__ __forceinline__ float quad_max(float m) {
    uint32_t u = as_u32(m);
    asm volatile(
        "s_nop 1\n\t"
        "v_max_u32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_max_u32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+v"(u));
    return as_f32(u);
}

// Sum over the 4 lanes of a quad, every lane receiving it: two adds with the lane permute folded in
// (((v0 + v1) + (v2 + v3)) in lanes 0, 1 and the mirror image in lanes 2, 3: the same value, since fp32
// addition is commutative).  Same DPP read-after-write spacing rule as above.
__device__ __forceinline__ float quad_sum(float v) {
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+v"(v));
    return v;
}

// cnt += how many of the wavefront's values v are above lim, by magnitude (MAG) or as they are: the comparison writes
// a lane mask to scalar registers and the scalar unit counts its bits.  Written out, and volatile, because the
// compiler takes a comparison for something to be done early wherever its result is only used under a condition:
// with eight limits of which a caller uses two it made all the masks for every value, and moved them through vector
// registers one lane at a time for want of scalar ones.
template <bool MAG>
__device__ __forceinline__ void count_above(uint32_t& cnt, float v, float lim) {
    uint64_t m;
    uint32_t n;
    if constexpr (MAG)
        asm volatile("v_cmp_gt_f32_e64 %1, |%3|, %4\n\ts_bcnt1_i32_b64 %2, %1\n\ts_add_u32 %0, %0, %2"
                     : "+s"(cnt), "=&s"(m), "=&s"(n) : "v"(v), "v"(lim) : "scc");
    else
        asm volatile("v_cmp_gt_f32_e64 %1, %3, %4\n\ts_bcnt1_i32_b64 %2, %1\n\ts_add_u32 %0, %0, %2"
                     : "+s"(cnt), "=&s"(m), "=&s"(n) : "v"(v), "v"(lim) : "scc");
}
// The same for 8 values of a lane, two chains of comparison and count interleaved.
__device__ __forceinline__ void count_above8(uint32_t& cnt, const float (&y)[8], float lim) {
    uint64_t m0, m1, m2, m3;
    uint32_t n;
#pragma unroll
    for (int i = 0; i < 8; i += 4)
        asm volatile("v_cmp_gt_f32_e64 %1, |%6|, %10\n\tv_cmp_gt_f32_e64 %2, |%7|, %10\n\t"
                     "v_cmp_gt_f32_e64 %3, |%8|, %10\n\tv_cmp_gt_f32_e64 %4, |%9|, %10\n\t"
                     "s_bcnt1_i32_b64 %5, %1\n\ts_add_u32 %0, %0, %5\n\ts_bcnt1_i32_b64 %5, %2\n\ts_add_u32 %0, %0, %5\n\t"
                     "s_bcnt1_i32_b64 %5, %3\n\ts_add_u32 %0, %0, %5\n\ts_bcnt1_i32_b64 %5, %4\n\ts_add_u32 %0, %0, %5"
                     : "+s"(cnt), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3), "=&s"(n)
                     : "v"(y[i]), "v"(y[i + 1]), "v"(y[i + 2]), "v"(y[i + 3]), "v"(lim) : "scc");
}

// E8M0 byte of a group from its maximum magnitude: max(exponent field - 2, 0).
// (2 = exponent of the largest E2M1 value, 6 = 1.5 * 2^2.)
__device__ __forceinline__ uint32_t e8m0_from_amax(float amax) {
    uint32_t e = (as_u32(amax) >> 23) & 0xffu;
    return __builtin_elementwise_sub_sat(e, 2u);
}

// 8 fp32 values -> 8 packed E2M1 codes (element i in nibble i) under E8M0 byte `sb`.
// v_cvt_scalef32_pk_fp4_f32 divides by 2^(sb-127) (it reads only the exponent field of
// its scale operand, field 0 meaning 2^-127), rounds to nearest with ties to the even
// code and saturates at 6.  It keeps the sign of results that round to zero; those
// nibbles are cleared afterwards so that a zero magnitude is always code 0.
// encode8_e2m1_signed_zero is the instruction's own result (a zero magnitude may carry a sign bit): enough
// where the codes are only decoded again.
__device__ __forceinline__ uint32_t encode8_e2m1_signed_zero(const float (&y)[8], uint32_t sb) {
    float scale = as_f32(sb << 23);
    uint32_t w = 0;
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[0], y[1], scale, 0);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[2], y[3], scale, 1);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[4], y[5], scale, 2);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[6], y[7], scale, 3);
    return w;
}
__device__ __forceinline__ uint32_t encode8_e2m1(const float (&y)[8], uint32_t sb) {
    const uint32_t w = encode8_e2m1_signed_zero(y, sb);
    uint32_t mag = w & 0x77777777u;
    uint32_t nz = mag + 0x77777777u;            // bit 3 of a nibble set <=> magnitude != 0
    return w & (nz | 0x77777777u);
}

// ---- the tiled operand layout

// Byte offsets of chunk kc (8 elements = 4 code bytes) of row `row` in the tiled layout.
__device__ __forceinline__ uint64_t tiled_code_offset(uint32_t row, uint32_t kc, uint32_t stages) {
    return ((uint64_t)(row >> 6) * stages + (kc >> 4)) * 4096u + (row & 63u) * 64u + (kc & 15u) * 4u;
}
__device__ __forceinline__ uint64_t tiled_scale_offset(uint32_t row, uint32_t kc, uint32_t sstages) {
    return ((uint64_t)(row >> 6) * sstages + (kc >> 6)) * 1024u + (row & 63u) * 16u + ((kc >> 2) & 15u);
}

// Tiled layout, K not a multiple of 512: the groups between K and the next multiple of 512 are written as zeros (16
// zero code bytes, scale byte 0) for every row, so that the LDS-staged product kernels can run whole 512-element
// superstages over tiled operands of any K.  Every quantizing kernel does it itself, spread over all of its
// threads (rotations of B >= 512 have nothing to pad, B dividing K): as a launch of its own it cost 2 to 4 us in front
// of a kernel of 10.
struct KPad {
    uint8_t *codes, *scales;
    uint32_t rows, g0, n, stages, sstages;     // n groups per row from group g0 on; 0: nothing to do
    static KPad of(bool tiled, uint8_t* codes, uint8_t* scales, int64_t M, int64_t K) {
        const int64_t Kp = (K + 511) / 512 * 512;
        return KPad{codes, scales, (uint32_t)M, (uint32_t)(K / 32), tiled ? (uint32_t)((Kp - K) / 32) : 0u,
                    (uint32_t)(Kp / 128), (uint32_t)(Kp / 512)};
    }
    __device__ __forceinline__ void zero(uint32_t thread, uint32_t threads) const {
        if (n == 0) return;     // uniform
        for (uint64_t i = thread; i < (uint64_t)rows * n; i += threads) {
            const uint32_t row = (uint32_t)(i / n), g = g0 + (uint32_t)(i - (uint64_t)row * n);
            *reinterpret_cast<v4i*>(codes + tiled_code_offset(row, g * 4, stages)) = v4i{0, 0, 0, 0};
            scales[tiled_scale_offset(row, g * 4, sstages)] = 0;
        }
    }
};

// ---- LDS-DMA loads (global memory -> LDS without passing through VGPRs)

// One LDS-DMA load: 64 lanes x 16 bytes from base + voff(lane) to LDS lds_base + LDS_OFF +
// 16 * lane (M0 carries the LDS address).  lds_base and base must be wavefront-uniform.
// Between a write of M0 and the load that takes its LDS address from it the hardware wants one wait state and does not
// check (the compiler puts an s_nop 0 there, and sees none of this).
template <int LDS_OFF>
__device__ __forceinline__ void dma16(uint32_t lds_base, const uint8_t* base, uint32_t voff) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\t"
                 :: "s"(lds_base), "v"(voff), "s"(base), "n"(LDS_OFF)
                 : "memory", "scc", "m0");
}

// The same for the lanes of `mask` only (uniform); every lane of the wavefront is active around it.  (The write of the
// lane mask is the wait state.)
template <int LDS_OFF>
__device__ __forceinline__ void dma16_masked(uint32_t lds_base, const uint8_t* base, uint32_t voff, uint64_t mask) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_mov_b64 exec, %4\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1\n\t"
                 :: "s"(lds_base), "v"(voff), "s"(base), "n"(LDS_OFF), "s"(mask)
                 : "memory", "scc", "m0");
}

// dma16 with the non-temporal hint, for data that is read once.
template <int LDS_OFF>
__device__ __forceinline__ void dma16_stream(uint32_t lds_base, const uint8_t* base, uint32_t voff) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\t"
                 :: "s"(lds_base), "v"(voff), "s"(base), "n"(LDS_OFF)
                 : "memory", "scc", "m0");
}

// Kernel arguments, all asked for here: left to the compiler each is loaded where it is first used, and the first global load
// waits for three or four of these one after the other, 0.1 us each.  us, before -> now: k_gemm_smallm 28672 x 2048 tiled 8.9 -> 8.6;
// one-tile product 1000 x 4096 x 1024 6.57 -> 6.41, 200 x 4096 x 4096 8.98 -> 8.81; k_rowwise_reg 4096 x 8192, B = 8192 25.9 -> 25.15.
// Nothing in k_rowwise and k_rowwise_t4, where other workgroups fill the time; the one-launch decode call is slower with it,
// its x loads then wait for the arguments of its product too (9.7 -> 10.0).
template <class... T>
__device__ __forceinline__ void load_args(T... a) { ([](auto v) __attribute__((always_inline)) { asm volatile("" :: "s"(v)); }(a), ...); }

// A pointer that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ const uint8_t* uniform_ptr(const uint8_t* p) {
    uint64_t b = (uint64_t)p;
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return (const uint8_t*)(((uint64_t)hi << 32) | lo);
}

}  // namespace brq
