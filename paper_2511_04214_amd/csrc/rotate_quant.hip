// Row-wise kernels of the block-rotation MXFP4 path for gfx950: block Hadamard rotation
// (Sec. 4.3, Eq. 1), MXFP4 quantization (Sec. 4.1) and their fusion, the online step
// that precedes a quantized linear layer.  All of them stream X once from HBM.
//
// Work decomposition.  A "chunk" is 8 consecutive elements of a row (16 bytes of bf16,
// 32 bytes of fp32), held by one lane; 4 consecutive lanes (a DPP quad) hold one
// 32-element MXFP4 group, so the group maximum is two quad-permute steps and the group's
// 8 packed codes per lane form one dword store.  Rotation stages h = 1, 2, 4 run inside
// the lane, h = 8 ... 256 between lanes of the wavefront, larger h between the chunks a lane holds (bf16 values, B <= 8192:
// one or two wavefronts hold the whole block) or through LDS (fp32 values, and B = 16384).
#include "brq_device.h"
#include "brq_launch.h"

namespace brq {

enum RowMode { MODE_ROTATE = 0, MODE_QUANT = 1, MODE_FUSED = 2, MODE_STATS = 3 };

struct RowArgs {
    const void* x;      // [M][ldx]
    void* y;            // rotate: [M][ldy]
    uint32_t* codes;    // quant/fused: [M][K/8] dwords
    uint8_t* scales;    // quant/fused: [M][K/32]
    int64_t ldx, ldy;   // in elements
    uint32_t cpr;       // chunks per row = K/8
    uint32_t through;   // how codes are stored: store_codes
    uint32_t nchunks;   // M * K/8
    // Tiled output (codes: 64 rows x 64 bytes per (slab, stage) block; scales: 64 rows x 16
    // bytes per (slab, superstage) block): blocks per slab, 0 = row-major output.
    uint32_t stages;    // Kp/128, Kp = K rounded up to a multiple of 512
    uint32_t sstages;   // Kp/512
    const int8_t* signs;   // [K] or null: element k is negated on load where signs[k] < 0
    const void* x2;        // producer kernels: the `up` matrix [M][ldx2] (x is then `gate`)
    int64_t ldx2;
    uint32_t hround;       // producer kernels: the activation passes through bf16
    uint32_t sign_fixed;   // the grid was sized so that a lane's column is the same in every pass
    uint32_t rows, nitems; // k_rowwise_t4 (next to the words it needs first: one scalar load)
    // MODE_STATS outputs (any may be null) and thresholds
    float* amax;                   // [M][K/32]
    float* sqerr;                  // [M][K/32]
    float* sqerr_bfp4;             // [M][K/32]
    unsigned long long* counts;    // [nt], added to
    uint32_t nt;
    float th[8];
    KPad pad;              // tiled output: the groups between K and the next multiple of 512
};

// The random sign diagonal of a randomized Hadamard rotation (Sec. 5.1 and the Appendix use
// "randomized"/"stochastic" Hadamard matrices): x_k -> s_k x_k before the butterfly, an exact
// flip of the fp32 sign bit.  `signs` points at the 8 sign bytes of this chunk (8-byte aligned).
// The same flip as 8 ready-made sign-bit masks: kernels whose lanes keep their column from one
// grid-stride pass to the next (the host sizes the grid for that: sign_fixed) expand the sign
// bytes once, and a chunk then costs 8 XORs.
__device__ __forceinline__ void sign_masks(uint32_t (&m)[8], const int8_t* signs) {
    const uint2 sg = *reinterpret_cast<const uint2*>(signs);
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = (((i < 4) ? sg.x : sg.y) << (24 - 8 * (i & 3))) & 0x80000000u;
}
__device__ __forceinline__ void flip(float (&v)[8], const uint32_t (&m)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = as_f32(as_u32(v[i]) ^ m[i]);
}
// ---- chunk load / store ---------------------------------------------------------

// X is read exactly once and the outputs are next touched by another kernel: loads and the
// stores of rotated values and codes carry the non-temporal hint, so the stream does not
// displace what the caches hold (on a 16 B in / 4 B out stream this alone is worth about 10% of
// HBM throughput).  The scale bytes are stored plainly: a cache line of scales is completed by
// several wavefronts, and the L2 merges their pieces before the line goes to memory.
template <bool BF16>
__device__ __forceinline__ void store_chunk(void* p, const float (&v)[8]) {
    if constexpr (BF16) {
        v4i w;
        w.x = (int)(f32_to_bf16_bits(v[0]) | (f32_to_bf16_bits(v[1]) << 16));
        w.y = (int)(f32_to_bf16_bits(v[2]) | (f32_to_bf16_bits(v[3]) << 16));
        w.z = (int)(f32_to_bf16_bits(v[4]) | (f32_to_bf16_bits(v[5]) << 16));
        w.w = (int)(f32_to_bf16_bits(v[6]) | (f32_to_bf16_bits(v[7]) << 16));
        __builtin_nontemporal_store(w, reinterpret_cast<v4i*>(p));
    } else {
        __builtin_nontemporal_store(v4f{v[0], v[1], v[2], v[3]}, reinterpret_cast<v4f*>(p));
        __builtin_nontemporal_store(v4f{v[4], v[5], v[6], v[7]}, reinterpret_cast<v4f*>(p) + 1);
    }
}

// fp32 output of the rotation: a lane's 8 values are 32 contiguous bytes, and two 16-byte stores per
// lane would leave the lanes of either instruction 32 bytes apart - the store path then takes them
// one lane at a time (178 us on X 16384 x 8192, where a plain conversion copy of the same traffic takes
// 137).  The four lanes of a quad hold 128 contiguous bytes (consecutive lanes = consecutive chunks of
// one row): the 16-byte pieces are traded inside the quad so that store A writes pieces 0..3 and store
// B pieces 4..7, chunk t's lane piece t - 64 contiguous bytes per quad and instruction.  Piece k sits in chunk
// k >> 1, half k & 1.  A quad that holds its chunks in reverse order (chunk_of_lane) finds the pieces of store B where
// the others find those of store A.  Every lane of the quad must be active.
__device__ __forceinline__ void store_chunk_f32_quad(char* p, const float (&v)[8], uint32_t lane, uint32_t chunk) {
    const uint32_t t = chunk & 3u;
    const bool odd = (t & 1u) != 0;
    const int first = ((lane ^ chunk) & 3u) != 0 ? 64 : 0;     // 0 or 3: in order or reversed
    v4f a, b;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int lo = __builtin_bit_cast(int, v[k]), hi = __builtin_bit_cast(int, v[4 + k]);
        const int a_lo = __builtin_amdgcn_update_dpp(lo, lo, 0x50 /* quad_perm [0,0,1,1] */, 0xF, 0xF, true);
        const int a_hi = __builtin_amdgcn_update_dpp(hi, hi, 0x50, 0xF, 0xF, true);
        const int b_lo = __builtin_amdgcn_update_dpp(lo, lo, 0xFA /* quad_perm [2,2,3,3] */, 0xF, 0xF, true);
        const int b_hi = __builtin_amdgcn_update_dpp(hi, hi, 0xFA, 0xF, 0xF, true);
        a[k] = __builtin_bit_cast(float, odd ? a_hi : a_lo);
        b[k] = __builtin_bit_cast(float, odd ? b_hi : b_lo);
    }
    __builtin_nontemporal_store(a, reinterpret_cast<v4f*>(p + first - 16 * (int)t));
    __builtin_nontemporal_store(b, reinterpret_cast<v4f*>(p + (64 - first) - 16 * (int)t));
}

// The lane's 8 input values: the chunk at p, or (PROD) the gated activation of the chunks at p
// (gate) and p2 (up), computed here so that it never visits HBM.
template <bool BF16, bool PROD>
__device__ __forceinline__ void load_input(const void* p, const void* p2, bool hround, float (&v)[8]) {
    if constexpr (!PROD) {
        load_chunk<BF16>(p, v);
    } else if constexpr (BF16) {
        // both loads first, then the arithmetic
        const v4i a = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
        const v4i b = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p2));
        float w[8];
        v[0] = bf16_lo((uint32_t)a.x); v[1] = bf16_hi((uint32_t)a.x); v[2] = bf16_lo((uint32_t)a.y); v[3] = bf16_hi((uint32_t)a.y);
        v[4] = bf16_lo((uint32_t)a.z); v[5] = bf16_hi((uint32_t)a.z); v[6] = bf16_lo((uint32_t)a.w); v[7] = bf16_hi((uint32_t)a.w);
        w[0] = bf16_lo((uint32_t)b.x); w[1] = bf16_hi((uint32_t)b.x); w[2] = bf16_lo((uint32_t)b.y); w[3] = bf16_hi((uint32_t)b.y);
        w[4] = bf16_lo((uint32_t)b.z); w[5] = bf16_hi((uint32_t)b.z); w[6] = bf16_lo((uint32_t)b.w); w[7] = bf16_hi((uint32_t)b.w);
        swiglu8(v, w, hround);
    } else {
        const v4f a0 = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
        const v4f a1 = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p) + 1);
        const v4f b0 = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p2));
        const v4f b1 = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p2) + 1);
        const float w[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
        v[0] = a0.x; v[1] = a0.y; v[2] = a0.z; v[3] = a0.w; v[4] = a1.x; v[5] = a1.y; v[6] = a1.z; v[7] = a1.w;
        swiglu8(v, w, hround);
    }
}

// Element offset of chunk c.  Contiguous rows (ld == K) need no division.
template <bool CONTIG>
__device__ __forceinline__ int64_t chunk_offset(uint32_t c, uint32_t cpr, int64_t ld) {
    if constexpr (CONTIG) {
        return (int64_t)c * 8;
    } else {
        uint32_t row = c / cpr;
        return (int64_t)row * ld + (int64_t)(c - row * cpr) * 8;
    }
}

// A lane's 8 codes.  They are read next by another kernel, on all XCDs.  With the streaming hint they go to memory and the
// product fetches them from there; stored through the L2 (a store at device scope, `through`, uniform) they are also in the
// memory-side cache.  What the two give is in code_stores_through.
__device__ __forceinline__ void store_codes(uint32_t* p, uint32_t w, uint32_t through) {
    if (through) __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else __builtin_nontemporal_store(w, p);
}

// ---- in-wavefront rotation, 32 <= B <= 512 ------------------------------------------

// fl(1/sqrt(2^LOG2B)) as fp32 bits: sqrt(2)/2 = 0x3F3504F3 scaled by a power of two.
__host__ __device__ constexpr uint32_t norm_bits(int log2b) {
    return (log2b & 1) ? (0x3F3504F3u - ((uint32_t)((log2b - 1) / 2) << 23))
                       : (0x3F800000u - ((uint32_t)(log2b / 2) << 23));
}

// Quantize the lane's 8 values (quad = one group) and store codes + scale.
// Chunk kc of row `row`.
__device__ __forceinline__ void quant_store(const float (&y)[8], uint32_t row, uint32_t kc, uint32_t lane,
                                            const RowArgs& a) {
    uint32_t sb = e8m0_from_amax(quad_max(absmax8(y)));
    uint32_t w = encode8_e2m1(y, sb);
    if (a.stages == 0) {
        uint32_t c = row * a.cpr + kc;
        store_codes(&a.codes[c], w, a.through);
        if ((lane & 3) == 0) *(&a.scales[c >> 2]) = (uint8_t)sb;
    } else {
        store_codes(reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(a.codes) + tiled_code_offset(row, kc, a.stages)), w, a.through);
        if ((lane & 3) == 0) *(a.scales + tiled_scale_offset(row, kc, a.sstages)) = (uint8_t)sb;
    }
}

// ---- block statistics (Sec. 4.1, 4.2, Appendix "Rotation Comparison") ----------------------
// For the lane's 8 (rotated) values, quad = one 32-element block: the block-wise scale max|y|, the
// block's MXFP4 quantization loss sum (y - deq(q(y)))^2 (fp32; each difference is exact, the
// squares and the 32-term sum round), and per threshold the number of values with |y| above it.
//
// Counting costs one vector instruction per value and threshold (count_above8): the comparison writes a lane mask
// to scalar registers, and the scalar unit, which has nothing else to do in this kernel, counts its bits
// and keeps the wavefront's running sums (`cnt`, wavefront-uniform; a wavefront meets fewer than 2^32
// values per launch).  Per-lane counters cost a second vector instruction per value and threshold on a
// kernel whose vector units are the busiest part.
//
// The per-block outputs of a wavefront's 16 blocks sit in lanes 0, 4, 8, ...; stored from there they are
// 16 separate 4-byte accesses.  One lane permute brings them to lanes 0..15, which store 64 contiguous
// bytes.  gidx0 = block index of the wavefront's first chunk; `live` = this lane's chunk exists.
// (MIRRORED: block b sits in quad b ^ (bit 1 of b), chunk_of_lane's order.)
template <bool MIRRORED>
__device__ __forceinline__ float gather_quads(float v, uint32_t lane) {
    const uint32_t quad = MIRRORED ? lane ^ ((lane >> 1) & 1u) : lane;
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((int)((quad & 15u) << 4), __builtin_bit_cast(int, v)));
}
template <bool MIRRORED>
__device__ __forceinline__ void stats_chunk(const float (&y)[8], uint32_t gidx0, bool live, uint32_t lane,
                                            const RowArgs& a, uint32_t (&cnt)[8]) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const float am = quad_max(absmax8(y));
    const uint32_t sb = e8m0_from_amax(am);
    const uint32_t w = encode8_e2m1_signed_zero(y, sb);      // decoded again below: the sign of a zero does not matter
    const float sc = as_f32(sb ? sb << 23 : 0x00400000u);   // 2^(sb - 127); scale byte 0 is the subnormal 2^-127
    float e2 = 0.0f;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        f2 d;   // the two codes of byte p as fp32 (scale 1); value * 2^(sb - 127) is exact, and so is y - that
        if (p == 0) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 0);
        if (p == 1) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 1);
        if (p == 2) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 2);
        if (p == 3) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 3);
        const float e0 = __builtin_fmaf(-d.x, sc, y[2 * p]), e1 = __builtin_fmaf(-d.y, sc, y[2 * p + 1]);
        e2 = __builtin_fmaf(e0, e0, e2);
        e2 = __builtin_fmaf(e1, e1, e2);
    }
    e2 = quad_sum(e2);
    // lane j < 16 takes over block j of the wavefront and stores it
    const bool st = lane < 16u && gidx0 + lane < (a.nchunks >> 2);
    if (a.amax) {   // uniform
        const float g = gather_quads<MIRRORED>(am, lane);
        if (st) a.amax[gidx0 + lane] = g;
    }
    if (a.sqerr) {
        const float g = gather_quads<MIRRORED>(e2, lane);
        if (st) a.sqerr[gidx0 + lane] = g;
    }
    if (a.sqerr_bfp4) {   // uniform
        // The FP16-scale counterpart (Sec. 3, 4.1): scale s = half(max / 6), codes = E2M1 rounding of
        // the correctly rounded quotient y / s, loss against code value * s (an exact product).
        const float s = (float)(_Float16)fminf(am / 6.0f, 65504.0f);
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = (s > 0.0f) ? y[i] / s : 0.0f;
        const uint32_t wb = encode8_e2m1_signed_zero(r, 127u);
        float eb = 0.0f;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            f2 d;
            if (p == 0) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wb, 1.0f, 0);
            if (p == 1) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wb, 1.0f, 1);
            if (p == 2) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wb, 1.0f, 2);
            if (p == 3) d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wb, 1.0f, 3);
            const float e0 = __builtin_fmaf(-d.x, s, y[2 * p]), e1 = __builtin_fmaf(-d.y, s, y[2 * p + 1]);
            eb = __builtin_fmaf(e0, e0, eb);
            eb = __builtin_fmaf(e1, e1, eb);
        }
        eb = quad_sum(eb);
        const float g = gather_quads<MIRRORED>(eb, lane);
        if (st) a.sqerr_bfp4[gidx0 + lane] = g;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if (t < (int)a.nt) {   // uniform
            const float th = a.th[t];
            // a lane without a chunk carries a copy of the last one: its comparisons are masked out
            const float lim = live ? th : __builtin_inff();
            count_above8(cnt[t], y, lim);
        }
    }
}

// The wavefront's sums go to LDS (`red`: 8 words, zeroed by the caller before a barrier) through one lane,
// then one lane per threshold adds the workgroup's sum to the global counter.
__device__ __forceinline__ void stats_flush(const uint32_t (&cnt)[8], uint32_t* red, const RowArgs& a) {
    if ((threadIdx.x & 63u) == 0) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (t < (int)a.nt && cnt[t]) atomicAdd(&red[t], cnt[t]);
    }
    __syncthreads();
    if (threadIdx.x < a.nt && red[threadIdx.x]) atomicAdd(&a.counts[threadIdx.x], (unsigned long long)red[threadIdx.x]);
}

// Threads of a workgroup of k_rowwise (statistics: see stats_grid).
constexpr int row_threads(int mode) { return mode == MODE_STATS ? 1024 : 256; }      // at most

// One chunk per lane per step, U steps in flight (the launcher uses U = 1).  LOG2B = 0 means "no rotation":
// the quantizer alone, or (MODE_ROTATE with a producer) the gated activation alone, stored to y.
template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool CONTIG, int U, bool PROD>
__global__ void __launch_bounds__(row_threads(MODE)) k_rowwise(RowArgs a) {
    const uint32_t NT = MODE == MODE_STATS ? blockDim.x : (uint32_t)row_threads(MODE);
    const uint32_t lane = threadIdx.x & 63;
    constexpr bool ROT = MODE != MODE_QUANT && LOG2B > 0;   // LOG2B = 0 with MODE_ROTATE: the producer alone
    __shared__ uint32_t red[8];
    uint32_t cnt[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (MODE == MODE_STATS) {
        if (threadIdx.x < 8) red[threadIdx.x] = 0;
        __syncthreads();
    }
    const uint32_t lc = wht_mirrored(LOG2B) ? chunk_of_lane(lane) : lane;      // this lane's chunk of the wavefront's 64
    const uint32_t tc = (threadIdx.x & ~63u) + lc;                              // ... of the workgroup's
    const float cs = as_f32(norm_bits(LOG2B)) * wht_sign<LOG2B>(lc);
    const uint32_t step = gridDim.x * NT * U;
    uint32_t sm[U][8];
    const bool presigned = ROT && a.signs && a.sign_fixed;   // uniform
    if (presigned) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            sign_masks(sm[u], a.signs + (size_t)((blockIdx.x * NT * U + u * NT + tc) % a.cpr) * 8);
    }
    // `bb` is uniform over the workgroup and nothing below branches on the lane: chunks past
    // the end re-read the last chunk (clamped index) and only their stores are masked, so
    // every lane exchange sees a full wavefront.
    // The statistics run a fixed number of workgroups through many passes: the next pass's chunk is requested before
    // this one's is worked on (the short-lived workgroups of the other modes overlap each other instead).
    auto chunk_at = [&](uint32_t c) { return (const char*)a.x + chunk_offset<CONTIG>(min(c, a.nchunks - 1u), a.cpr, a.ldx) * (IN_BF16 ? 2 : 4); };
    RawChunk<IN_BF16> ahead[MODE == MODE_STATS ? U : 1];
    if constexpr (MODE == MODE_STATS) {
#pragma unroll
        for (int u = 0; u < U; ++u) ahead[u] = load_raw<IN_BF16>(chunk_at(blockIdx.x * NT * U + u * NT + tc));
    }
    for (uint32_t bb = blockIdx.x * NT * U; bb < a.nchunks; bb += step) {
        float v[U][8];
        if constexpr (MODE == MODE_STATS) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                widen<IN_BF16>(ahead[u], v[u]);
                ahead[u] = load_raw<IN_BF16>(chunk_at(bb + step + u * NT + tc));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t c = min(bb + u * NT + tc, a.nchunks - 1u);
            const char* p = (const char*)a.x + chunk_offset<CONTIG>(c, a.cpr, a.ldx) * (IN_BF16 ? 2 : 4);
            const char* p2 = PROD ? (const char*)a.x2 + chunk_offset<CONTIG>(c, a.cpr, a.ldx2) * (IN_BF16 ? 2 : 4) : nullptr;
            if constexpr (MODE != MODE_STATS) load_input<IN_BF16, PROD>(p, p2, a.hround != 0, v[u]);
            if constexpr (ROT) {
                if (presigned) {
                    flip(v[u], sm[u]);
                } else if (a.signs) {   // uniform
                    uint32_t kc;
                    if ((a.cpr & 63u) == 0) {   // a wavefront's 64 chunks lie in one row: scalar modulo
                        const uint32_t cb = __builtin_amdgcn_readfirstlane(c);
                        kc = cb % a.cpr + (c - cb);
                    } else {
                        kc = c % a.cpr;
                    }
                    apply_signs(v[u], a.signs + (size_t)kc * 8);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c = bb + u * NT + tc;
            const bool live = c < a.nchunks;
            if constexpr (ROT) {
                wht_inwave<LOG2B>(v[u], lc);
#pragma unroll
                for (int i = 0; i < 8; ++i) v[u][i] *= cs;
            }
            if constexpr (MODE == MODE_ROTATE) {
                if (live) {
                    char* p = (char*)a.y + chunk_offset<CONTIG>(c, a.cpr, a.ldy) * (OUT_BF16 ? 2 : 4);
                    // (a quad's four chunks are live together: the chunk count is a multiple of 4)
                    if constexpr (OUT_BF16) store_chunk<true>(p, v[u]);
                    else store_chunk_f32_quad(p, v[u], lane, lc);
                }
            } else if constexpr (MODE == MODE_STATS) {
                stats_chunk<wht_mirrored(LOG2B)>(v[u], (c - lc) >> 2, live, lane, a, cnt);
            } else {
                uint32_t sb = e8m0_from_amax(quad_max(absmax8(v[u])));
                uint32_t w = encode8_e2m1(v[u], sb);
                if (a.stages == 0) {
                    if (live) {
                        store_codes(&a.codes[c], w, a.through);
                        if ((lane & 3) == 0) *(&a.scales[c >> 2]) = (uint8_t)sb;
                    }
                } else if ((a.cpr & 63u) == 0) {
                    // K % 512 == 0: the 64 chunks of a wavefront lie in one row and one scale
                    // superstage, so the row arithmetic is scalar and a lane adds a constant
                    const uint32_t cb = __builtin_amdgcn_readfirstlane(c);       // lane 0's chunk
                    const uint32_t row = cb / a.cpr, kc0 = cb - row * a.cpr;     // kc0 % 64 == 0
                    uint8_t* cbase = reinterpret_cast<uint8_t*>(a.codes) + tiled_code_offset(row, kc0, a.stages);
                    uint8_t* sbase = a.scales + tiled_scale_offset(row, kc0, a.sstages);
                    if (live) {
                        store_codes(reinterpret_cast<uint32_t*>(cbase + (lc >> 4) * 4096u + (lc & 15u) * 4u), w, a.through);
                        if ((lane & 3) == 0) *(sbase + (lc >> 2)) = (uint8_t)sb;
                    }
                } else if (live) {
                    const uint32_t row = c / a.cpr, kc = c - row * a.cpr;
                    store_codes(reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(a.codes) + tiled_code_offset(row, kc, a.stages)), w, a.through);
                    if ((lane & 3) == 0) *(a.scales + tiled_scale_offset(row, kc, a.sstages)) = (uint8_t)sb;
                }
            }
        }
    }
    // (a block of 512 and more divides K: nothing to pad)
    if constexpr ((MODE == MODE_QUANT || MODE == MODE_FUSED) && LOG2B < 9) a.pad.zero(blockIdx.x * NT + threadIdx.x, gridDim.x * NT);
    if constexpr (MODE == MODE_STATS) {
        if (a.counts) stats_flush(cnt, red, a);   // uniform
    }
}

// Quantize / fused rotate+quantize into the tiled layout, B <= 128 and K % 128 == 0.  In that
// layout 128 contiguous bytes of codes are one stage (128 elements) of TWO rows, so the
// row-wise mapping above would write half cache lines.  Here a wavefront takes 4 rows x one
// stage: lane l holds chunk (l & 15) of row 4 rq + (l >> 4), reads 4 x 256 contiguous bytes and
// writes 256 contiguous bytes of codes (two whole lines).  Every address is a wavefront-uniform
// base plus a per-lane constant.  Rotation blocks of up to 16 chunks stay inside one row's lanes.
// PAD: K % 512 != 0.  (Where there is nothing to pad, testing for it costs 1 % of 56 us: the workgroups are short.)
template <int LOG2B, bool IN_BF16, int MODE, bool PROD, bool PAD>
__global__ void __launch_bounds__(256) k_rowwise_t4(RowArgs a) {
    const uint32_t rows = a.rows, nitems = a.nitems;
    static_assert(LOG2B == 0 || (LOG2B >= 3 && LOG2B <= 7), "a rotation block must fit 16 lanes");
    constexpr int ES = IN_BF16 ? 2 : 4;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lc = (wht_mirrored(LOG2B) ? chunk_of_lane(lane) : lane) & 15u;   // this lane's chunk of the stage
    const float cs = as_f32(norm_bits(LOG2B)) * wht_sign<LOG2B>(lc);
    const uint32_t spr = a.cpr >> 4;                                   // stages per row
    const uint32_t lrow = lane >> 4, out_lane = wht_mirrored(LOG2B) ? (lane & 48u) + lc : lane;
    uint32_t sm[8];
    const bool presigned = MODE != MODE_QUANT && a.signs && a.sign_fixed;   // uniform
    if (presigned) sign_masks(sm, a.signs + ((size_t)((blockIdx.x * 4u + wave) % spr) * 16u + lc) * 8);
    // Every address is a wavefront-uniform base plus a per-lane constant (the host checked that
    // 4 rows of pitch fit 32 bits): the loop body spends no vector instruction on addresses.
    const uint32_t in_lane = lrow * (uint32_t)a.ldx * ES + lc * (8u * ES);
    const uint32_t in_lane2 = PROD ? lrow * (uint32_t)a.ldx2 * ES + lc * (8u * ES) : 0u;
    const uint32_t step = gridDim.x * 4u;
    for (uint32_t it = blockIdx.x * 4u + wave; it < nitems; it += step) {
        const uint32_t rq = it / spr, st = it - rq * spr;              // scalar
        const uint32_t row0 = rq * 4u;
        const char* rowbase = (const char*)a.x + ((uint64_t)row0 * (uint64_t)a.ldx + (uint64_t)st * 128u) * ES;   // scalar
        const char* p = rowbase + in_lane;
        const char* p2 = nullptr;
        if constexpr (PROD)
            p2 = (const char*)a.x2 + ((uint64_t)row0 * (uint64_t)a.ldx2 + (uint64_t)st * 128u) * ES + in_lane2;
        if (row0 + 4u > rows) {   // uniform: M % 4 != 0, last item of a column; rows past the end
                                  // re-read the last row, their stores are masked below
            const uint32_t rrow = min(row0 + lrow, rows - 1u);
            p = (const char*)a.x + ((uint64_t)rrow * (uint64_t)a.ldx + (uint64_t)st * 128u + lc * 8u) * ES;
            if constexpr (PROD)
                p2 = (const char*)a.x2 + ((uint64_t)rrow * (uint64_t)a.ldx2 + (uint64_t)st * 128u + lc * 8u) * ES;
        }
        float v[8];
        load_input<IN_BF16, PROD>(p, p2, a.hround != 0, v);
        if constexpr (MODE != MODE_QUANT) {
            if (presigned) flip(v, sm);
            else if (a.signs) apply_signs(v, a.signs + ((size_t)st * 16u + lc) * 8);
            wht_inwave<LOG2B>(v, lc);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] *= cs;
        }
        const uint32_t sb = e8m0_from_amax(quad_max(absmax8(v)));
        const uint32_t w = encode8_e2m1(v, sb);
        uint8_t* cbase = reinterpret_cast<uint8_t*>(a.codes) + ((uint64_t)(row0 >> 6) * a.stages + st) * 4096u + (row0 & 63u) * 64u;
        uint8_t* sbase = a.scales + ((uint64_t)(row0 >> 6) * a.sstages + (st >> 2)) * 1024u + (row0 & 63u) * 16u + (st & 3u) * 4u;
        if (row0 + lrow < rows) {
            store_codes(reinterpret_cast<uint32_t*>(cbase + out_lane * 4u), w, a.through);
            if ((lane & 3) == 0) *(sbase + lrow * 16u + (lc >> 2)) = (uint8_t)sb;
        }
    }
    if constexpr (PAD) a.pad.zero(blockIdx.x * 256u + threadIdx.x, gridDim.x * 256u);
}

// ---- 1024 <= B <= 8192 in registers (includes the global, full-K rotation) ----
//
// A lane holds up to 8 chunks, one of each 512-element piece of the block: the stages h < 512 run between lanes, the
// others (still ascending) between a lane's own registers, and all of a block's loads are in flight at once.  Up to
// B = 4096 a wavefront has the whole block and there is no LDS and no barrier.  At B = 8192 two wavefronts (one
// workgroup) share it: for the last stage each gives half of its pieces to the other through LDS, 16 KB there and back.
// (One wavefront with 16 chunks a lane leaves room for 3 per SIMD and spills.)
// Through LDS altogether (two trips for the stages h >= 512, the stages h = 32 .. 256 through its swizzle) the block
// cost 34 LDS operations per 8 values of a lane and was bound by them; now it is bound by the vector units (about 20
// instructions per value of a lane at B = 8192, 18 of the 25 us on 4096 x 8192; with x in a cache 25.0, in none 25.4).  A row's
// 128-byte lines of tiled codes (two rows each) are left to two wavefronts: no streaming hint (3000 x 8192, B = 2048, with the
// product behind it 39 us instead of 36); from 256 KB of codes on at device scope
// (store_codes; 4096 x 8192 B = 8192 with its product 57.6 -> 56.8), below that plain stores (1 x 8192: 0.4 us less).
// Quantizing X bf16, tiled codes, before -> after, us: 4096 x 8192 B = 1024 / 2048 / 4096 / 8192 30 / 31 / 28 / 31 ->
// 25 / 23 / 24 / 26; 16384 x 8192 101 / 102 / 102 / 108 -> 78 / 77 / 76 / 83.
constexpr int reg_waves(int log2b) { return log2b == 13 ? 2 : 1; }              // wavefronts per block
constexpr int reg_threads(int log2b) { return log2b == 13 ? 128 : 256; }        // threads per workgroup (statistics: see launch_reg)
// wavefronts per SIMD that the registers are to leave room for (storing rotated values takes an address per piece)
constexpr int reg_occ(int log2b, int mode) { return log2b >= 12 ? (mode == MODE_ROTATE ? 3 : 4) : log2b == 11 ? (mode == MODE_ROTATE ? 5 : 6) : 8; }
template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool PROD, int NT>
__global__ void __launch_bounds__(NT, reg_occ(LOG2B, MODE)) k_rowwise_reg(RowArgs a, uint32_t blocks_per_row, uint32_t nblocks) {
    static_assert(IN_BF16, "fp32 blocks go through LDS");
    if constexpr (MODE != MODE_STATS) load_args(a.x, a.codes, a.scales, a.ldx, a.cpr, a.through, a.stages, a.sstages, a.signs, blocks_per_row, nblocks);
    constexpr int W = reg_waves(LOG2B), BPW = NT / 64 / W;             // blocks per workgroup
    constexpr int NP = 1 << (LOG2B - 9), NJ = NP / W;                          // pieces per block and per wavefront
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t half = W == 2 ? wave : 0u;
    const uint32_t lc = chunk_of_lane(lane);
    const float cs = as_f32(norm_bits(LOG2B)) * wht_sign<9>(lc);
    __shared__ v4f xch[W == 2 ? 2 * NJ * 64 : 1];                               // [wavefront][piece][4 values][lane]
    __shared__ uint32_t red[8];
    uint32_t cnt[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (MODE == MODE_STATS) {
        if (threadIdx.x < 8) red[threadIdx.x] = 0;
        __syncthreads();
    }
    for (uint32_t bid = blockIdx.x * BPW + (W == 1 ? wave : 0u); bid < nblocks; bid += gridDim.x * BPW) {   // uniform per block
        const uint32_t row = bid / blocks_per_row, blk = bid - row * blocks_per_row;
        const uint32_t kc0 = blk * (64u * NP);                                  // the block's first chunk
        const uint32_t first = kc0 + half * (64u * NJ) + lc;                    // this lane's, in the wavefront's first piece
        const char* const p = (const char*)a.x + ((int64_t)row * a.ldx + (int64_t)first * 8) * 2;
        float v[NJ][8];
        {
            RawChunk<true> raw[NJ], raw2[PROD ? NJ : 1];
#pragma unroll
            for (int j = 0; j < NJ; ++j) raw[j] = load_raw<true>(p + j * 1024);
            if constexpr (PROD) {
                const char* const p2 = (const char*)a.x2 + ((int64_t)row * a.ldx2 + (int64_t)first * 8) * 2;
#pragma unroll
                for (int j = 0; j < NJ; ++j) raw2[j] = load_raw<true>(p2 + j * 1024);
            }
            __builtin_amdgcn_sched_barrier(0);      // all loads first
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                widen<true>(raw[j], v[j]);
                if constexpr (PROD) {
                    float u[8];
                    widen<true>(raw2[j], u);
                    swiglu8(v[j], u, a.hround != 0);
                }
            }
        }
        if (a.signs) {   // uniform
#pragma unroll
            for (int j = 0; j < NJ; ++j) apply_signs(v[j], a.signs + (size_t)(first + 64u * j) * 8);
        }
        // (one chunk after the other, here and below: the scheduler interleaves them all and runs out of registers)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            wht_inwave<9>(v[j], lc);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int g = 1; g < NJ; g *= 2)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if ((j & g) == 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float s0 = v[j][i], s1 = v[j + g][i];
                        v[j][i] = s0 + s1;
                        v[j + g][i] = s0 - s1;
                    }
                }
        if constexpr (W == 2) {
            // the last stage: piece j of the first wavefront with piece j of the second.  The first keeps its lower
            // pieces and takes the second's, the second keeps its upper ones and takes the first's.
            constexpr int H = NJ / 2;
            auto give = [&](const float (&y)[8], int j) {
                xch[((half * H + j) * 2 + 0) * 64 + lane] = v4f{y[0], y[1], y[2], y[3]};
                xch[((half * H + j) * 2 + 1) * 64 + lane] = v4f{y[4], y[5], y[6], y[7]};
            };
            if (half == 0) {
#pragma unroll
                for (int j = 0; j < H; ++j) give(v[H + j], j);
            } else {
#pragma unroll
                for (int j = 0; j < H; ++j) give(v[j], j);
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < H; ++j) {
                const v4f r0 = xch[(((1u - half) * H + j) * 2 + 0) * 64 + lane], r1 = xch[(((1u - half) * H + j) * 2 + 1) * 64 + lane];
                const float r[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
                if (half == 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) { const float s0 = v[j][i]; v[j][i] = s0 + r[i]; v[H + j][i] = s0 - r[i]; }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) { const float s1 = v[H + j][i]; v[j][i] = r[i] + s1; v[H + j][i] = r[i] - s1; }
                }
            }
        }
        // (every value is made here: the compiler sinks sums and differences to where they are used and keeps both of
        // their operands instead)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[j][i] *= cs;
                asm volatile("" : "+v"(v[j][i]));
            }
        // v[j] is now piece `piece(j)` of the block, counted from the wavefront's first
        constexpr auto piece = [](int j) { return W == 1 || j < NJ / 2 ? j : NJ / 2 + j; };
        const uint32_t out0 = kc0 + half * (64u * (NJ / 2)) + lc;
        // where this lane's codes and scales of the first piece go, and from piece to piece
        const bool rm = a.stages == 0;
        uint8_t* const cd = reinterpret_cast<uint8_t*>(a.codes) + (rm ? (uint64_t)(row * a.cpr + out0) * 4u : tiled_code_offset(row, out0, a.stages));
        uint8_t* const sd = a.scales + (rm ? (uint64_t)((row * a.cpr + out0) >> 2) : tiled_scale_offset(row, out0, a.sstages));
        const uint32_t cstep = rm ? 256u : 16384u, sstep = rm ? 16u : 1024u;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t kc = out0 + 64u * piece(j);
            if constexpr (MODE == MODE_ROTATE) {
                static_assert(OUT_BF16, "fp32 blocks go through LDS");
                store_chunk<true>((char*)a.y + ((int64_t)row * a.ldy + (int64_t)kc * 8) * 2, v[j]);
            } else if constexpr (MODE == MODE_STATS) {
                stats_chunk<true>(v[j], (row * a.cpr + kc - lc) >> 2, true, lane, a, cnt);
            } else {
                const uint32_t sb = e8m0_from_amax(quad_max(absmax8(v[j])));
                const uint32_t w = encode8_e2m1(v[j], sb);
                uint32_t* const c = reinterpret_cast<uint32_t*>(cd + piece(j) * cstep);
                if (a.through) store_codes(c, w, 1u);                           // uniform
                else *c = w;
                if ((lane & 3u) == 0) sd[piece(j) * sstep] = (uint8_t)sb;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (W == 2 && MODE == MODE_STATS) __syncthreads();            // the next block's pieces go where this one's were read
    }
    if constexpr (MODE == MODE_STATS) {
        if (a.counts) stats_flush(cnt, red, a);   // uniform
    }
}

// ---- LDS-staged rotation: B = 16384, and fp32 values from B = 1024 on (more registers than a wavefront has, or slower, see
// launch_wide) ----
//
// One workgroup of NT = min(256, B/8) lanes transforms one B-block of one row.  Each
// lane holds CH = B/(8*NT) chunks.  Stages h < 512 run as above; the remaining
// R = log2(B) - 9 stages (h = 512 ... B/2, still ascending) run as one radix-2^R pass
// over LDS: a lane gathers the 2^R elements {g + 512 j}, does the R stages in registers
// and scatters them back.  Then every lane re-reads its own chunks and finishes.
template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool PROD>
__global__ void __launch_bounds__(256) k_rowwise_lds(RowArgs a, uint32_t blocks_per_row, uint32_t nblocks) {
    constexpr int B = 1 << LOG2B;
    constexpr int NT = (B / 8 < 256) ? B / 8 : 256;
    constexpr int CH = B / 8 / NT;
    constexpr int R = LOG2B - 9;
    constexpr int RADIX = 1 << R;
    constexpr int GROUPS_PER_LANE = 512 / NT;
    extern __shared__ float lds[];   // B floats

    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t lc = chunk_of_lane(lane);
    const float sigma = wht_sign<9>(lc);
    __shared__ uint32_t red[8];
    uint32_t cnt[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (MODE == MODE_STATS) {
        if (tid < 8) red[tid] = 0;    // barriers follow below before anyone adds
    }
    // One block per pass; the launcher gives every block its own workgroup except for the
    // statistics, where fewer workgroups mean fewer atomics on the counters.
    for (uint32_t bid = blockIdx.x; bid < nblocks; bid += gridDim.x) {
        const uint32_t row = bid / blocks_per_row, blk = bid - row * blocks_per_row;
        const int64_t xoff = (int64_t)row * a.ldx + (int64_t)blk * B;
        const int64_t xoff2 = PROD ? (int64_t)row * a.ldx2 + (int64_t)blk * B : 0;

#pragma unroll
        for (int c = 0; c < CH; ++c) {
            float v[8];
            uint32_t q = c * NT + (tid & ~63u) + lc;   // chunk index inside the block
            load_input<IN_BF16, PROD>((const char*)a.x + (xoff + (int64_t)q * 8) * (IN_BF16 ? 2 : 4),
                                      PROD ? (const char*)a.x2 + (xoff2 + (int64_t)q * 8) * (IN_BF16 ? 2 : 4) : nullptr,
                                      a.hround != 0, v);
            if (a.signs) apply_signs(v, a.signs + ((size_t)blk * B + (size_t)q * 8));
            wht_inwave<9>(v, lc);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] *= sigma;   // exact: back to the true sign
            float4* dst = reinterpret_cast<float4*>(lds + q * 8);
            dst[0] = make_float4(v[0], v[1], v[2], v[3]);
            dst[1] = make_float4(v[4], v[5], v[6], v[7]);
        }
        __syncthreads();
#pragma unroll
        for (int gi = 0; gi < GROUPS_PER_LANE; ++gi) {
            uint32_t g = gi * NT + tid;   // 0 .. 511
            float r[RADIX];
#pragma unroll
            for (int j = 0; j < RADIX; ++j) r[j] = lds[g + 512 * j];
#pragma unroll
            for (int h = 1; h < RADIX; h *= 2) {
#pragma unroll
                for (int j = 0; j < RADIX; ++j) {
                    if ((j & h) == 0) {
                        float p = r[j], m = r[j + h];
                        r[j] = p + m;
                        r[j + h] = p - m;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < RADIX; ++j) lds[g + 512 * j] = r[j];
        }
        __syncthreads();
        const float cn = as_f32(norm_bits(LOG2B));
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            uint32_t q = c * NT + tid;
            const float4* src = reinterpret_cast<const float4*>(lds + q * 8);
            float4 lo = src[0], hi = src[1];
            float y[8] = {lo.x * cn, lo.y * cn, lo.z * cn, lo.w * cn, hi.x * cn, hi.y * cn, hi.z * cn, hi.w * cn};
            if constexpr (MODE == MODE_ROTATE) {
                int64_t yoff = (int64_t)row * a.ldy + (int64_t)blk * B + (int64_t)q * 8;
                if constexpr (OUT_BF16) store_chunk<true>((char*)a.y + yoff * 2, y);
                else store_chunk_f32_quad((char*)a.y + yoff * 4, y, lane, lane);
            } else if constexpr (MODE == MODE_STATS) {
                stats_chunk<false>(y, (row * a.cpr + blk * (B / 8) + q - lane) >> 2, true, lane, a, cnt);
            } else {
                quant_store(y, row, blk * (B / 8) + q, lane, a);
            }
        }
        __syncthreads();   // the next pass overwrites the LDS this pass has just read
    }
    if constexpr (MODE == MODE_STATS) {
        if (a.counts) stats_flush(cnt, red, a);   // uniform
    }
}

// ---- host side ---------------------------------------------------------------------

// Whether codes are stored through the L2 (store_codes).  Online step and product together, us, streaming hint -> through:
// row-major 256 x 4096 x 4096 16.2 -> 13.9, 1000 x 4096 x 11008 49.1 -> 43.6, 2000 x 4096 x 11008 79.2 -> 69.4, 4096 x 4096 x
// 4096 51.2 -> 49.7, 64 x 4096 x 4096 (128 KB of codes) 13.1 -> 13.3, 16 x 4096 x 4096 12.3 -> 12.6.  Tiled operands from 1
// to 10 MB gain little by little as K grows.  Time through the L2 over that with the hint, geometric mean (best, worst) over
// N 512 .. 28672, 28 to 49 shapes each: K = 2048 0.991 (0.94, 1.07), 4096 0.993 (0.96, 1.04), 6144 0.987 (0.90, 1.05), 8192
// 0.982 (0.90, 1.02), 10240 0.981 (0.85, 1.01), 11008 0.980 (0.91, 1.02).  More than K it is N, which the quantizer does not
// know: 0.961 with 512 columns, 0.98 with 1024 and 2048, 0.995 up to 14336, 1.001 with 28672.  So no line in M and K is
// sharp, and this one, K > 8192, is on the careful side: beyond it hardly a shape loses more than 2 % (1000 x 4096 x 11008
// with its activation 38.2 -> 34.9, 721 x 4096 x 11008 32.8 -> 30.6, 274 x 1024 x 14336 27.7 -> 24.4; but 358 x 14336 x 11008
// 42.8 -> 43.8, 194 x 14336 x 11008 33.0 -> 34.0, 209 x 28672 x 10240 51 -> 53.4), and K = 8192, left out, would gain as much
// as what is in.  From 16 MB on the quantizer itself is faster (16384 x 8192 58.0 -> 57.0, 8000 x 8192 29.9 -> 29.3, 3000 x
// 8192 as before).
static bool code_stores_through(bool tiled, int64_t M, int64_t K) {
    return M * (K / 2) >= (int64_t(1) << (!tiled ? 18 : K > 8192 ? 20 : 24));
}

// Workgroups per compute unit of a statistics launch of k_rowwise_lds and k_rowwise_reg.
constexpr int STATS_LDS_WGS_PER_CU = 8;
// ... and of k_rowwise.  Every workgroup ends with an atomic per counter, all of them on one cache line: two counters and 768
// workgroups were 10 us at the end of every launch (1000 x 8192 13.6 us, of 17 MB).  So the wavefronts a CU needs come in few
// large workgroups, the fewer the more the atomics weigh: three of 512 threads, two of 768, one of 1024.  us, B = 1 / 32 / 128,
// three (before: always), one, two: 1000 x 8192 13.6 / 14.0 / 14.4, 8.6 / 9.1 / 9.7, 11.0 / 11.4 / 11.5; 4000 x 4096 15.8 /
// 16.1 / 16.5, 11.4 / 12.9 / 13.6, 12.8 / 13.3 / 13.6; 6000 x 8192 26.5 / 28.1 / 30.1, 24.9 / 29.0 / 31.3, 24.3 / 27.5 / 30.2;
// 16384 x 8192 59.0 / 65.4 / 70.6, 66.3 / 70.9 / 76.9, 60.0 / 64.7 / 70.5.  (Two chunks requested ahead instead of one: 2 % slower.)
// Up to 80 workgroups the atomics are nothing and the chunks are on more CUs in workgroups of 512, B = 32, 1024 threads ->
// 512: 16 x 4096 3.97 -> 3.59, 64 x 736 3.92 -> 3.53, 31 x 8192 4.19 -> 4.08; 42 x 8192 (84 workgroups of 512) 4.32 either way,
// 54 x 8192 4.42 -> 4.59.
struct StatsGrid { int workgroups, threads; };
static StatsGrid stats_grid(uint32_t chunks, int cus) {
    const int per_cu = chunks <= (1u << 21) ? 1 : chunks <= (1u << 23) ? 2 : 3;
    const int threads = per_cu == 2 ? 768 : per_cu == 3 || chunks <= 80u * 512u ? 512 : 1024;
    const int cap = cus * per_cu, need = (int)((chunks + threads - 1) / threads);
    return {need < cap ? need : cap, threads};
}

// Workgroups of a streaming launch.  Measured on X 16384 x 8192 (bf16, B = 32): one chunk in
// flight per lane and many short-lived workgroups beat a persistent grid (8 per CU, two
// chunks in flight: 63 us; 64 per CU, one chunk: 55 us): the dispatcher keeps every CU topped up
// and the loads of a finished workgroup's successor overlap the arithmetic of its neighbours.
// Each workgroup still makes about 3 passes so that small inputs do not pay for launching
// thousands of workgroups (1 pass: 15 % slower; 2, 4 and 8 passes: 1 - 4 % slower than 3, on 32 to 340 MB).
static int rowwise_grid(uint32_t nchunks, int U, int cus) {
    const uint32_t need = (nchunks + 256u * U - 1) / (256u * U);
    uint32_t grid = need / 3;
    const uint32_t lo = (uint32_t)cus * 8, hi = (uint32_t)cus * 64;
    if (grid < lo) grid = lo;
    if (grid > hi) grid = hi;
    return (int)(need < grid ? need : grid);
}

// Signed rotations: round `grid` down to a multiple of period / gcd(period, per_wg), so that one
// grid-stride pass (grid * per_wg work items) is a whole number of rows' worth of columns and
// every lane meets the same column, hence the same signs, in every pass.  Returns 1 if the grid
// could be sized that way (it is left alone, and 0 returned, when that would shrink it by more
// than half).
static uint32_t fix_columns(int& grid, uint32_t period, uint32_t per_wg) {
    uint32_t x = period, y = per_wg;
    while (y) { uint32_t t = x % y; x = y; y = t; }
    const uint32_t unit = period / x;
    const uint32_t g = (uint32_t)grid / unit * unit;
    if (g == 0 || g * 2 < (uint32_t)grid) return 0;
    grid = (int)g;
    return 1;
}

// The same for a statistics launch, whose few workgroups feel every one that rounding takes away.  A launch of one pass would
// become one of two: it stays as it is below 100 workgroups, from where the atomics saved pay for the second pass (us,
// rounded : not: 300 x 736 5.08 : 4.33, 1000 x 736 5.45 : 5.29, 300 x 4128 5.69 : 6.01, 500 x 4128 6.53 : 7.37).  With
// several passes reading the signs in each costs up to 20 % on 4 M values and more, 5 % on fewer: a grid that loses more than
// a quarter is not taken above 2^19 chunks (1000 x 4128, 129 of 256 workgroups, 8.29 : 8.66, 2000 x 4128 12.0 : 11.1, 4000 x
// 4128 19.9 : 16.4; 1000 x 11008, 215 of 256, 11.6 : 12.7).
static uint32_t fix_stats_columns(int& grid, uint32_t chunks, uint32_t period, uint32_t threads) {
    int g = grid;
    if (!fix_columns(g, period, threads)) return 0;
    const bool one_pass = (uint64_t)grid * threads >= chunks;
    if (one_pass ? grid < 100 : g * 4 < grid * 3 && chunks > (1u << 19)) return 0;
    grid = g;
    return 1;
}

template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool PROD = false>
static hipError_t launch_inwave(const RowArgs& a, bool contig, hipStream_t s) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
    if constexpr ((MODE == MODE_QUANT || MODE == MODE_FUSED) && LOG2B <= 7) {
        if (a.stages != 0 && (a.cpr & 15u) == 0 && a.ldx * (IN_BF16 ? 2 : 4) * 4 < (int64_t(1) << 32) &&
            (!PROD || a.ldx2 * (IN_BF16 ? 2 : 4) * 4 < (int64_t(1) << 32))) {
            const uint32_t rows = a.nchunks / a.cpr, nitems = ((rows + 3u) / 4u) * (a.cpr >> 4);
            int grid = rowwise_grid(nitems * 64u, 1, cus);
            RowArgs b = a;
            b.sign_fixed = a.signs ? fix_columns(grid, a.cpr >> 4, 4) : 0;
            b.rows = rows;
            b.nitems = nitems;
            if (b.pad.n) hipLaunchKernelGGL((k_rowwise_t4<LOG2B, IN_BF16, MODE, PROD, true>), dim3(grid), dim3(256), 0, s, b);
            else hipLaunchKernelGGL((k_rowwise_t4<LOG2B, IN_BF16, MODE, PROD, false>), dim3(grid), dim3(256), 0, s, b);
            return hipGetLastError();
        }
    }
    constexpr int U = 1;
    int grid = rowwise_grid(a.nchunks, U, cus), NT = row_threads(MODE);
    if constexpr (MODE == MODE_STATS) {
        const StatsGrid g = stats_grid(a.nchunks, cus);
        grid = g.workgroups;
        NT = g.threads;
    }
    RowArgs b = a;
    if (a.signs && MODE != MODE_QUANT && LOG2B > 0)
        b.sign_fixed = MODE == MODE_STATS ? fix_stats_columns(grid, a.nchunks, a.cpr, NT) : fix_columns(grid, a.cpr, NT * U);
    if (contig)
        hipLaunchKernelGGL((k_rowwise<LOG2B, IN_BF16, MODE, OUT_BF16, true, U, PROD>), dim3(grid), dim3(NT), 0, s, b);
    else
        hipLaunchKernelGGL((k_rowwise<LOG2B, IN_BF16, MODE, OUT_BF16, false, U, PROD>), dim3(grid), dim3(NT), 0, s, b);
    return hipGetLastError();
}

template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool PROD = false>
static hipError_t launch_lds(const RowArgs& a, int64_t M, int64_t K, hipStream_t s) {
    constexpr int B = 1 << LOG2B;
    constexpr int NT = (B / 8 < 256) ? B / 8 : 256;
    uint32_t bpr = (uint32_t)(K / B);
    const uint32_t nblocks = (uint32_t)(M * bpr);
    uint32_t grid = nblocks;
    if (MODE == MODE_STATS) {
        int cus = 0;
        if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
        const uint32_t cap = (uint32_t)cus * (uint32_t)STATS_LDS_WGS_PER_CU;
        if (grid > cap) grid = cap;
    }
    hipLaunchKernelGGL((k_rowwise_lds<LOG2B, IN_BF16, MODE, OUT_BF16, PROD>), dim3(grid), dim3(NT),
                       B * sizeof(float), s, a, bpr, nblocks);
    return hipGetLastError();
}

template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool PROD, int NT = reg_threads(LOG2B)>
static hipError_t launch_reg(const RowArgs& a, int64_t M, int64_t K, hipStream_t s) {
    const uint32_t bpr = (uint32_t)(K >> LOG2B), nblocks = (uint32_t)M * bpr;
    // Statistics with B = 1024: workgroups of 1024 threads where the atomics of those of 256 weigh more than the CUs that
    // fewer workgroups leave idle, us, 256 : 1024 threads, M x 8192: 16 4.4 : 6.0, 100 6.4 : 6.5, 112 6.7 : 6.6, 400 13.9 : 8.6,
    // 4000 37.2 : 29.0, 6000 42.0 : 40.3, 7000 45.3 : 46.0, 12000 72.3 : 74.1.  (The number of threads as an argument: 1 % slower.)
    if constexpr (MODE == MODE_STATS && LOG2B == 10 && NT == 256)
        if (nblocks > 800u && nblocks <= 3u << 14) return launch_reg<LOG2B, IN_BF16, MODE, OUT_BF16, PROD, 1024>(a, M, K, s);
    RowArgs b = a;
    b.through = code_stores_through(false, M, K) ? 1u : 0u;
    constexpr uint32_t per_wg = NT / 64 / reg_waves(LOG2B);
    uint32_t grid = (nblocks + per_wg - 1u) / per_wg;
    if (MODE == MODE_STATS) {
        int cus = 0;
        if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
        const uint32_t cap = (uint32_t)cus * (uint32_t)(NT == 1024 ? 2 : STATS_LDS_WGS_PER_CU);
        if (grid > cap) grid = cap;
    }
    hipLaunchKernelGGL((k_rowwise_reg<LOG2B, IN_BF16, MODE, OUT_BF16, PROD, NT>), dim3(grid), dim3(NT), 0, s, b, bpr, nblocks);
    return hipGetLastError();
}

// 1024 <= B <= 8192: in registers where the values come and go as bf16 (or go as codes or statistics);
// blocks of fp32 values through LDS (X 16384 x 8192 fp32, B = 1024 / 4096, us: 107 / 117, in registers 119 / 130;
// fp32 out of bf16: 139 / 137 against 154 / 163).
template <int LOG2B, bool IN_BF16, int MODE, bool OUT_BF16, bool PROD>
static hipError_t launch_wide(const RowArgs& a, int64_t M, int64_t K, hipStream_t s) {
    if constexpr (IN_BF16 && (MODE != MODE_ROTATE || OUT_BF16)) return launch_reg<LOG2B, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
    else return launch_lds<LOG2B, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
}

template <bool IN_BF16, int MODE, bool OUT_BF16, bool PROD = false>
static hipError_t dispatch_b(int log2b, const RowArgs& a, bool contig, int64_t M, int64_t K, hipStream_t s) {
    switch (log2b) {
        case 3: return launch_inwave<3, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 4: return launch_inwave<4, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 5: return launch_inwave<5, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 6: return launch_inwave<6, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 7: return launch_inwave<7, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 8: return launch_inwave<8, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 9: return launch_inwave<9, IN_BF16, MODE, OUT_BF16, PROD>(a, contig, s);
        case 10: return launch_wide<10, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
        case 11: return launch_wide<11, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
        case 12: return launch_wide<12, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
        case 13: return launch_wide<13, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
        case 14: return launch_lds<14, IN_BF16, MODE, OUT_BF16, PROD>(a, M, K, s);
        default: return hipErrorInvalidValue;
    }
}

// mode: RowMode; log2b: 0 for MODE_QUANT, else 3..14.  Arguments are already validated.
hipError_t launch_rowwise(int mode, int log2b, bool in_bf16, bool out_bf16, const void* x, int64_t M,
                          int64_t K, int64_t ldx, void* y, int64_t ldy, uint8_t* codes, uint8_t* scales,
                          bool tiled, const int8_t* signs, const Producer* prod, hipStream_t s, const StatsOut* stats) {
    RowArgs a;
    a.amax = stats ? stats->amax : nullptr;
    a.sqerr = stats ? stats->sqerr : nullptr;
    a.sqerr_bfp4 = stats ? stats->sqerr_bfp4 : nullptr;
    a.counts = stats ? stats->counts : nullptr;
    a.nt = stats ? (uint32_t)stats->nt : 0u;
    for (int t = 0; t < 8; ++t) a.th[t] = (stats && t < stats->nt) ? stats->thresholds[t] : 0.0f;
    a.x2 = prod ? prod->up : nullptr;
    a.ldx2 = prod ? prod->ldu : 0;
    a.hround = (prod && prod->through_bf16) ? 1u : 0u;
    a.signs = signs;
    a.sign_fixed = 0;
    a.rows = a.nitems = 0;
    a.x = x; a.y = y; a.codes = reinterpret_cast<uint32_t*>(codes); a.scales = scales;
    a.ldx = ldx; a.ldy = ldy; a.cpr = (uint32_t)(K / 8); a.nchunks = (uint32_t)(M * (K / 8));
    const int64_t Kp = (K + 511) / 512 * 512;
    a.through = code_stores_through(tiled, M, K) ? 1u : 0u;
    a.stages = tiled ? (uint32_t)(Kp / 128) : 0u;
    a.sstages = tiled ? (uint32_t)(Kp / 512) : 0u;
    a.pad = KPad::of(tiled && mode != MODE_ROTATE && mode != MODE_STATS, codes, scales, M, K);
    bool contig = (ldx == K) && (mode != MODE_ROTATE || ldy == K) && (!prod || prod->ldu == K);
    if (mode == MODE_STATS) {   // log2b = 0: no rotation
        if (log2b == 0)
            return in_bf16 ? launch_inwave<0, true, MODE_STATS, false>(a, contig, s)
                           : launch_inwave<0, false, MODE_STATS, false>(a, contig, s);
        return in_bf16 ? dispatch_b<true, MODE_STATS, false>(log2b, a, contig, M, K, s)
                       : dispatch_b<false, MODE_STATS, false>(log2b, a, contig, M, K, s);
    }
    if (prod && mode == MODE_ROTATE) {   // the activation alone, written to y (log2b = 0)
        if (in_bf16) return out_bf16 ? launch_inwave<0, true, MODE_ROTATE, true, true>(a, contig, s)
                                     : launch_inwave<0, true, MODE_ROTATE, false, true>(a, contig, s);
        return out_bf16 ? launch_inwave<0, false, MODE_ROTATE, true, true>(a, contig, s)
                        : launch_inwave<0, false, MODE_ROTATE, false, true>(a, contig, s);
    }
    if (mode == MODE_ROTATE) {
        if (in_bf16) return out_bf16 ? dispatch_b<true, MODE_ROTATE, true>(log2b, a, contig, M, K, s)
                                     : dispatch_b<true, MODE_ROTATE, false>(log2b, a, contig, M, K, s);
        return out_bf16 ? dispatch_b<false, MODE_ROTATE, true>(log2b, a, contig, M, K, s)
                        : dispatch_b<false, MODE_ROTATE, false>(log2b, a, contig, M, K, s);
    }
    if (prod) {   // gated-activation producer in front of the quantizer / the fused step
        if (mode == MODE_QUANT)
            return in_bf16 ? launch_inwave<0, true, MODE_QUANT, false, true>(a, contig, s)
                           : launch_inwave<0, false, MODE_QUANT, false, true>(a, contig, s);
        return in_bf16 ? dispatch_b<true, MODE_FUSED, false, true>(log2b, a, contig, M, K, s)
                       : dispatch_b<false, MODE_FUSED, false, true>(log2b, a, contig, M, K, s);
    }
    if (mode == MODE_QUANT)
        return in_bf16 ? launch_inwave<0, true, MODE_QUANT, false>(a, contig, s)
                       : launch_inwave<0, false, MODE_QUANT, false>(a, contig, s);
    return in_bf16 ? dispatch_b<true, MODE_FUSED, false>(log2b, a, contig, M, K, s)
                   : dispatch_b<false, MODE_FUSED, false>(log2b, a, contig, M, K, s);
}

// ---- tiled -> row-major copy of a quantized operand (inspection and parity checks) ----
// One lane per 32-element group: its 16 code bytes and its scale byte.
__global__ void __launch_bounds__(256) k_to_rowmajor(const uint8_t* __restrict__ ct, const uint8_t* __restrict__ st,
                                                     uint32_t rows, uint32_t K, uint32_t stages, uint32_t sstages,
                                                     uint8_t* __restrict__ codes, uint8_t* __restrict__ scales) {
    const uint32_t gpr = K / 32;                       // groups (16 code bytes, 1 scale byte) per row
    const uint64_t n = (uint64_t)rows * gpr;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
        const uint32_t row = (uint32_t)(i / gpr), g = (uint32_t)(i - (uint64_t)row * gpr);
        const v4i c = *reinterpret_cast<const v4i*>(ct + tiled_code_offset(row, g * 4, stages));
        *reinterpret_cast<v4i*>(codes + i * 16) = c;
        scales[i] = st[tiled_scale_offset(row, g * 4, sstages)];
    }
}

hipError_t launch_to_rowmajor(const uint8_t* codes_t, const uint8_t* scales_t, int64_t rows, int64_t K,
                              uint8_t* codes, uint8_t* scales, hipStream_t s) {
    const int64_t Kp = (K + 511) / 512 * 512;
    const int64_t n = rows * (K / 32);
    const int64_t want = (n + 255) / 256;
    const int grid = (int)(want < 16384 ? want : 16384);
    hipLaunchKernelGGL(k_to_rowmajor, dim3(grid), dim3(256), 0, s, codes_t, scales_t, (uint32_t)rows, (uint32_t)K,
                       (uint32_t)(Kp / 128), (uint32_t)(Kp / 512), codes, scales);
    return hipGetLastError();
}

}  // namespace brq
