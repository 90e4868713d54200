// W4A4 product on MXFP4 operands for gfx950 (Sec. 2 and Sec. 4.1 of the paper: the product
// the rotation leaves invariant, evaluated on E2M1 codes with E8M0 group scales).
//
// The contraction runs on CDNA4's block-scaled MFMA.  Operand layout of
// v_mfma_scale_f32_32x32x64_f8f6f4 with fp4 inputs: lane l supplies, for row (l & 31), the
// 32 consecutive K elements of group (l >> 5) as 16 packed bytes (low nibble first), and
// one E8M0 byte for exactly that group; accumulator register i of lane l is element
// (row 8*(i/4) + 4*(l>>5) + i%4, column l & 31).  The 16x16x128 form: row (l & 15), group
// (l >> 4); accumulator i is (row 4*(l>>4) + i, column l & 15).
#include <type_traits>
#include "mfma_fp4.h"
#include "brq_launch.h"

namespace brq {

// Addressing of one row of a quantized operand, valid for both layouts: the 16 code bytes of
// group g sit at codes + (g >> 2) * cstep + (g & 3) * 16 and its scale at scales + (g >> 4) * sstep
// + (g & 15), with (cstep, sstep) = (64, 16) for row-major rows and (4096, 1024) for the tiled
// layout (64-row slabs; 64 code bytes per row and stage, 16 scale bytes per row and superstage).
struct RowView {
    const uint8_t* codes;
    const uint8_t* scales;
    uint32_t cstep, sstep;
    __device__ __forceinline__ RowView(const uint8_t* c, const uint8_t* s, bool tiled, int64_t row, int K) {
        if (tiled) {
            const int64_t Kp = ((int64_t)K + 511) / 512 * 512;
            codes = c + (row >> 6) * (Kp / 128) * 4096 + (row & 63) * 64;
            scales = s + (row >> 6) * (Kp / 512) * 1024 + (row & 63) * 16;
            cstep = 4096; sstep = 1024;
        } else {
            codes = c + row * (K / 2);
            scales = s + row * (K / 32);
            cstep = 64; sstep = 16;
        }
    }
    __device__ __forceinline__ v4i group(int g) const {
        return *reinterpret_cast<const v4i*>(codes + (int64_t)(g >> 2) * cstep + (g & 3) * 16);
    }
    __device__ __forceinline__ int scale(int g) const { return scales[(int64_t)(g >> 4) * sstep + (g & 15)]; }
};

__device__ __forceinline__ void store_out(void* y, bool out_bf16, int64_t idx, float v) {
    if (out_bf16) reinterpret_cast<uint16_t*>(y)[idx] = (uint16_t)f32_to_bf16_bits(v);
    else reinterpret_cast<float*>(y)[idx] = v;
}

// ---- general shapes: one 32x32 output tile per wavefront, operands straight from global ----
// The K groups are taken in the order of the LDS-staged kernels (step j of a 128-element stage: groups j and 2 + j),
// so that a product does not depend on which of them it runs on.
__global__ void __launch_bounds__(256) k_gemm_direct(const uint8_t* __restrict__ aq, const uint8_t* __restrict__ as,
                                                     int a_tiled, const uint8_t* __restrict__ wq,
                                                     const uint8_t* __restrict__ ws, int w_tiled, int M, int N, int K,
                                                     void* __restrict__ y, int out_bf16, int64_t ldy) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = blockIdx.y * 64 + (wave >> 1) * 32, n0 = blockIdx.x * 64 + (wave & 1) * 32;
    if (m0 >= M || n0 >= N) return;   // whole wavefront leaves together
    const int r = lane & 31, h = lane >> 5;
    const int64_t ra = min(m0 + r, M - 1), rw = min(n0 + r, N - 1);   // clamp: rows past the edge are computed, not stored
    const int groups = K / 32;
    const RowView va(aq, as, a_tiled != 0, ra, K), vw(wq, ws, w_tiled != 0, rw, K);
    v16f acc = {};
    for (int g0 = 0; g0 < groups; g0 += (g0 & 1) ? 3 : 1) {   // step j = g0 & 1 of a stage
        int g = g0 + 2 * h;
        v8i a = {}, b = {};
        int sca = 0, scb = 0;
        if (g < groups) {   // past the last group: zeros
            v4i ta = va.group(g);
            v4i tb = vw.group(g);
            a[0] = ta[0]; a[1] = ta[1]; a[2] = ta[2]; a[3] = ta[3];
            b[0] = tb[0]; b[1] = tb[1]; b[2] = tb[2]; b[3] = tb[3];
            sca = va.scale(g); scb = vw.scale(g);
        }
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 4, 0, sca, 0, scb);
    }
    const int col = n0 + r;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        int row = m0 + 8 * (i / 4) + 4 * h + (i % 4);
        if (row < M && col < N) store_out(y, out_bf16, (int64_t)row * ldy + col, acc[i]);
    }
}

// ---- M <= 16 (decode): weight streaming, 16 output columns per workgroup -------------------
// Each of the 4 wavefronts takes every 4th 128-wide K step for the same 16 weight rows; the
// partial 16x16 tiles are summed through LDS in a fixed order.
__global__ void __launch_bounds__(256) k_gemm_skinny(const uint8_t* __restrict__ aq, const uint8_t* __restrict__ as,
                                                     int a_tiled, const uint8_t* __restrict__ wq,
                                                     const uint8_t* __restrict__ ws, int w_tiled, int M, int N, int K,
                                                     void* __restrict__ y, int out_bf16, int64_t ldy) {
    __shared__ float part[4][64][4];
    load_args(aq, as, a_tiled, wq, ws, w_tiled, M, N, K, y, out_bf16, ldy);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const int n0 = blockIdx.x * 16;
    const int groups = K / 32;
    const int64_t rw = min(n0 + r, N - 1);
    const bool arow = r < M;
    const RowView va(aq, as, a_tiled != 0, arow ? r : 0, K), vw(wq, ws, w_tiled != 0, rw, K);
    v4f acc = {};
    for (int g0 = wave * 4; g0 < groups; g0 += 16) {
        int g = g0 + kq;
        v8i a = {}, b = {};
        int sca = 0, scb = 0;
        if (g < groups) {
            v4i tb = vw.group(g);
            b[0] = tb[0]; b[1] = tb[1]; b[2] = tb[2]; b[3] = tb[3];
            scb = vw.scale(g);
            if (arow) {
                v4i ta = va.group(g);
                a[0] = ta[0]; a[1] = ta[1]; a[2] = ta[2]; a[3] = ta[3];
                sca = va.scale(g);
            }
        }
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, acc, 4, 4, 0, sca, 0, scb);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) part[wave][lane][i] = acc[i];
    __syncthreads();
    if (wave == 0) {
        const int col = n0 + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float s = ((part[0][lane][i] + part[1][lane][i]) + part[2][lane][i]) + part[3][lane][i];
            int row = 4 * kq + i;
            if (row < M && col < N) store_out(y, out_bf16, (int64_t)row * ldy + col, s);
        }
    }
}

// ---- M <= 16 (decode batches): weight streaming with the activations in LDS ----------------
// HBM-bound: every weight byte is read exactly once.  A wavefront owns its weight rows for the whole
// of K (no cross-wavefront reduction, fixed summation order) and streams them through registers,
// SETS 512-element superstages in rotation.  Every wavefront would re-read all of A, so the 4 wavefronts of a
// workgroup share the activations: one superstage of A at a time goes into LDS by LDS-DMA (SETS
// buffers, one barrier per superstage), wavefront w bringing stage w.  The MFMA is the 32x32x64
// one, a wavefront per 32 weight rows, of which a workgroup has nw = 1, 2 or 4 (streaming_waves); the wavefronts
// from nw on bring their share of A and no more.  Rows past M repeat row M - 1.  (More rows than one tile of 32 go to the
// one-tile kernel: with two to four row tiles a turn waits for the latency of two superstages and multiplies longer
// than it waits, 28672 x 8192 with 64 / 128 rows 28.9 / 34.7 us against 24.8 / 28.9.)
// Operand fragments (32x32x64: lane (r, h) = (lane & 31, lane >> 5) supplies 32 consecutive K
// elements of row r): within a 128-element stage (64 code bytes per row) lane half h owns bytes
// [32 h, 32 h + 32), MFMA step j of the stage takes bytes 32 h + 16 j, i.e. group 2 h + j of the
// stage, for both operands and both scales.  A in LDS: [stage][row][64 bytes] with the 16-byte
// chunks of row i XOR-swizzled by (i >> 2) & 3 (the 16 rows of one read then spread over all
// banks), scales [tile][64 rows][16 bytes].  Output: lane (r, h) holds D[8 q + 4 h + i][r] for
// weight row n0 + r, so the 32 lanes of a half store 32 consecutive columns of one output row.

// A wavefront's 32 weight rows, a superstage at a time in 8 registers of 16 bytes per lane, and the fragments from them.
// Tiled weights: a row's 64 bytes of a stage lie between those of its neighbours, so lane (r, h) loads its fragments
// directly, 2 KB by two instructions.  Plain loads: one instruction takes half of every cache line it touches and the next
// one the other half, and a streaming load does not leave the line in the cache for it (the weights would cross HBM twice).
// Row-major weights (without ROWS they are loaded like that too): a fragment is 32 rows x 32 bytes, a quarter of each of 32
// lines, and by the time the fourth instruction asks for the last quarter the other wavefronts' lines have pushed it out.  With
// ROWS an instruction loads 8 rows x 128 bytes, whole lines and once, and the wavefront turns the four of two stages round in 4 KB of LDS that no other
// touches (row i's 16-byte chunk c at c ^ (i & 7): 8 lanes write a row, 8 rows' chunks are read, all banks either way).  A
// wavefront's LDS operations are done in order, so nothing waits there but for the data.  us, weights in no cache, 1 row,
// each lane its fragments -> now: 28672 x 8192 36.1 -> 30.5 (tiled weights 24), 14336 x 4096 10.0 -> 9.3; the one-launch call, 28672 x
// 8192 36.6 -> 30.2, 21752 x 10240 42.2 -> 28.9.  No streaming hint here either: it fetches weights past the memory-side cache that lie there.
// Both calls, 240 shapes of 8 to 230 MB of weights, 1 to 16 rows, the hint's time over that without: weights in no cache, up to 32 MB 0.99,
// above 0.96 (0.92 to 1.00; the four above 28.5, 8.8, 28.1, 27.3); in the memory-side cache 1.01, above 32 MB 1.08 (0.96 to 1.30).
template <bool ROWS>
struct WeightRows {
    const uint8_t* codes;                               // this lane's row.  ROWS: the first row (uniform), `off` from there
    const uint8_t* scales;                              // this lane's row
    uint32_t cstep, sstep, off[4];
    uint8_t *wr, *rd;                                   // ROWS: this lane's place in the 4 KB
    uint32_t sw;
    int h;
    __device__ __forceinline__ WeightRows(const uint8_t* wq, const uint8_t* ws, bool tiled, int n0, int N, int K, int lane, uint8_t* turn_lds) {
        const int r = lane & 31;
        h = lane >> 5;
        const RowView v(wq, ws, tiled, min(n0 + r, N - 1), K);
        scales = v.scales;
        cstep = v.cstep;
        sstep = v.sstep;
        if constexpr (ROWS) {
            const int first = min(n0, N - 1);           // (uniform; a wavefront without columns of its own reads the last one)
            codes = wq + (int64_t)first * (K / 2);
            const int i = lane >> 3, c = lane & 7;
#pragma unroll
            for (int q = 0; q < 4; ++q) off[q] = (uint32_t)min(8 * q + i, N - 1 - first) * (uint32_t)(K / 2) + (uint32_t)c * 16;
            wr = turn_lds + i * 128 + ((c ^ i) << 4);
            rd = turn_lds + r * 128;
            sw = (uint32_t)(r & 7);
        } else {
            codes = v.codes;
            // (a 4096 that the compiler sees lets it take a line's two halves apart)
            asm("" : "+s"(cstep));
        }
    }
    __device__ __forceinline__ void load(int ss, v4i (&c)[8], v4i& sc) const {
        if constexpr (ROWS) {
            const uint8_t* b = codes + (int64_t)ss * 256;
#pragma unroll
            for (int i = 0; i < 8; ++i) c[i] = *reinterpret_cast<const v4i*>(b + off[i & 3] + (i >> 2) * 128);
            sc = *reinterpret_cast<const v4i*>(scales + (int64_t)ss * 16);   // (a line holds those of 8 superstages)
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) c[i] = *reinterpret_cast<const v4i*>(codes + (int64_t)(4 * ss + (i >> 1)) * cstep + h * 32 + (i & 1) * 16);
            sc = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(scales + (int64_t)ss * sstep));
        }
    }
    // ROWS: the fragments of steps 4 half .. 4 half + 3 (stage 2 half + t, step j at 2 t + j).  (Without: c[step].)
    __device__ __forceinline__ void turn(const v4i (&c)[8], int half, v4i (&f)[4]) const {
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<v4i*>(wr + q * 1024) = c[4 * half + q];
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const v4i*>(rd + ((((uint32_t)(4 * (i >> 1) + 2 * h + (i & 1))) ^ sw) << 4));
    }
};
constexpr int turn_bytes(bool rows) { return rows ? 4 * 4096 : 0; }

// Weight register sets = LDS buffers of A; SETS - 1 superstages are in flight.
constexpr int smallm_buf_bytes = 4096 + 4096;
constexpr int smallm_lds_bytes(int sets, bool rows) { return sets * smallm_buf_bytes + turn_bytes(rows); }

// TAIL = (K / 512) % SETS: the superstages left after the main loop, which takes them SETS at a time in
// one basic block (no load behind a branch: the compiler's count of the outstanding weight loads is
// then exact; with early exits inside the loop it falls back to waiting for all of them).
template <bool ROWS, int SETS, int TAIL>
__global__ void __launch_bounds__(256) k_gemm_smallm(const uint8_t* __restrict__ aq, const uint8_t* __restrict__ as,
                                                     int a_tiled, const uint8_t* __restrict__ wq,
                                                     const uint8_t* __restrict__ ws, int M, int N, int K,
                                                     void* __restrict__ y, int out_bf16, int64_t ldy, int nw) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr int STG = 1024;                           // one stage of A codes: 16 rows x 64 bytes
    constexpr int BUF = smallm_buf_bytes;               // codes [4 stages][16 rows][64], then scales, 1 KB per wavefront
    constexpr int NA = 2;                               // LDS-DMA instructions per wavefront and superstage
    load_args(aq, as, a_tiled, wq, ws, M, N, K, y, out_bf16, ldy, nw);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int n0 = (blockIdx.x * nw + wave) * 32;       // (of the first nw wavefronts)
    const int nss = (K + 511) / 512;                    // tiled operands are zero-padded to whole superstages
    const int64_t Kp = (int64_t)nss * 512;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const WeightRows<ROWS> vw(wq, ws, !ROWS, n0, N, K, lane, lds + SETS * BUF + wave * 4096);

    const uint32_t a_cstep = a_tiled ? 4096u : 64u, a_sstep = a_tiled ? 1024u : 16u;
    auto row_off_c = [&](int row) -> uint32_t {
        row = min(row, M - 1);
        return a_tiled ? (uint32_t)((row >> 6) * (Kp / 128) * 4096 + (row & 63) * 64) : (uint32_t)((int64_t)row * (K / 2));
    };
    auto row_off_s = [&](int row) -> uint32_t {
        row = min(row, M - 1);
        return a_tiled ? (uint32_t)((row >> 6) * (Kp / 512) * 1024 + (row & 63) * 16) : (uint32_t)((int64_t)row * (K / 32));
    };
    // one DMA instruction = 16 rows x 64 bytes; lane i brings chunk (i & 3) ^ ((i >> 4) & 3) of row i >> 2
    const uint32_t voc = row_off_c(lane >> 2) + (uint32_t)((lane & 3) ^ ((lane >> 4) & 3)) * 16u;
    // ... and one more scale rows into 1 KB of its own: wavefront 0 those of A, the others row M - 1 over and over, which
    // nobody reads (lanes 32..63 repeat lanes 0..31): every wavefront issues the same number of loads, which the
    // counted waits below rely on
    const uint32_t vos = row_off_s(32 * wave + r);
    // wavefront `wave` brings stage `wave` of the superstage
    auto dma_a = [&](int ss, uint32_t buf) {
        const uint8_t* cb = uniform_ptr(aq + (int64_t)(4 * ss + wave) * a_cstep);
        const uint32_t lb = lds0 + buf * BUF + (uint32_t)wave * STG;
        dma16<0>(lb, cb, voc);
        dma16<0>(lds0 + buf * BUF + 4 * STG + (uint32_t)wave * 1024, uniform_ptr(as + (int64_t)ss * a_sstep), vos);
    };
    v16f acc = {};
    const uint32_t ra = (uint32_t)r & 15u;              // lanes 16..31 of a half repeat rows 0..15: never stored
    const uint32_t sw = (ra >> 2) & 3u;
    // The 8 steps (stage t, half-step j) of a superstage; the A fragment of step s + 1 is read while step s multiplies.
    auto superstage = [&](uint32_t buf, const v4i (&c)[8], const v4i& sc) {
        const uint8_t* cb = lds + buf * BUF + ra * 64;
        const v4i asc = *reinterpret_cast<const v4i*>(lds + buf * BUF + 4 * STG + ra * 16);
        v4i af[2], wf[4];
        auto read_step = [&](int st) -> v4i {
            return *reinterpret_cast<const v4i*>(cb + (st >> 1) * STG + (((uint32_t)(2 * h + (st & 1)) ^ sw) << 4));
        };
        af[0] = read_step(0);
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            const int t = st >> 1, j = st & 1;
            if constexpr (ROWS) { if (st % 4 == 0) vw.turn(c, st / 4, wf); }
            if (st + 1 < 8) af[(st + 1) & 1] = read_step(st + 1);
            __builtin_amdgcn_sched_barrier(0);   // keeps the read ahead of this step's MFMA
            // group 4 t + 2 h + j of the superstage: byte 2 h + j of scale dword t
            const int scb = (int)(((uint32_t)sc[t] >> (16 * h + 8 * j)) & 0xffu);
            const int sca = (int)(((uint32_t)asc[t] >> (16 * h + 8 * j)) & 0xffu);
            v8i a = {}, b = {};
            const v4i w = ROWS ? wf[st & 3] : c[st];
            b[0] = w[0]; b[1] = w[1]; b[2] = w[2]; b[3] = w[3];
            a[0] = af[st & 1][0]; a[1] = af[st & 1][1]; a[2] = af[st & 1][2]; a[3] = af[st & 1][3];
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 4, 0, sca, 0, scb);
        }
    };
    // D = SETS - 1 superstages ahead.  Issue order per wavefront: A(0), W(0), .., A(D - 1), W(D - 1); then turn
    // ss issues A(ss + D), W(ss + D) - A into the LDS buffer, W into the register set that turn ss - 1
    // consumed - and computes superstage ss.  Loads return in order: at the top of turn ss everything
    // younger than W(ss) is the (D - 1) x (NA + 9) loads of the superstages after it, so waiting until at
    // most that many are outstanding means A(ss) and W(ss) have landed while D - 1 superstages stay in
    // flight across the barrier.  Every turn of the main loop issues its loads, past the end of K those of
    // the last superstage once more (into a free buffer and register set, and out of the L2), so the turns
    // are all alike; the TAIL turns after it issue none.
    constexpr int D = SETS - 1;
    if (wave >= nw) {                                   // uniform: bring a share of A, turn for turn with the others
        for (int i = 0; i < D; ++i) dma_a(min(i, nss - 1), (uint32_t)i);
        uint32_t buf = D;                               // where superstage ss + D goes
        for (int ss = 0; ss < nss - TAIL; ++ss) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((D - 1) * NA) : "memory");
            dma_a(min(ss + D, nss - 1), buf);
            buf = buf + 1 == SETS ? 0u : buf + 1;
        }
        for (int i = 0; i < TAIL; ++i) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }
    v4i c[SETS][8], s4[SETS];
#pragma unroll
    for (int i = 0; i < D; ++i) {
        dma_a(min(i, nss - 1), (uint32_t)i);
        vw.load(min(i, nss - 1), c[i], s4[i]);
    }
    // k = the turn's register set and LDS buffer (superstage mod SETS), G = superstages in flight behind it
    auto turn = [&](auto Kc, auto Gc, auto Issue, int ss) {
        constexpr int k = decltype(Kc)::value, G = decltype(Gc)::value, kn = (k + D) % SETS;
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(G * (NA + 9)) : "memory");
        // The compiler counts only the weight loads it can see, not the LDS-DMA ones: where it first needs
        // W(ss) it waits until no more loads are outstanding than the weight loads it knows to be younger.
        // Asking for W(ss) here, before this turn's loads are issued, makes that count the 9 G of the
        // superstages in flight (which also asks for their A shares, fetched from the L2 long ago); asked
        // for after this turn's loads it would be 9 more, fewer than are really outstanding, and the oldest
        // superstage in flight would have to land first.
        asm volatile("" ::"v"(c[k][0]), "v"(c[k][1]), "v"(c[k][2]), "v"(c[k][3]), "v"(c[k][4]), "v"(c[k][5]), "v"(c[k][6]),
                     "v"(c[k][7]), "v"(s4[k]));
        // (scheduling fences: without them the compiler sinks the weight loads below the turn's MFMAs and
        // lifts the next turn's scale arithmetic, which needs the youngest load, up into this one)
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(Issue)::value) {
            const int nx = min(ss + D, nss - 1);
            dma_a(nx, (uint32_t)kn);
            vw.load(nx, c[kn], s4[kn]);
        }
        __builtin_amdgcn_sched_barrier(0);
        superstage((uint32_t)k, c[k], s4[k]);
        __builtin_amdgcn_sched_barrier(0);
    };
    using Yes = std::true_type;
    using No = std::false_type;
    int ss = 0;
    for (; ss + SETS <= nss; ss += SETS)
        static_for([&](auto Kc) __attribute__((always_inline)) { turn(Kc, IC<D - 1>{}, Yes{}, ss + decltype(Kc)::value); }, IC<SETS>{});
    // TAIL superstages are left; the loads of the D - 1 after superstage ss, real or repeated, are in flight
    static_for([&](auto Kc) __attribute__((always_inline)) { turn(Kc, IC<D - 1 - decltype(Kc)::value>{}, No{}, ss + decltype(Kc)::value); }, IC<TAIL>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the repeated loads land before the LDS is released
    const int col = n0 + r;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * q + 4 * h + i;
            if (row < M && col < N) store_out(y, out_bf16, (int64_t)row * ldy + col, acc[4 * q + i]);
        }
}

// ---- M <= 16 with the online step inside (Sec. 4.3: the rotation R_4 and the quantizer in front of the
// quantized layer, here folded into the product's own prologue) ---------------------------------------
// Every workgroup first rotates (B = 32) and quantizes ALL of the activations, M <= 16 rows x K, into LDS -
// the same arithmetic as the row-wise kernels, a quad of lanes per 32-element group - in the layout the
// weight-streaming loop reads: codes [stage][16 rows][64 bytes] with the 16-byte chunks of row i XOR-swizzled
// by (i >> 2) & 3, scales [superstage][16 rows][16 bytes].  Then its first nw wavefronts stream their 32 weight rows each exactly like
// k_gemm_smallm, without any barrier (the activations never change), so the result is bit
// for bit that of brq_mxfp4_gemm on the output of brq_rotate_quantize_fused.  The first superstages of
// weights are requested before the prologue and arrive under it.  What this saves is one small launch; what
// it costs is that every one of the N / (32 nw) workgroups repeats the quantization of the same activations.
constexpr __host__ __device__ int decode_fused_operand_bytes(int64_t K) { return (int)(K / 128 * 1024 + K / 512 * 256); }
constexpr int decode_fused_lds_bytes(int64_t K, bool rows) { return decode_fused_operand_bytes(K) + turn_bytes(rows); }

template <bool IN_BF16, bool ROWS, int SETS, int TAIL>
__global__ void __launch_bounds__(256) k_gemm_decode_fused(const void* __restrict__ x, int64_t ldx, const int8_t* __restrict__ signs,
                                                           const uint8_t* __restrict__ wq, const uint8_t* __restrict__ ws,
                                                           int w_tiled, int M, int N, int K, void* __restrict__ y, int out_bf16,
                                                           int64_t ldy, int nw) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int n0 = (blockIdx.x * nw + (wave & (nw - 1))) * 32;      // (from wavefront nw on: another's rows, to no use)
    const int nss = K / 512;
    uint8_t* const scl = lds + (K / 128) * 1024;          // scales behind the codes
    const WeightRows<ROWS> vw(wq, ws, !ROWS && w_tiled, n0, N, K, lane, lds + decode_fused_operand_bytes(K) + wave * 4096);
    constexpr int D = SETS - 1;
    v4i c[SETS][8], s4[SETS];
    // ---- prologue: the online step on all M rows.  A wavefront takes 64 chunks (512 elements: one
    // superstage of one row) at a time; chunk kc of a row lies in stage kc / 16, 16-byte chunk (kc % 16) / 4.
    // Four passes' loads are issued before the first is used: a wavefront is alone on its SIMD, and nothing else would hide
    // their latency.  The first four come before the weights' loads: loads return in order, x lies in a cache and the weights
    // do not.  The next four are requested before these are worked on.  N x K = 28672 x 8192, 1 / 3 / 8 rows, us: the weights
    // first and each four by themselves 25.4 / 28.7 / 36.8, x first 25.0 / 28.4 / 36.6, now 24.0 / 27.0 / 33.5; 4096 x 4096,
    // 1 row 7.2 -> 6.2.
    {
        const uint32_t cpr = (uint32_t)K / 8u, nchunks = (uint32_t)M * cpr;
        const float sigma = (__builtin_popcount(lane & 3) & 1) ? -1.0f : 1.0f;
        const float cs = as_f32(0x3E3504F3u) * sigma;      // fl(1 / sqrt(32)), sign of the cross-lane stages folded in
        constexpr uint32_t U = 4;
        RawChunk<IN_BF16> raw[U];
        auto fetch = [&](uint32_t cb0) {
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t cb = min(cb0 + 256u * u, nchunks - 64u);      // past the end: the last pass again, not written
                const uint32_t row = cb / cpr, kc = cb - row * cpr + (uint32_t)lane;
                raw[u] = load_raw<IN_BF16>((const char*)x + ((int64_t)row * ldx + (int64_t)kc * 8) * (IN_BF16 ? 2 : 4));
            }
        };
        auto quantize = [&](uint32_t cb0) {                      // four passes; the next four are requested first
            RawChunk<IN_BF16> cur[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) cur[u] = raw[u];
            if (cb0 + 256u * U < nchunks) fetch(cb0 + 256u * U);             // uniform
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t cb = cb0 + 256u * u;
                if (cb >= nchunks) break;                                     // uniform
                const uint32_t row = cb / cpr, kc = cb - row * cpr + (uint32_t)lane;
                float v[8];
                widen<IN_BF16>(cur[u], v);
                if (signs) apply_signs(v, signs + (size_t)kc * 8);   // uniform
                wht_inwave<5>(v, (uint32_t)lane);
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] *= cs;
                const uint32_t sb = e8m0_from_amax(quad_max(absmax8(v)));
                const uint32_t w = encode8_e2m1(v, sb);
                const uint32_t st = kc >> 4, q16 = (kc >> 2) & 3u;
                *reinterpret_cast<uint32_t*>(lds + st * 1024u + row * 64u + ((q16 ^ ((row >> 2) & 3u)) << 4) + (kc & 3u) * 4u) = w;
                if ((lane & 3) == 0) scl[(kc >> 6) * 256u + row * 16u + ((kc >> 2) & 15u)] = (uint8_t)sb;
            }
        };
        fetch((uint32_t)wave * 64u);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < D; ++i) vw.load(min(i, nss - 1), c[i], s4[i]);
        __builtin_amdgcn_sched_barrier(0);
        quantize((uint32_t)wave * 64u);
        for (uint32_t cb0 = (uint32_t)wave * 64u + 256u * U; cb0 < nchunks; cb0 += 256u * U) quantize(cb0);
    }
    __syncthreads();
    if (wave >= nw) {                                     // uniform: here for the prologue
#pragma unroll
        for (int i = 0; i < D; ++i)
            asm volatile("" ::"v"(c[i][0]), "v"(c[i][1]), "v"(c[i][2]), "v"(c[i][3]), "v"(c[i][4]), "v"(c[i][5]), "v"(c[i][6]), "v"(c[i][7]), "v"(s4[i]));
        return;
    }

    v16f acc = {};
    const uint32_t ra = (uint32_t)(r & 15);               // lanes 16..31 of a half repeat rows 0..15: never stored
    const uint32_t sw = (ra >> 2) & 3u;
    auto superstage = [&](int ss, const v4i (&cw)[8], const v4i& sc) {
        const uint8_t* cbase = lds + (uint32_t)ss * 4096u + ra * 64u;
        const v4i asc = *reinterpret_cast<const v4i*>(scl + (uint32_t)ss * 256u + ra * 16u);
        v4i af[2], wf[4];
        af[0] = *reinterpret_cast<const v4i*>(cbase + (((uint32_t)(2 * h) ^ sw) << 4));
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            const int t = st >> 1, j = st & 1;
            if constexpr (ROWS) { if (st % 4 == 0) vw.turn(cw, st / 4, wf); }
            if (st + 1 < 8) af[(st + 1) & 1] = *reinterpret_cast<const v4i*>(cbase + ((st + 1) >> 1) * 1024 + (((uint32_t)(2 * h + ((st + 1) & 1)) ^ sw) << 4));
            __builtin_amdgcn_sched_barrier(0);
            const int scb = (int)(((uint32_t)sc[t] >> (16 * h + 8 * j)) & 0xffu);
            const int sca = (int)(((uint32_t)asc[t] >> (16 * h + 8 * j)) & 0xffu);
            v8i a = {}, b = {};
            const v4i w = ROWS ? wf[st & 3] : cw[st];
            b[0] = w[0]; b[1] = w[1]; b[2] = w[2]; b[3] = w[3];
            a[0] = af[st & 1][0]; a[1] = af[st & 1][1]; a[2] = af[st & 1][2]; a[3] = af[st & 1][3];
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 4, 0, sca, 0, scb);
        }
    };
    // Register sets in rotation, SETS - 1 superstages of weights in flight; the loop body is one basic block of
    // SETS turns and every load is visible to the compiler, whose wait counts are then exact.
    auto turn = [&](auto Kc, auto Issue, int ss) {
        constexpr int k = decltype(Kc)::value, kn = (k + D) % SETS;
        if constexpr (decltype(Issue)::value) vw.load(min(ss + D, nss - 1), c[kn], s4[kn]);
        __builtin_amdgcn_sched_barrier(0);
        superstage(ss, c[k], s4[k]);
        __builtin_amdgcn_sched_barrier(0);
    };
    using Yes = std::true_type;
    using No = std::false_type;
    int ss = 0;
    for (; ss + SETS <= nss; ss += SETS)
        static_for([&](auto Kc) __attribute__((always_inline)) { turn(Kc, Yes{}, ss + decltype(Kc)::value); }, IC<SETS>{});
    static_for([&](auto Kc) __attribute__((always_inline)) { turn(Kc, No{}, ss + decltype(Kc)::value); }, IC<TAIL>{});
    const int col = n0 + r;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * q + 4 * h + i;
            if (row < M && col < N) store_out(y, out_bf16, (int64_t)row * ldy + col, acc[4 * q + i]);
        }
}

// ---- measurement aid: the block-scaled fp4 MFMA back to back from registers ------------------
// 4 wavefronts per workgroup, one per SIMD, the register tile of the large-shape product kernel: 4 W
// fragments x 4 A fragments -> 16 independent 32x32 accumulators, every MFMA on another pair of fragments
// (so that the operand registers switch between consecutive instructions as they do in the product).  The
// fragments are 16 bytes per lane from `operands`: W fragment t from bytes [1024 t, 1024 t + 1024), A fragment
// t from [4096 + 1024 t, ...); scale bytes 127.  What a launch of this sustains is the ceiling of any product
// kernel on the same operand bit patterns: it includes the instruction's own issue overhead and whatever
// clock the chip holds under that load, and nothing else.
__global__ void __launch_bounds__(256, 1) k_mfma_ceiling(const uint8_t* __restrict__ operands, int iters,
                                                         float* __restrict__ sink) {
    const int lane = threadIdx.x & 63;
    v8i w8[4], a8[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const v4i w = *reinterpret_cast<const v4i*>(operands + t * 1024 + lane * 16);
        const v4i a = *reinterpret_cast<const v4i*>(operands + 4096 + t * 1024 + lane * 16);
        w8[t] = v8i{};
        a8[t] = v8i{};
        w8[t][0] = w[0]; w8[t][1] = w[1]; w8[t][2] = w[2]; w8[t][3] = w[3];
        a8[t][0] = a[0]; a8[t][1] = a[1]; a8[t][2] = a[2]; a8[t][3] = a[3];
    }
    v16f acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = v16f{};
    // Shader-clock cycles and 100 MHz reference ticks around the loop give the clock the chip held.
    // The loop bound passes through an asm statement after the first pair of timestamps and the
    // accumulators' sum through one before the second, so the loop cannot move across either.
    const uint64_t c0 = __builtin_readcyclecounter(), r0 = __builtin_amdgcn_s_memrealtime();
    asm volatile("" : "+s"(iters) : "s"(c0), "s"(r0));
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8[i >> 2], a8[i & 3], acc[i], 4, 4, 0, 127, 0, 127);
    }
    float t = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) t += acc[i][j];
    asm volatile("" : "+v"(t));
    const uint64_t c1 = __builtin_readcyclecounter(), r1 = __builtin_amdgcn_s_memrealtime();
    if (blockIdx.x == 0 && threadIdx.x < 2) t = (float)(threadIdx.x == 0 ? c1 - c0 : r1 - r0);
    sink[blockIdx.x * 256 + threadIdx.x] = t;
}

hipError_t launch_mfma_ceiling(const uint8_t* operands, int iters, int workgroups, float* sink, hipStream_t s) {
    hipLaunchKernelGGL(k_mfma_ceiling, dim3(workgroups), dim3(256), 0, s, operands, iters, sink);
    return hipGetLastError();
}

using SmallmKern = void (*)(const uint8_t*, const uint8_t*, int, const uint8_t*, const uint8_t*, int, int, int, void*, int, int64_t, int);
constexpr int FEW = 3, MANY = 5;      // register sets
#define BRQ_FEW(ROWS) {k_gemm_smallm<ROWS, FEW, 0>, k_gemm_smallm<ROWS, FEW, 1>, k_gemm_smallm<ROWS, FEW, 2>}
#define BRQ_MANY(ROWS) {k_gemm_smallm<ROWS, MANY, 0>, k_gemm_smallm<ROWS, MANY, 1>, k_gemm_smallm<ROWS, MANY, 2>, k_gemm_smallm<ROWS, MANY, 3>, \
                        k_gemm_smallm<ROWS, MANY, 4>}
static const SmallmKern smallm_few[2][FEW] = {BRQ_FEW(false), BRQ_FEW(true)};          // [weights row-major][K / 512 % sets]
static const SmallmKern smallm_many[2][MANY] = {BRQ_MANY(false), BRQ_MANY(true)};
#undef BRQ_FEW
#undef BRQ_MANY
using DecodeKern = void (*)(const void*, int64_t, const int8_t*, const uint8_t*, const uint8_t*, int, int, int, int, void*, int, int64_t, int);
#define BRQ_DECODE(BF16, ROWS) {k_gemm_decode_fused<BF16, ROWS, FEW, 0>, k_gemm_decode_fused<BF16, ROWS, FEW, 1>, k_gemm_decode_fused<BF16, ROWS, FEW, 2>}
static const DecodeKern decode_kern[2][2][FEW] = {{BRQ_DECODE(false, false), BRQ_DECODE(false, true)},   // [x bf16][row-major weights turned round]
                                                  {BRQ_DECODE(true, false), BRQ_DECODE(true, true)}};
#undef BRQ_DECODE

// Wavefronts of a streaming workgroup that own columns, 32 each: as many as still leave every compute unit a workgroup. A
// CU's address path takes the four wavefronts' weight loads one after the other (half lines, 32 cycles each: 1150 cycles per
// superstage for 264 of MFMA), so columns on other CUs are faster than columns on the same.  With one wavefront a CU more
// superstages in flight help too.  us, weights in no cache, 1 row, four wavefronts and 3 sets -> now: N x K = 2048 x 8192
// 14.5 -> 7.3 (3 sets 8.9), 8192 x 8192 15.8 -> 10.0, 500 x 16384 20.9 -> 10.7, 4096 x 4096 9.3 -> 5.9, 300 x 2048 5.3 ->
// 3.4; 14336 x 4096 (two wavefronts; 5 sets 8.5) 9.9 -> 8.2; 28672 x 8192 (four; two 23.3, with 16 rows 24.7 for 24.0) 23.6
// -> 23.5. The one-launch call, whose workgroups all quantize x, stays at 3 sets: 2048 x 8192 16.6 -> 9.8 (5 sets 10.4),
// 14336 x 4096 11.2 -> 9.7.
static int streaming_waves(int64_t N, int cus) { return N <= (int64_t)32 * cus ? 1 : N <= (int64_t)64 * cus ? 2 : 4; }

hipError_t setup_gemm_decode_fused() {
    for (const auto& in : decode_kern)
        for (int rows = 0; rows < 2; ++rows)
            for (DecodeKern k : in[rows])
                if (hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, decode_fused_lds_bytes(DECODE_FUSED_MAX_K, rows));
                    e != hipSuccess) return e;
    return hipSuccess;
}

hipError_t launch_gemm_decode_fused(const void* x, bool in_bf16, int64_t M, int64_t K, int64_t ldx, const int8_t* signs,
                                    const Operand& w, int64_t N, void* y, bool out_bf16, int64_t ldy, hipStream_t s) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
    const int nw = streaming_waves(N, cus);
    // Up to 32 columns no other wavefront's lines push a row-major line out between its quarters, and turning it round is only in the
    // way: fragments.  us, whole lines -> fragments: 1 row, 5 x 4096 5.4 -> 4.7, 2 rows, 3 x 9216 10.8 -> 9.4, 8 rows, 8 x 4096 10.1 -> 9.3 (111 shapes
    // 5 % faster); of 33 to 128 columns (31 shapes) whole lines are 6 % faster.
    const bool turned = !w.tiled && N > 32;
    hipLaunchKernelGGL(decode_kern[in_bf16][turned][K / 512 % FEW], dim3((uint32_t)((N + 32 * nw - 1) / (32 * nw))), dim3(256),
                       decode_fused_lds_bytes(K, turned), s, x, ldx, signs, w.codes, w.scales, (int)w.tiled, (int)M, (int)N, (int)K, y, (int)out_bf16, ldy, nw);
    return hipGetLastError();
}

// ---- which LDS-staged kernel and output tile -------------------------------------------------
// The candidates: the persistent kernel with its 256 x 256 and 128 x 256 tiles, and the one-tile-per-workgroup
// kernel's family.  They are told apart by an estimate of the time, in microseconds:
//     fixed + |stages * alone * ceil(tiles / places), stages * full * tiles / CUs * filled, bytes / 5 TB/s|_4 + store * output
// `alone`: a stage of a tile while the chip is not full (the issue, load and LDS bound of one workgroup, at the
// full clock); `full`: a stage's share of a chip full of them, which is what its energy costs (the chip holds 1.6
// to 1.8 GHz of 2.4 with every CU multiplying); places = CUs x workgroups that fit one; filled: rows past M
// are zeros in the one-tile kernel and cost half; bytes: both operands, from HBM; output: 0.6 us per MB of bf16, by
// whether its rows begin on 128-byte lines, by pitch and by address (outputs 32 or 64 bytes off a line, over the best of the seven
// where only the pitch was asked -> now: row-major 1.0 -> 0.3 %, tiled 4.0 -> 3.5, 40 shapes each).  Rows on half lines count
// as off, though the one-tile kernels store them as those on lines: as on lines for these, tiled 2.7 -> 1.9 %, but row-major 0.2 ->
// 1.4, 36 shapes each.  The three bounds blend into each other (4-norm).  The constants are fitted to
// the candidates' times, weights not in any cache, on 147 tiled and 160 row-major shapes (M 10 .. 8192, N 256 .. 28672 in
// eights, K 512 .. 13824): the choice cost 0.9 % over the best of the seven on average, row-major 0.5 % (15 % and 27 % at
// worst); the fit to the kernels before them (row-major stages by themselves, every row stored past the L2) cost 4 % (67 %).
// Two changes to the one-tile kernels came after the fit (six stages of both operands in 64 x 128 row-major, the hint on half
// lines); with them, on 64 other shapes of each layout, a quarter each on lines, half lines, 16 bytes and anywhere, it is 1.6 /
// 2.9 / 1.0 / 0.9 % tiled and 0.2 / 0.1 / 0.3 / 0.3 % row-major (22 % and 4 % at worst; tiled 3234 x 5040 x 1536 25.6 -> 26.4 us
// since the table before).  `singles`, row-major with K up to 1024, is fitted to 1839 shapes (M 1 .. 8192, N 64 .. 28672): 0.8 %
// over the best (34 % at worst); fitted to one half 0.9 % on the other.
struct TileCost { float fixed, alone, full, store, store_off; int per_cu; };    // store_off: rows off lines
struct Tile { int na, mb, route; TileCost tiled, rowmajor, singles; };          // 64 mb x 64 na; singles: row-major by single stages
static const Tile TILES[] = {
    {4, 4, ROUTE_256x256, {5.984f, 0.535f, 0.758f, 0.292f, 0.481f, 1}, {6.801f, 0.508f, 0.978f, 0.439f, 0.893f, 1}, {}},
    {4, 2, ROUTE_128x256, {3.696f, 0.280f, 0.474f, 0.377f, 0.649f, 1}, {3.535f, 0.514f, 0.682f, 0.402f, 0.724f, 1}, {}},
    {2, 1, ROUTE_ONE_TILE, {3.141f, 0.178f, 0.205f, 0.406f, 0.923f, 2}, {3.749f, 0.196f, 0.264f, 0.512f, 0.585f, 2},
     {3.382f, 0.118f, 0.348f, 0.442f, 0.597f, 2}},
    {2, 2, ROUTE_ONE_TILE + 1, {3.731f, 0.206f, 0.292f, 0.348f, 0.560f, 2}, {3.585f, 0.261f, 0.356f, 0.889f, 1.014f, 1},
     {3.958f, 0.267f, 0.356f, 0.307f, 0.489f, 2}},
    {2, 3, ROUTE_ONE_TILE + 2, {4.774f, 0.268f, 0.313f, 0.568f, 1.091f, 1}, {5.290f, 0.268f, 0.433f, 0.736f, 1.070f, 1},
     {3.629f, 0.362f, 0.359f, 0.619f, 0.950f, 1}},
    {4, 3, ROUTE_ONE_TILE + 3, {6.545f, 0.397f, 0.552f, 0.422f, 0.864f, 1}, {5.012f, 0.522f, 0.751f, 0.529f, 1.038f, 1}, {}},
    {2, 5, ROUTE_ONE_TILE + 4, {6.659f, 0.363f, 0.494f, 0.545f, 0.950f, 1}, {6.735f, 0.399f, 0.639f, 0.624f, 0.976f, 1}, {}},
};

// The cheapest of these that take the shape, or -1.  (The one-tile kernels' sixth tile is not among them: see tall_tile.)
static int pick_tile(const GemmShape& g, int cus) {
    const bool tiled = g.a_tiled && g.w_tiled;
    const float stages = (float)((g.K + 511) / 512 * 4), output = 0.6e-6f * (float)g.M * (float)g.N * (g.out_bf16 ? 1.0f : 2.0f);
    const float bytes = 0.53125f * ((float)g.M + (float)g.N) * (float)g.K / 5.0e6f;
    const bool lines = g.N * (g.out_bf16 ? 2 : 4) % 16 == 0 && rows_on(128, g.y, g.ldy * (g.out_bf16 ? 2 : 4));
    auto pow4 = [](float x) { return x * x * x * x; };
    int best = -1;
    float least = 0.0f;
    for (const Tile& t : TILES) {
        if (!gemm_route_supported(t.route, g)) continue;
        const bool one_tile = t.route >= ROUTE_ONE_TILE;
        const TileCost& c = tiled ? t.tiled : one_tile && !mid_gemm_pairs(t.route - ROUTE_ONE_TILE, tiled, g.K) ? t.singles : t.rowmajor;
        const int64_t tm = (g.M + 64 * t.mb - 1) / (64 * t.mb), T = tm * ((g.N + 64 * t.na - 1) / (64 * t.na)), places = (int64_t)cus * c.per_cu;
        const float filled = one_tile ? 0.5f + 0.5f * (float)g.M / (float)(64 * t.mb * tm) : 1.0f;
        const float alone = stages * c.alone * (float)((T + places - 1) / places);
        const float full = stages * c.full * (float)T / (float)cus * filled;
        const float cost = c.fixed + sqrtf(sqrtf(pow4(alone) + pow4(full) + pow4(bytes))) + (lines ? c.store : c.store_off) * output;
        if (best < 0 || cost < least) { best = t.route; least = cost; }
    }
    return best;
}

bool gemm_route_supported(int route, const GemmShape& g) {
    switch (route) {
        case ROUTE_GENERAL: return true;
        case ROUTE_SKINNY: return g.M <= 16;
        case ROUTE_STREAM: return g.M <= 16 && g.whole_k() && g.padded_k() < (int64_t(1) << 26);
        case ROUTE_256x256:
        case ROUTE_128x256: return tiled_gemm_supported(g.M, g.N, g.K, g.out_bf16, g.ldy, g.a_tiled && g.w_tiled);
        case ROUTE_ANY_K: return g.K >= 256;
        default: return route >= ROUTE_ONE_TILE && route < ROUTE_ANY_K && mid_gemm_supported(route - ROUTE_ONE_TILE, g);
    }
}

// Where the estimate takes 320 x 128 or 192 x 256: whether tiles of 256 x 128 go round the chip as often.  Then each is that
// much shorter and nothing is lost.  Row-major, on all of 133 such shapes (of 2029: M 100 .. 8192, N 512 .. 28672 in eights, K
// 1152 .. 13824, weights in no cache) faster by 3 to 23 %, 11 % on average; with a round more slower on 94 % (17 % on average).
// us: 2000 x 4096 x 11008 fp32 59.1 -> 56.5, 250 x 28672 x 8192 48.0 -> 45.4, 1000 x 8192 x 4096 27.2 -> 23.3, 4642 x 2744 x 8064
// 92.3 -> 80.3.  Tiled, over 320 x 128, 830 shapes, K from 2304: 1 % slower to 14 % faster, 6.5 % on average (6046 x 2568 x 8192 76.8 ->
// 72.1); over 192 x 256 in two rounds and more, 127 shapes, faster by 2 to 16 %, in one round not always (3776 x 2080 x 4224 fp32 26.0 :
// 28.6).  K below was not looked at.  Same order of summation, same bits.
constexpr int TALL_TILE = ROUTE_ONE_TILE + 5;
static bool tall_tile(int route, const GemmShape& g, int cus) {
    constexpr int TILE_192x256 = ROUTE_ONE_TILE + 3, TILE_320x128 = ROUTE_ONE_TILE + 4;
    const bool tiled = g.a_tiled && g.w_tiled;
    if ((route != TILE_192x256 && route != TILE_320x128) || g.K <= (tiled ? 2048 : 1024)) return false;
    auto rounds = [&](int64_t tm, int64_t tn) { return ((g.M + tm - 1) / tm * ((g.N + tn - 1) / tn) + cus - 1) / cus; };
    const int64_t n = rounds(256, 128);
    return n == (route == TILE_192x256 ? rounds(192, 256) : rounds(320, 128)) && !(tiled && route == TILE_192x256 && n == 1);
}

// What no staged kernel takes: through LDS (k_gemm_any_k) from where its pairs of stages have something to hide behind.  Up to 64 rows
// that is enough of them or enough tiles; above, enough of them or enough tiles of 32 x 32, of which k_gemm_direct's wavefronts have
// one each (counted in tiles of 128 x 128 a few columns pass for many).  k_gemm_any_k's time over k_gemm_direct's, 1002 shapes of
// more than 64 rows, weights in no cache / in the L2, by tiles of 32 x 32 and K, on either side of the line: 256 x 2500 0.89 / 1.28,
// 256 x 5000 0.66 / 0.93; 512 x 1700 0.83 / 1.19, 512 x 2400 0.74 / 0.85; 1024 x 860 0.90 / 0.97, 1024 x 1200 0.73 / 0.85; 4096 x 300
// 0.85 / 0.90; K from 4096 below the line 0.71 / 1.07.  us, either kernel, weights in the L2: 15897 x 2 x 672 4.9 : 7.6, 4182 x 5 x 3872 14.0 :
// 17.5, 141 x 5692 x 1088 7.4 : 9.3; in no cache 2000 x 4096 x 10976 656 : 88, 128 x 2048 x 10976 84 : 43, 1000 x 8192 x 544 21.3 : 11.9.  Of
// 64 rows (198 shapes, none slower beyond the line) 64 x 1024 x 1056 6.8 : 6.8, 64 x 1024 x 2080 12.0 : 9.0, 64 x 16384 x 544 6.9 : 6.7.
static bool any_k(const GemmShape& g) {
    if (g.K < 256) return false;
    if (g.M <= 64) return g.K >= 2048 || (g.N + 127) / 128 * g.K >= 65536;
    return g.K >= 4096 || (double)((g.M + 31) / 32) * (double)((g.N + 31) / 32) * (double)g.K >= (double)(1 << 20);
}

int gemm_route(const GemmShape& g, int cus) {
    // Up to 16 rows: the weights are streamed (k_gemm_smallm).  The staged 64 x 128 kernel and the K-split one (ROUTE_SKINNY, which
    // sums in another order) against it, us, weights in no cache, 1 / 16 rows, streaming : 64 x 128 : K-split:
    //   weights tiled      N x K = 256 x 512 2.4 / 2.8 : 3.5 / 3.6 : 2.0 / 2.4,  2048 x 2048 4.0 / 4.3 : 5.9 / 5.9 : 3.8 / 4.2,
    //                      2048 x 8192 7.4 / 7.9 : 13.9 / 14.7 : 11.7 / 12.0,  8192 x 4096 7.3 / 7.6 : 9.4 / 9.7 : 8.0 / 8.3,
    //                      28672 x 2048 8.7 / 9.0 : 8.7 / 8.7 : 9.1 / 10.4,  28672 x 8192 24.9 / 25.3 : 25.5 / 25.8 : 30.6 / 33.3
    //   weights row-major  64 x 512 2.4 / 2.7 : 3.5 / 3.5,  28672 x 512 4.6 / 5.0 : 5.2 / 5.2 : 4.3 / 5.3,  28672 x 1024 6.4 / 6.8 :
    //                      6.6 / 6.7 : 6.8 / 8.1,  28672 x 2048 9.1 / 9.6 : 9.7 / 9.9 : 11.4 / 13.1,  28672 x 8192 30.5 / 31.1 : 31.2 /
    //                      31.3 : 38.0 / 42.8,  2048 x 8192 8.7 / 9.1 : 18.6 / 19.2 : 12.6 / 13.0,  14336 x 4096 9.3 / 9.8 : 12.4 / 12.9
    if (gemm_route_supported(ROUTE_STREAM, g)) return ROUTE_STREAM;
    const int t = g.M > 16 || g.K % 512 == 0 ? pick_tile(g, cus) : -1;
    if (tall_tile(t, g, cus)) return TALL_TILE;
    return t >= 0 ? t : g.M <= 16 ? ROUTE_SKINNY : any_k(g) ? ROUTE_ANY_K : ROUTE_GENERAL;
}

hipError_t launch_gemm_route(int route, const Operand& a, const Operand& w, const GemmShape& g, void* y, hipStream_t s) {
    const int64_t M = g.M, N = g.N, K = g.K;
    switch (route) {
        case ROUTE_GENERAL:
            hipLaunchKernelGGL(k_gemm_direct, dim3((uint32_t)((N + 63) / 64), (uint32_t)((M + 63) / 64)), dim3(256), 0, s, a.codes, a.scales,
                               (int)a.tiled, w.codes, w.scales, (int)w.tiled, (int)M, (int)N, (int)K, y, (int)g.out_bf16, g.ldy);
            return hipGetLastError();
        case ROUTE_ANY_K: return launch_gemm_any_k(a, w, M, N, K, y, g.out_bf16, g.ldy, s);
        case ROUTE_SKINNY:
            hipLaunchKernelGGL(k_gemm_skinny, dim3((uint32_t)((N + 15) / 16)), dim3(256), 0, s, a.codes, a.scales, (int)a.tiled, w.codes,
                               w.scales, (int)w.tiled, (int)M, (int)N, (int)K, y, (int)g.out_bf16, g.ldy);
            return hipGetLastError();
        case ROUTE_STREAM: {
            int cus = 0;
            if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
            const int64_t nss = g.padded_k() / 512;
            const int nw = streaming_waves(N, cus), sets = nw == 1 && nss >= MANY ? MANY : FEW;
            const SmallmKern* const kern = sets == MANY ? smallm_many[!w.tiled] : smallm_few[!w.tiled];
            hipLaunchKernelGGL(kern[nss % sets], dim3((uint32_t)((N + 32 * nw - 1) / (32 * nw))), dim3(256), smallm_lds_bytes(sets, !w.tiled),
                               s, a.codes, a.scales, (int)a.tiled, w.codes, w.scales, (int)M, (int)N, (int)K, y, (int)g.out_bf16, g.ldy, nw);
            return hipGetLastError();
        }
        case ROUTE_256x256:
        case ROUTE_128x256: return launch_gemm_tiled(a, w, M, N, K, y, g.out_bf16, g.ldy, s, route == ROUTE_128x256);
        default: return launch_gemm_mid(route - ROUTE_ONE_TILE, a, w, M, N, K, y, g.out_bf16, g.ldy, s);
    }
}

hipError_t launch_mxfp4_gemm(const Operand& a, const Operand& w, const GemmShape& g, void* y, hipStream_t s) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;      // (also the per-device kernel set-up)
    return launch_gemm_route(gemm_route(g, cus), a, w, g, y, s);
}

}  // namespace brq
