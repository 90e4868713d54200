// Medium-shape W4A4 MXFP4 product for gfx950: one output tile per workgroup, the tile chosen from a family
// (64 MB rows x 64 NA columns) so that the shape fills the chip (the product of Sec. 2 on the MXFP4 operands
// of Sec. 4.1; which tile takes a shape: gemm_route).  The persistent 256 x 256 kernel is the better one where there are many tiles; here are the
// shapes in between: a chunk of a prompt, a few hundred rows against wide weights, a projection with few columns.
//
// Workgroup = 4 wavefronts (2 x 2), each with NA x MB MFMA tiles of 32 x 32.  As in the persistent kernel the
// weights are the MFMA's row operand, K is consumed in stages of 128 elements, within a stage lane half h owns
// groups 2h and 2h + 1, and operands travel HBM -> LDS by LDS-DMA into a ring of D stages whose 64-byte rows
// have their 16-byte chunks XOR-swizzled by (row >> 2) & 3.
//
// What differs is the fragment schedule.  A stage of these tiles is 4 to 24 MFMAs (130 to 800 cycles) long,
// too short to hide an LDS read between its barrier and its use.  The register file has room (32 to 192
// accumulators of 512 registers), so ALL fragments of stage t + 1 are read while stage t multiplies:
//   start of stage t   stage t + 1 has landed, everyone's reads of stage t's buffer are done: one barrier
//   during stage t     2 (NA + MB) fragment reads of stage t + 1, the loads of stage t + D into stage t's
//                      buffer, and the MFMAs of stage t from registers filled a stage ago.
// Nothing between the barrier and the MFMAs waits for LDS.
//
// K: whole superstages of 4 stages.  Tiled operands are zero-padded to that.  Row-major operands with
// K % 512 != 0 (K % 128 == 0, K >= 512) take as their last superstage the window [K - 512, K): every load is in
// bounds, and the stages that the window shares with the superstage before get scale bytes 0 in BOTH operands
// (2^-127 * 2^-127 times at most 36 * 32 vanishes in an fp32 sum).
//
// Pairs (PAIR: an operand is row-major; mid_gemm_pairs).  A stage of a row-major operand is half of a 128-byte line of every row.  Taken
// stage by stage each line crosses from the L2 to the CU twice, and from HBM its halves come at two times: with
// 128 x 128 tiles 1000 x 4096 x 11008 ran at 936 cycles a stage (681 with W in the memory-side cache), tiled operands at 490.
// So two stages are loaded as one: 8 rows x 128 bytes per load, 128-byte rows in LDS, chunk c of row i at c ^ ((i >> 1) & 7)
// (16 rows of one chunk then cover all banks).  A slot of the ring is free once the second of its stages has been read,
// in the first half of that stage, so loads are issued in the odd stages: A's first, then W's.  W comes from HBM and
// A from the L2 or the memory-side cache, where the quantizer has just left it, and loads complete in order: behind
// A's they have two stages more to arrive (DW > DA), where the LDS has no room for as many of both.
// Cycles a stage and us, row-major, weights in no cache, before -> now: 1000 x 4096 x 11008 936 -> 705, 41.2 -> 35.7; 300 x
// 28672 x 8192 (320 x 128) 1340 -> 1046, 57.6 -> 50.9; 2000 x 4096 x 11008 1200 -> 1010, 67 -> 58; 1000 x 4096 x 11008 on 64 x 128
// 56 -> 45.  What is left over tiled operands is the order in which HBM is read (hot: 495 cycles).
// Both kinds take either layout; tiled operands keep single stages (4 of them in LDS twice a CU: 29.5 against 30.4 us).
// So do row-major ones with K up to 1024 on the tiles of at most 192 x 128: there the prologue, which loads all the stages there
// are, and two workgroups a CU weigh more than whole lines.  Pairs : single stages, us: 128 x 128 2000 x 4096 x 512 10.4 : 7.3, 4000
// x 8192 x 512 35.4 : 23.5, 2000 x 4096 x 1024 11.9 : 10.2; 192 x 128 134 x 64 x 1024 6.9 : 6.2; 64 x 128 16 x 2048 x 512 4.1 : 3.9, 16 x
// 2048 x 1024 5.0 : 4.7; with K = 2048 64 x 128 2000 x 4096 17.0 : 18.7, 128 x 128 514 x 16064 23.9 : 22.5 but 100 x 8192 x 3072 13.1 :
// 14.7; 320 x 128 2000 x 4096 x 1024 10.4 : 10.9, 192 x 256 10.8 : 11.1.
//
// What bounds a stage where one workgroup runs on a CU is what the CU can have on its way: an L2 hit costs it 16 cycles a KB, but of
// what misses the L2 at most 32 KB (the L1's size) are in flight, some 1000 cycles each, and hits wait behind misses; deeper
// rings, other orders and wavefronts that only load change nothing or hand the cycles back to the clock (300 x 28672 x 8192: the
// loads of a stage by themselves 34 us, the product 43).
//
// LDS map (bytes), S = NA + MB: W's DW stages x 4K NA | A's DA stages x 4K MB; then ceil(DW / 4) scale buffers x
// (W 1K NA | A 1K MB), 16 scale bytes (one superstage) per row.  The output is turned round in the rings.
//
// DW, DA: as many stages as the LDS takes where that measured faster.  Single stages: two workgroups of 64 x 128 on a CU with
// 6 stages each instead of 4: 200 x 4096 x 4096 11.2 -> 9.7 us, 300 x 28672 x 8192 75 -> 68.  The other tiles gain nothing
// from depth (128 x 128 with 8 stages and one workgroup a CU instead of 4 and two: 58 -> 65 us on the latter); 320 x 128, for
// a few hundred rows, has 5 and reads its weights once: 47.6 -> 44.8 us on the latter.  Pairs: 4 stages of both wait for
// every load (128 x 128: 1082 cycles a stage, 6 of both 705, 8 the same); 64 x 128 with 6 and 4 instead of 6 of both, 1000 x
// 4096 x 11008 45.1 us against 47.0, but 1 x 936 x 8192 13.4 against 12.9, 200 x 4096 x 4096 12.0 against 11.8: it is for the
// small shapes.
#include "mfma_fp4.h"
#include "brq_launch.h"

namespace brq {
namespace mid {

// DW and DA code stages of W and A, and the scales of every superstage that has a stage among W's
constexpr int scale_bufs(int DW) { return (DW + 3) / 4; }
constexpr int lds_bytes(int NA, int MB, int DW, int DA) { return 4096 * (NA * DW + MB * DA) + scale_bufs(DW) * 1024 * (NA + MB); }

// lines: the output's rows begin on half lines of 64 bytes, and the streaming hint goes with every store.  Where they do not,
// a store of 128 bytes is the end of one line and the beginning of the next, in pieces of 16 or 32 bytes more or less: with
// the hint such pieces go to memory as they are, without it the L2 puts the line together.  (Halves of lines it had better
// not wait for: 1668 x 1072 x 7680 fp32 14.2 us with the hint, 14.8 without, 3234 x 5040 x 1536 fp32 25.8, 27.3.)  Rows that
// are not 16-byte aligned are stored in the same way (the memory system takes any alignment); only a row's last N % (16 /
// sizeof(out)) elements go one by one.  128 x 128, us, before -> now: 600 x 6004 x 4096 bf16 (rows on 8 bytes, element by
// element before) 18.9 -> 13.5, fp32 (the hint before) 17.1 -> 14.7; 600 x 6016 x 4096 12.7.
// The output of a workgroup's tile, 64 MB rows from m0 on and 64 NA columns from n0 on.  `lds`: 16 KB that nobody reads any more.
template <bool OUT_BF16, int NA, int MB>
__device__ __forceinline__ void store_tile(v16f (&acc)[NA][MB], uint8_t* lds, void* y, int64_t ldy, int64_t m0, int64_t n0, int M, int N, int lines) {
    constexpr int NM = NA * MB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31, h = lane >> 5, wn = wave >> 1, wm = wave & 1;
    // The accumulators were last written by MFMAs hidden in inline assembly: the compiler does not
    // know to keep the wait states between a 16-pass MFMA and a read of its result.  Each wavefront turns its
    // 32-row x 128-byte blocks round in 4 KB of the ring (whose last reads are behind the last barrier):
    // chunk c of row i at i * 128 + ((c ^ (i & 7)) << 4), stored as 8 rows x 128 contiguous bytes.
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    constexpr int ES = OUT_BF16 ? 2 : 4, EPC = 16 / ES, XPB = OUT_BF16 ? 2 : 1;
    const int64_t pitch = ldy * ES;
    uint8_t* const ebuf = lds + wave * 4096;
    uint8_t* const ytile = reinterpret_cast<uint8_t*>(y) + (m0 + wm * 32 * MB) * pitch + (n0 + wn * 32 * NA) * ES;
    uint8_t* const ewr = ebuf + r * 128;
    const uint32_t wsw = (uint32_t)((r & 7) ^ h) << 4;
    const uint8_t* const erd = ebuf + (lane >> 3) * 128 + (((lane & 7) ^ ((lane >> 3) & 7)) << 4);
    const int64_t mrem = M - m0 - wm * 32 * MB - (lane >> 3), nrem = N - n0 - wn * 32 * NA - (lane & 7) * EPC;
    static_for([&](auto Xc) __attribute__((always_inline)) {
        constexpr int X = decltype(Xc)::value, A = PairA<X, MB>::value, B = PairB<X, MB>::value;
        float c[16];
        read_acc8(acc[A][B], IC<0>{}, c);
        read_acc8(acc[A][B], IC<8>{}, c);
        if constexpr (OUT_BF16) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const uint32_t x0 = pack_bf16x2(c[8 * p + 0], c[8 * p + 1]), x1 = pack_bf16x2(c[8 * p + 2], c[8 * p + 3]);
                const uint32_t y0 = pack_bf16x2(c[8 * p + 4], c[8 * p + 5]), y1 = pack_bf16x2(c[8 * p + 6], c[8 * p + 7]);
                const auto s0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
                *reinterpret_cast<uint4*>(ewr + (wsw ^ (uint32_t)(((A & 1) * 4 + 2 * p) << 4))) = make_uint4(s0[0], s1[0], s0[1], s1[1]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(ewr + (wsw ^ (uint32_t)(q << 5))) = make_float4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
        }
        if constexpr (X % XPB == XPB - 1) {
            constexpr int row = B * 32, colbytes = (OUT_BF16 ? A / 2 : A) * 128;
            uint8_t* const dst = ytile + (row + (lane >> 3)) * pitch + colbytes + (lane & 7) * 16;
            const int64_t cols = nrem - colbytes / ES;          // columns left from this lane's chunk on
            typedef unsigned int u4 __attribute__((ext_vector_type(4)));
            u4 ob[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) ob[j] = *reinterpret_cast<const u4*>(erd + j * 1024);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (row + 8 * j < mrem && cols > 0) {
                    if (lines) {                                // uniform
                        __builtin_nontemporal_store(ob[j], reinterpret_cast<u4*>(dst + 8 * j * pitch));
                    } else if (cols >= EPC) {
                        typedef unsigned int u4_any __attribute__((ext_vector_type(4), aligned(2)));
                        *reinterpret_cast<u4_any*>(dst + 8 * j * pitch) = ob[j];
                    } else {
#pragma unroll
                        for (int e = 0; e < EPC; ++e)
                            if (e < cols) {
                                if constexpr (OUT_BF16) reinterpret_cast<uint16_t*>(dst + 8 * j * pitch)[e] = (uint16_t)(ob[j][e >> 1] >> (16 * (e & 1)));
                                else reinterpret_cast<uint32_t*>(dst + 8 * j * pitch)[e] = ob[j][e];
                            }
                    }
                }
        }
    }, IC<NM>{});
}

// DW == DA unless PAIR.
template <bool OUT_BF16, int NA, int MB, int DW, int DA, bool PAIR>
__global__ void __launch_bounds__(256, (lds_bytes(NA, MB, DW, DA) <= 81920 ? 2 : 1))
k_gemm_mid(const uint8_t* __restrict__ aq, const uint8_t* __restrict__ as, const uint8_t* __restrict__ wq,
           const uint8_t* __restrict__ ws, int M, int N, int K, void* __restrict__ y, int64_t ldy, int a_tiled,
           int w_tiled, int lines) {
    constexpr int S = NA + MB, NM = NA * MB, NS = 2 * NM;      // MFMAs per step and per stage
    constexpr int TM = 64 * MB, TN = 64 * NA, G = PAIR ? 2 : 1;       // G: stages per slot of the rings
    constexpr int WSLOT = 4096 * NA * G, ASLOT = 4096 * MB * G, ABASE = 4096 * NA * DW;
    constexpr int NSB = scale_bufs(DW), SCALE_BASE = ABASE + 4096 * MB * DA, SCALE_BUF = 1024 * S;
    constexpr int PW = DW / 2, PA = DA / 2;                    // pairs: how far ahead of the one that is read they are loaded
    static_assert(PAIR ? DW % 2 == 0 && DA % 2 == 0 && PW >= PA && PA >= 2 : DW == DA, "");
    constexpr int SPW = (S + 3) / 4;                           // scale loads per wavefront and superstage
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    load_args(aq, as, wq, ws, M, N, K, a_tiled, w_tiled);
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int wn = wave >> 1, wm = wave & 1;

    TileWalk tw;
    tw.tiles_m = (M + TM - 1) / TM;
    tw.tiles_n = (N + TN - 1) / TN;
    {
        const int T = tw.tiles_m * tw.tiles_n, per_xcd = (T + 7) / 8;
        tw.first = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
        tw.end = min(((int)(blockIdx.x & 7) + 1) * per_xcd, T);
        tw.stride = 1;
    }
    if (tw.first >= tw.end) return;                            // uniform over the workgroup
    int tm, tn;
    tw.tile(0, tm, tn);
    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * TN;
    const int KQ = (K + 511) / 512;
    const int64_t Kp = (int64_t)KQ * 512;
    const int ovd = (K == Kp || w_tiled) ? 0 : (int)((Kp - K) / 128);   // stages the last window shares with the one before

    // ---- loads.  A wavefront brings 16 NA rows of W and 16 MB rows of A per stage, 16 rows x 64 bytes per
    // instruction (lane i: chunk (i & 3) ^ ((i >> 4) & 3) of row i >> 2), or 8 rows x 128 bytes of a pair, and its share of the scale rows, 64
    // rows x 16 bytes per instruction, once per superstage (wavefronts without a share repeat the last one, so that
    // all count the same).  Every per-lane offset is relative to one uniform base per operand that moves along
    // K; rows past the last one are clamped to it and never stored.
    const int lrow = PAIR ? lane >> 3 : lane >> 2;             // this lane's row of the 16 / G that a load brings
    auto code_off = [&](int64_t row, int q, int64_t rows, bool tiled) -> uint32_t {
        row = min(row + lrow, rows - 1);
        const uint32_t c = PAIR ? (uint32_t)((lane & 7) ^ ((q & 1) * 4 + (lane >> 4))) : (uint32_t)((lane & 3) ^ ((lane >> 4) & 3));
        return tiled ? (uint32_t)((row >> 6) * (Kp / 128) * 4096 + (row & 63) * 64) + (c & 3) * 16 + (c >> 2) * 4096
                     : (uint32_t)(row * (K / 2)) + c * 16;
    };
    auto scale_off = [&](int64_t row, int64_t rows, bool tiled) -> uint32_t {
        row = min(row, rows - 1);
        return tiled ? (uint32_t)((row >> 6) * (Kp / 512) * 1024 + (row & 63) * 16) : (uint32_t)(row * (K / 32));
    };
    // (bases moved to the tile's first row, so that the offsets stay below 2^32 for any M and N)
    const int64_t wslab = n0 >> 6, aslab = m0 >> 6;            // TM and TN are multiples of 64
    const uint8_t* const wbase = uniform_ptr(wq + (w_tiled ? wslab * (Kp / 128) * 4096 : n0 * (K / 2)));
    const uint8_t* const abase = uniform_ptr(aq + (a_tiled ? aslab * (Kp / 128) * 4096 : m0 * (K / 2)));
    const int64_t nrows = N - n0, mrows = M - m0;
    uint32_t vw[G * NA], va[G * MB], vsc[SPW];
#pragma unroll
    for (int q = 0; q < G * NA; ++q) vw[q] = code_off(wave * 16 * NA + 16 / G * q, q, nrows, w_tiled != 0);
#pragma unroll
    for (int q = 0; q < G * MB; ++q) va[q] = code_off(wave * 16 * MB + 16 / G * q, q, mrows, a_tiled != 0);
    // Rows of A past M: their lanes' loads are masked off and their LDS rows are zero in all stages.  (A load
    // without any lane is issued and counted like another: the waits below are the same for every wavefront.)  The
    // matrix cores' power depends on what they multiply, and this kernel runs at the board's power limit: a tile
    // half of whose rows repeat row M - 1 costs as much as a full one, half of zeros close to half.
    uint64_t ma[G * MB];
#pragma unroll
    for (int q = 0; q < G * MB; ++q) {
        const int row = wave * 16 * MB + 16 / G * q + lrow;
        ma[q] = __builtin_amdgcn_ballot_w64(row < mrows);
        if (row >= mrows) {
#pragma unroll
            for (int u = 0; u < DA / G; ++u)
                *reinterpret_cast<v4i*>(lds + ABASE + u * ASLOT + row * (64 * G) + (lane & (4 * G - 1)) * 16) = v4i{0, 0, 0, 0};
        }
    }
    const uint8_t* sbase[SPW];
    uint32_t sdst[SPW];
    int sstep[SPW], slast[SPW];                                // superstage to superstage, and where the last one starts
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int idx = min(wave + 4 * i, S - 1);              // uniform
        const bool isw = idx < NA, tl = isw ? w_tiled != 0 : a_tiled != 0;
        vsc[i] = isw ? scale_off(64 * idx + lane, nrows, tl) : scale_off(64 * (idx - NA) + lane, mrows, tl);
        const uint8_t* b = isw ? ws + (tl ? wslab * (Kp / 512) * 1024 : n0 * (K / 32))
                               : as + (tl ? aslab * (Kp / 512) * 1024 : m0 * (K / 32));
        sbase[i] = uniform_ptr(b);
        sdst[i] = lds0 + SCALE_BASE + idx * 1024;
        sstep[i] = tl ? 1024 : 16;
        slast[i] = tl ? (KQ - 1) * 1024 : K / 32 - 16;
    }
    const int w_stage = w_tiled ? 4096 : 64, w_last = w_tiled ? (KQ - 1) * 16384 : K / 2 - 256;
    const int a_stage = a_tiled ? 4096 : 64, a_last = a_tiled ? (KQ - 1) * 16384 : K / 2 - 256;
    const uint32_t dst_w = lds0 + wave * (WSLOT / 4), dst_a = lds0 + ABASE + wave * (ASLOT / 4);
    const uint8_t *pw = wbase, *pa = abase;                    // superstages that are being loaded
    uint32_t ld_buf = 0, rd_buf = 0;                           // scale buffers of the superstages being loaded and read
    auto mask_if_less = [](int a, int b) -> uint64_t {         // all lanes if a < b (uniform), in scalar registers
        uint32_t m;                                            // (written out: the compiler makes vector registers of it)
        asm("s_sub_i32 %0, %1, %2\n\ts_ashr_i32 %0, %0, 31" : "=s"(m) : "s"(a), "s"(b) : "scc");
        return ((uint64_t)m << 32) | m;
    };
    auto load_super_w = [&](int q) {                           // (past the last superstage nothing is loaded: see dma_w)
        const int qc = min(q, KQ - 1);
        pw = wbase + (qc == KQ - 1 ? w_last : qc * 4 * w_stage);
    };
    auto load_super_a = [&](int q) {
        const int qc = min(q, KQ - 1);
        pa = abase + (qc == KQ - 1 ? a_last : qc * 4 * a_stage);
    };
    auto dma_scales = [&](int q) {
        const int qc = min(q, KQ - 1);
        const uint64_t live = mask_if_less(q, KQ);
#pragma unroll
        for (int i = 0; i < SPW; ++i)
            dma16_masked<0>(sdst[i] + ld_buf, sbase[i] + (qc == KQ - 1 ? slast[i] : qc * sstep[i]), vsc[i], live);
        ld_buf = ld_buf + SCALE_BUF == NSB * SCALE_BUF ? 0u : ld_buf + SCALE_BUF;
    };
    // load q of stage U (and U + 1) of that superstage into the ring's slot at byte `slot`.  Past the last superstage
    // (`live` = 0) no lane takes part: nothing is read or written, and the counted waits below see the same number of
    // instructions in every stage.
    auto dma_w = [&](auto Uc, auto Qc, uint32_t slot, auto Sure, uint64_t live) {
        constexpr int U = decltype(Uc)::value, q = decltype(Qc)::value;
        if constexpr (decltype(Sure)::value != 0) dma16<q * 1024>(dst_w + slot, pw + U * w_stage, vw[q]);
        else dma16_masked<q * 1024>(dst_w + slot, pw + U * w_stage, vw[q], live);
    };
    auto dma_a = [&](auto Uc, auto Qc, uint32_t slot, auto Sure, uint64_t live) {
        constexpr int U = decltype(Uc)::value, q = decltype(Qc)::value;
        if constexpr (decltype(Sure)::value != 0) dma16_masked<q * 1024>(dst_a + slot, pa + U * a_stage, va[q], ma[q]);
        else dma16_masked<q * 1024>(dst_a + slot, pa + U * a_stage, va[q], ma[q] & live);
    };
    // load I of a stage, W and A alternating while there are both
    auto dma_code = [&](auto Uc, auto Ic, uint32_t wslot, uint32_t aslot, auto Sure, uint64_t live) {
        constexpr int I = decltype(Ic)::value, MN = NA < MB ? NA : MB;
        constexpr bool W = I < 2 * MN ? (I & 1) == 0 : NA > MB;
        constexpr int q = I < 2 * MN ? I / 2 : I - MN;
        if constexpr (W) dma_w(Uc, IC<q>{}, wslot, Sure, live);
        else dma_a(Uc, IC<q>{}, aslot, Sure, live);
    };

    // ---- fragments and scales
    uint32_t wo[2 * G], ao[2 * G];                             // [step, in a pair both stages']: this lane's bytes in slot 0
#pragma unroll
    for (int j = 0; j < 2 * G; ++j) {
        const int c = PAIR ? ((j >> 1) * 4 + 2 * h + (j & 1)) ^ ((r >> 1) & 7) : (2 * h + j) ^ ((r >> 2) & 3);
        wo[j] = (uint32_t)((wn * 32 * NA + r) * (64 * G) + c * 16);
        ao[j] = (uint32_t)(ABASE + (wm * 32 * MB + r) * (64 * G) + c * 16);
    }
    const uint8_t* const wsp = lds + SCALE_BASE + (wn * 32 * NA + r) * 16;
    const uint8_t* const asp = lds + SCALE_BASE + 1024 * NA + (wm * 32 * MB + r) * 16;
    const int hshift = h * 16;
    v4i wf[2][2][NA], af[2][2][MB];                            // [stage parity][step][tile]
    int scw[2][NA], sca[2][MB];
    v4i srw[NA], sra[MB];                                      // a superstage's 16 scale bytes of this lane's rows
    v16f acc[NA][MB];
    // read I of the 2 S fragments of a stage of parity P in these slots, in the order the MFMAs take them
    auto read_frag = [&](auto Pc, auto Ic, uint32_t wslot, uint32_t aslot) {
        constexpr int P = decltype(Pc)::value, J = decltype(Ic)::value / S, k = decltype(Ic)::value % S, O = PAIR ? 2 * P + J : J;
        if constexpr (k >= 1 && k <= MB) af[P][J][k - 1] = *reinterpret_cast<const v4i*>(lds + (ao[O] + aslot) + (k - 1) * (2048 * G));
        else {
            constexpr int t = k == 0 ? 0 : k - MB;
            wf[P][J][t] = *reinterpret_cast<const v4i*>(lds + (wo[O] + wslot) + t * (2048 * G));
        }
    };
    auto read_scales = [&](auto Ic, uint32_t buf) {            // scale rows of W tile I and A tile I
        constexpr int I = decltype(Ic)::value;
        if constexpr (I < NA) srw[I] = *reinterpret_cast<const v4i*>(wsp + buf + I * 512);
        if constexpr (I < MB) sra[I] = *reinterpret_cast<const v4i*>(asp + buf + I * 512);
    };
    // scale registers of stage U from the rows: dword U, this lane half's two bytes; `keep` is 0 for a masked stage
    auto set_scale = [&](auto Uc, auto Pc, auto Ic, int keep) {
        constexpr int U = decltype(Uc)::value, P = decltype(Pc)::value, I = decltype(Ic)::value;
        if constexpr (I < NA) scw[P][I] = (int)((uint32_t)(srw[I][U] & keep) >> hshift);
        else sca[P][I - NA] = (int)((uint32_t)(sra[I - NA][U] & keep) >> hshift);
    };

    // Pairs.  In stage 2 p + 1 pair p has been read and the loads of A's pair p + PA are issued, then the scale loads if W's
    // pair p + PW is a superstage's first, then the loads of that pair.  How many loads are younger than the last one
    // of pair u (odd or not): A's if W's are older, in the stage that issued it and the PA - 2 after it.
    constexpr auto pair_wait = [](int odd) constexpr {
        int n = (PA - 2) * 2 * S + (PW > PA ? 2 * NA : 0);
        for (int b = PW > PA ? PA : PA - 1; b >= 2; --b) n += (odd - b + PW) % 2 == 0 ? SPW : 0;     // issued for p = u - b
        return n;
    };

    // ---- stage U of superstage kq.  LAST: the last superstage, nothing is loaded any more.
    uint32_t wslot = 0, aslot = 0;                             // this stage's slots of the rings (bytes)
    auto stage = [&](auto Uc, auto Lastc, int kq) __attribute__((always_inline)) {
        constexpr int U = decltype(Uc)::value, P = U & 1, NU = (U + 1) & 3;
        constexpr bool LAST = decltype(Lastc)::value != 0, NEXT = !(LAST && U == 3);
        // the stages of W and A that are loaded (pairs: the first ones): stage LU of superstage kq + LQ
        constexpr int WD = PAIR ? U - 1 + DW : U + DW, AD = PAIR ? U - 1 + DA : U + DA;
        constexpr int WU = WD & 3, WQ = WD / 4, AU = AD & 3, AQ = AD / 4;
        constexpr bool LOADS = !LAST && (!PAIR || U % 2 == 1);
        // The next stage's loads have landed once only those of the D - 2 stages after it are outstanding: S each, and
        // the scale loads of the superstages that begin among them (a superstage's scale loads are issued right before
        // its first stage's).  In the last superstage there are fewer, and leaving the scale loads out is only stricter.
        constexpr int BEGIN = (U + DW - 1) / 4 - (U + 1) / 4;   // multiples of 4 in [U + 2, U + D - 1]
        if constexpr (PAIR) {
            if constexpr (U % 2 == 0 || !NEXT) lds_wait_and_barrier();     // the same pair as this stage
            else wait_vm_and_barrier<pair_wait(U == 1 ? 1 : 0)>();
        }
        else if constexpr (!LAST) wait_vm_and_barrier<(DW - 2) * S + BEGIN * SPW>();
        else if constexpr (U < 3) wait_vm_and_barrier<(DW - 2 - U) * S>();
        else lds_wait_and_barrier();
        const int nq = U == 3 ? kq + 1 : kq;                   // superstage of the next stage
        const int keep = (nq == KQ - 1 && NU < ovd) ? 0 : -1;  // uniform
        const bool stay = PAIR && U % 2 == 0;
        const uint32_t nwslot = stay ? wslot : wslot + WSLOT == DW / G * WSLOT ? 0u : wslot + WSLOT;
        const uint32_t naslot = stay ? aslot : aslot + ASLOT == DA / G * ASLOT ? 0u : aslot + ASLOT;
        constexpr int RPS = NS >= 2 * S + 2 ? 1 : 2;           // fragment reads per slot
        const uint64_t live = mask_if_less(kq + WQ, KQ), alive = mask_if_less(kq + AQ, KQ);
        if constexpr (WU == 0 && LOADS) load_super_w(kq + WQ);
        if constexpr (AU == 0 && LOADS) load_super_a(kq + AQ);
        static_for([&](auto Sc) __attribute__((always_inline)) {
            constexpr int s = decltype(Sc)::value, J = s / NM, X = s % NM, A = X / MB, B = X % MB;
            mfma_fp4(acc[A][B], wf[P][J][A], af[P][J][B], IC<J>{}, scw[P][A], sca[P][B]);
            if constexpr (NEXT) {
                static_for([&](auto Ic) __attribute__((always_inline)) {
                    constexpr int i = s * RPS + decltype(Ic)::value;
                    if constexpr (i < 2 * S) read_frag(IC<P ^ 1>{}, IC<i>{}, nwslot, naslot);
                }, IC<RPS>{});
                if constexpr (U == 3 && s < (NA > MB ? NA : MB)) read_scales(IC<s>{}, rd_buf);
                constexpr int first = NS - 1 - (S + 1) / 2;    // two scale registers per slot, done one slot before the end
                static_assert(first >= (NA > MB ? NA : MB) - 1, "the rows are read before the registers are made from them");
                static_for([&](auto Ic) __attribute__((always_inline)) {
                    constexpr int i = (s - first) * 2 + decltype(Ic)::value;
                    if constexpr (s >= first && i < S) set_scale(IC<NU>{}, IC<P ^ 1>{}, IC<i>{}, keep);
                }, IC<2>{});
            }
            if constexpr (LOADS) {
                if constexpr (!PAIR && WU == 0 && s == 0) dma_scales(kq + WQ);
                static_for([&](auto Ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(Ic)::value;
                    if constexpr ((2 * i + 1) * NM / (G * S) == s) {
                        if constexpr (!PAIR) dma_code(IC<WU>{}, Ic, wslot, aslot, IC<(WQ < 2)>{}, live);
                        else if constexpr (i < 2 * MB) dma_a(IC<AU>{}, Ic, aslot, IC<(AQ < 2)>{}, alive);
                        else {
                            if constexpr (i == 2 * MB && WU == 0) dma_scales(kq + WQ);
                            dma_w(IC<WU>{}, IC<i - 2 * MB>{}, wslot, IC<(WQ < 2)>{}, live);
                        }
                    }
                }, IC<G * S>{});
            }
            __builtin_amdgcn_sched_barrier(0);
        }, IC<NS>{});
        wslot = nwslot;
        aslot = naslot;
        if constexpr (U == 3) rd_buf = rd_buf + SCALE_BUF == NSB * SCALE_BUF ? 0u : rd_buf + SCALE_BUF;
    };
    auto superstage = [&](auto Lastc, int kq) __attribute__((always_inline)) {
        stage(IC<0>{}, Lastc, kq);
        stage(IC<1>{}, Lastc, kq);
        stage(IC<2>{}, Lastc, kq);
        stage(IC<3>{}, Lastc, kq);
    };

    // ---- prologue: the first D stages in flight, accumulators cleared meanwhile, stage 0 in registers
    if constexpr (PAIR) {
        static_for([&](auto Tc) __attribute__((always_inline)) {        // as in stage 2 p + 1, p = -PW, .., -1
            constexpr int w = decltype(Tc)::value, a = w - PW + PA;     // the pairs of W and A
            if constexpr (a >= 0) {
                if constexpr (a % 2 == 0) load_super_a(a / 2);
                static_for([&](auto Qc) { dma_a(IC<(2 * a & 3)>{}, Qc, (uint32_t)(a * ASLOT), IC<(a < 2)>{}, mask_if_less(a / 2, KQ)); }, IC<2 * MB>{});
            }
            if constexpr (w % 2 == 0) { load_super_w(w / 2); dma_scales(w / 2); }
            static_for([&](auto Qc) { dma_w(IC<(2 * w & 3)>{}, Qc, (uint32_t)(w * WSLOT), IC<(w < 2)>{}, mask_if_less(w / 2, KQ)); }, IC<2 * NA>{});
        }, IC<PW>{});
    } else {
        static_for([&](auto Tc) __attribute__((always_inline)) {
            constexpr int T = decltype(Tc)::value;
            if constexpr (T % 4 == 0) { load_super_w(T / 4); load_super_a(T / 4); dma_scales(T / 4); }
            static_for([&](auto Ic) { dma_code(IC<(T & 3)>{}, Ic, (uint32_t)(T * WSLOT), (uint32_t)(T * ASLOT), IC<(T < 4)>{}, mask_if_less(T / 4, KQ)); }, IC<S>{});
        }, IC<DW>{});
    }
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            // One definition the compiler cannot see into: from a constant it made one set of zeros for a K of a single
            // superstage and another for the loop, and moved all accumulators from register to register between the
            // loop and the last superstage, reading some 10 wait states after the MFMA that writes them (12 are needed,
            // and it does not know that these are MFMAs).
            acc[a][b] = v16f{};
            asm volatile("" : "+a"(acc[a][b]));
        }
    wait_vm_and_barrier<(PAIR ? pair_wait(0) : (DW - 1) * S + (NSB - 1) * SPW)>();
    static_for([&](auto Ic) { read_frag(IC<0>{}, Ic, 0u, 0u); }, IC<2 * S>{});
    static_for([&](auto Ic) { read_scales(Ic, 0); }, IC<(NA > MB ? NA : MB)>{});
    static_for([&](auto Ic) { set_scale(IC<0>{}, IC<0>{}, Ic, -1); }, IC<S>{});   // (a single superstage shares nothing)
    rd_buf = NSB == 1 ? 0u : (uint32_t)SCALE_BUF;
    for (int kq = 0; kq < KQ - 1; ++kq) superstage(IC<0>{}, kq);
    superstage(IC<1>{}, KQ - 1);

    store_tile<OUT_BF16, NA, MB>(acc, lds, y, ldy, m0, n0, M, N, lines);
}

// ---- any K of at least 256 elements, any mix of layouts: what the kernels above do not take (row-major K that is not a multiple
// of 128, mixed layouts with K % 512 != 0, K below 512).  A row's scales then begin at any byte and its codes on any 16, which
// LDS-DMA is not for: tiles of 64 MB x 128 whose operands pass through registers, two pairs of stages ahead, into two halves of LDS (the
// image of PAIR above), one barrier a pair.  The last pair's groups past K load the last one's codes, in bounds, and have scale
// byte 0 in both operands.  Same order of summation as everywhere.
// Bound by the address path, which takes a load by the lines it touches: two stages at once are 8 rows x 128 bytes an instruction,
// 8 to 16 lines for what takes 32 stage by stage, and a row's scales cost a line whether four or eight are taken.  us, bf16 out,
// one 32 x 32 tile a wavefront straight from global memory (k_gemm_direct) : stage by stage : now: 2000 x 4096 x 10976 656 : 125 : 88,
// 300 x 4096 x 4000 32.6 : 20.3 : 19.5, 2629 x 26904 x 832 315 : 104 : 104 (there the tiles' two ends are most of it).
template <bool OUT_BF16, int MB>
__global__ void __launch_bounds__(256, 2)
k_gemm_any_k(const uint8_t* __restrict__ aq, const uint8_t* __restrict__ as, const uint8_t* __restrict__ wq, const uint8_t* __restrict__ ws,
             int M, int N, int K, void* __restrict__ y, int64_t ldy, int a_tiled, int w_tiled, int lines) {
    constexpr int NA = 2, TM = 64 * MB, TN = 128, SETS = 2, CODES = 128 * (TN + TM), BUF = CODES + 8 * 256;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];                            // 2 BUF
    load_args(aq, as, wq, ws, M, N, K, a_tiled, w_tiled);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5, wn = wave >> 1, wm = wave & 1;
    const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + TN - 1) / TN, T = tiles_m * tiles_n, per_xcd = (T + 7) / 8;
    TileWalk tw{(int)((blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3)), min((int)((blockIdx.x & 7) + 1) * per_xcd, T), 1, tiles_m, tiles_n};
    if (tw.first >= tw.end) return;                            // uniform over the workgroup
    int tm, tn;
    tw.tile(0, tm, tn);
    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * TN;
    const int groups = K / 32, pairs = (groups + 7) / 8;
    // codes: thread i brings chunk i & 7 of rows i >> 3, + 32, ..; scales: of row i of the 128 of W and the TM of A
    const uint8_t *wp[4], *ap[2 * MB];
    const int64_t Kp = ((int64_t)K + 511) / 512 * 512;
    auto code_row = [&](const uint8_t* c, bool tiled, int64_t row) { return c + (tiled ? (row >> 6) * (Kp / 128) * 4096 + (row & 63) * 64 : row * (K / 2)); };
    auto scale_row = [&](const uint8_t* s, bool tiled, int64_t row) { return s + (tiled ? (row >> 6) * (Kp / 512) * 1024 + (row & 63) * 16 : row * (K / 32)); };
#pragma unroll
    for (int q = 0; q < 4; ++q) wp[q] = code_row(wq, w_tiled, min(n0 + 32 * q + (tid >> 3), (int64_t)N - 1));
#pragma unroll
    for (int q = 0; q < 2 * MB; ++q) ap[q] = code_row(aq, a_tiled, min(m0 + 32 * q + (tid >> 3), (int64_t)M - 1));
    const bool st = wave < 2 ? w_tiled : a_tiled;
    const uint8_t* const sp = wave < 2 ? scale_row(ws, st, min(n0 + tid, (int64_t)N - 1)) : scale_row(as, st, min(m0 + tid - TN, (int64_t)M - 1));
    const int64_t wstep = w_tiled ? 4096 : 64, astep = a_tiled ? 4096 : 64;
    v4i cw[SETS][4], ca[SETS][2 * MB];
    uint64_t sc[SETS];
    auto load = [&](int t, v4i (&w)[4], v4i (&a)[2 * MB], uint64_t& s) {
        t = min(t, pairs - 1);                                 // past the end: the last pair again, which nobody reads
        const int g = min(8 * t + (tid & 7), groups - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const v4i*>(wp[q] + (g >> 2) * wstep + (g & 3) * 16);
#pragma unroll
        for (int q = 0; q < 2 * MB; ++q) a[q] = *reinterpret_cast<const v4i*>(ap[q] + (g >> 2) * astep + (g & 3) * 16);
        typedef uint64_t any __attribute__((aligned(1)));
        s = *reinterpret_cast<const any*>(sp + pair_scales(st, t, groups));      // (one load: none behind a branch)
        __builtin_amdgcn_sched_barrier(0);
    };
    uint8_t* const wr = lds + (tid >> 3) * 128 + (((tid & 7) ^ ((tid >> 4) & 7)) << 4);
    auto put = [&](int t, uint32_t buf, const v4i (&w)[4], const v4i (&a)[2 * MB], uint64_t s) {
        const int over = 8 * max(8 * min(t, pairs - 1) - (groups - 8), 0);       // bits of the last pair's scales that are past K
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<v4i*>(wr + buf + q * 4096) = w[q];
#pragma unroll
        for (int q = 0; q < 2 * MB; ++q) *reinterpret_cast<v4i*>(wr + buf + (4 + q) * 4096) = a[q];
        *reinterpret_cast<uint64_t*>(lds + buf + CODES + tid * 8) = st ? s & (~uint64_t(0) >> over) : s >> over;
        __builtin_amdgcn_sched_barrier(0);
    };
    v16f acc[NA][MB];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[a][b] = v16f{};
    const uint8_t* const wrd = lds + (wn * 64 + r) * 128;
    const uint8_t* const ard = lds + (TN + wm * 32 * MB + r) * 128;
    const uint8_t* const wsp = lds + CODES + (wn * 64 + r) * 8;
    const uint8_t* const asp = lds + CODES + (TN + wm * 32 * MB + r) * 8;
    const uint32_t sw = (uint32_t)(r >> 1) & 7u;
    auto multiply = [&](uint32_t buf) {
        uint64_t sw_[NA], sa_[MB];
#pragma unroll
        for (int k = 0; k < NA; ++k) sw_[k] = *reinterpret_cast<const uint64_t*>(wsp + buf + k * 256);
#pragma unroll
        for (int k = 0; k < MB; ++k) sa_[k] = *reinterpret_cast<const uint64_t*>(asp + buf + k * 256);
#pragma unroll
        for (int u = 0; u < 2; ++u)                            // stage u of the pair, step j
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t c = ((uint32_t)(4 * u + 2 * h + j) ^ sw) << 4;
                v8i w[NA], a[MB];
#pragma unroll
                for (int k = 0; k < NA; ++k) {
                    const v4i f = *reinterpret_cast<const v4i*>(wrd + buf + k * 4096 + c);
                    w[k] = v8i{f[0], f[1], f[2], f[3], 0, 0, 0, 0};
                }
#pragma unroll
                for (int k = 0; k < MB; ++k) {
                    const v4i f = *reinterpret_cast<const v4i*>(ard + buf + k * 4096 + c);
                    a[k] = v8i{f[0], f[1], f[2], f[3], 0, 0, 0, 0};
                }
#pragma unroll
                for (int x = 0; x < NA * MB; ++x) {
                    v16f& d = acc[x / MB][x % MB];
                    const int s0 = (int)((uint32_t)(sw_[x / MB] >> (32 * u)) >> (16 * h)), s1 = (int)((uint32_t)(sa_[x % MB] >> (32 * u)) >> (16 * h));
                    if (j == 0) d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[x / MB], a[x % MB], d, 4, 4, 0, s0, 0, s1);
                    else d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[x / MB], a[x % MB], d, 4, 4, 1, s0, 1, s1);
                }
            }
    };
    // turn t: pair t + 1 into the half of LDS that pair t - 1 was read from, pair t + 1 + SETS requested, pair t multiplied
    uint32_t buf = 0;
    auto turn = [&](auto Kc, int t) __attribute__((always_inline)) {
        constexpr int k = (decltype(Kc)::value + 1) % SETS;
        put(t + 1, BUF - buf, cw[k], ca[k], sc[k]);
        load(t + 1 + SETS, cw[k], ca[k], sc[k]);
        multiply(buf);
        lds_wait_and_barrier();
        buf = BUF - buf;
    };
    static_for([&](auto Kc) __attribute__((always_inline)) { load(decltype(Kc)::value, cw[decltype(Kc)::value], ca[decltype(Kc)::value], sc[decltype(Kc)::value]); }, IC<SETS>{});
    put(0, 0, cw[0], ca[0], sc[0]);
    load(SETS, cw[0], ca[0], sc[0]);
    lds_wait_and_barrier();
    int t = 0;
    for (; t + SETS <= pairs; t += SETS) static_for([&](auto Kc) __attribute__((always_inline)) { turn(Kc, t + decltype(Kc)::value); }, IC<SETS>{});
    if (t < pairs) turn(IC<0>{}, t);
    store_tile<OUT_BF16, NA, MB>(acc, lds, y, ldy, m0, n0, M, N, lines);
}
constexpr int any_k_lds_bytes(int mb) { return 2 * (128 * (128 + 64 * mb) + 8 * 256); }

using Kern = void (*)(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*, int, int, int, void*, int64_t, int, int, int);
struct Variant { int na, mb, dw, da; Kern bf16, f32; };
#define BRQ_MID(NA, MB, DW, DA, PAIR) {NA, MB, DW, DA, k_gemm_mid<true, NA, MB, DW, DA, PAIR>, k_gemm_mid<false, NA, MB, DW, DA, PAIR>}
static const Variant singles[MID_TILES] = {BRQ_MID(2, 1, 6, 6, false), BRQ_MID(2, 2, 4, 4, false), BRQ_MID(2, 3, 4, 4, false),
                                           BRQ_MID(4, 3, 4, 4, false), BRQ_MID(2, 5, 5, 5, false), BRQ_MID(2, 4, 6, 6, false)};
static const Variant pairs[MID_TILES] = {BRQ_MID(2, 1, 6, 6, true), BRQ_MID(2, 2, 6, 6, true), BRQ_MID(2, 3, 6, 6, true),
                                         BRQ_MID(4, 3, 4, 4, true), BRQ_MID(2, 5, 6, 4, true),
                                         BRQ_MID(2, 4, 6, 4, true)};       // (6 stages of A: 0.5 % slower to 1 % faster)
#undef BRQ_MID
using AnyK = void (*)(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*, int, int, int, void*, int64_t, int, int, int);
static const AnyK any_k[2][2] = {{k_gemm_any_k<false, 1>, k_gemm_any_k<true, 1>}, {k_gemm_any_k<false, 2>, k_gemm_any_k<true, 2>}};    // [MB - 1][bf16 out]

}  // namespace mid

bool mid_gemm_pairs(int tile, bool both_tiled, int64_t K) { return !both_tiled && (K > 1024 || tile > 2); }

hipError_t setup_gemm_mid() {
    for (int i = 0; i < 2 * MID_TILES; ++i) {
        const mid::Variant& v = (i % 2 ? mid::singles : mid::pairs)[i / 2];
        for (mid::Kern k : {v.bf16, v.f32})
            if (hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   mid::lds_bytes(v.na, v.mb, v.dw, v.da)); e != hipSuccess) return e;
    }
    for (int mb = 1; mb <= 2; ++mb)
        for (mid::AnyK k : mid::any_k[mb - 1])
            if (hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, mid::any_k_lds_bytes(mb)); e != hipSuccess) return e;
    return hipSuccess;
}

// Whole superstages, or both operands row-major with K a multiple of 128 and at least one superstage.  A lane's offset
// inside the tile, below 64 max(NA, MB) rows of Kp / 2 bytes, has 32 bits, and the offset along K 31 (32 Kp bytes).
bool mid_gemm_supported(int tile, const GemmShape& g) {
    const mid::Variant& v = mid::singles[tile];
    const int64_t Kp = g.padded_k(), slabs = v.na > v.mb ? v.na : v.mb;
    return g.M > 0 && g.N > 0 && (g.whole_k() || (!g.a_tiled && !g.w_tiled && g.K % 128 == 0 && g.K >= 512)) &&
           Kp < (int64_t(1) << 26) && slabs * 32 * Kp <= (int64_t(1) << 32);
}

static int on_half_lines(const void* y, int64_t N, int64_t ldy, bool out_bf16) {
    const int es = out_bf16 ? 2 : 4;
    return N * es % 16 == 0 && rows_on(64, reinterpret_cast<uintptr_t>(y), ldy * es);
}

// Tiles of 64 rows where that is all there are.
hipError_t launch_gemm_any_k(const Operand& a, const Operand& w, int64_t M, int64_t N, int64_t K, void* y, bool out_bf16, int64_t ldy, hipStream_t s) {
    const int mb = M <= 64 ? 1 : 2;
    const int64_t T = (M + 64 * mb - 1) / (64 * mb) * ((N + 127) / 128);
    hipLaunchKernelGGL(mid::any_k[mb - 1][out_bf16], dim3((uint32_t)((T + 7) / 8 * 8)), dim3(256), mid::any_k_lds_bytes(mb), s, a.codes, a.scales, w.codes, w.scales, (int)M, (int)N, (int)K, y, ldy,
                       (int)a.tiled, (int)w.tiled, on_half_lines(y, N, ldy, out_bf16));
    return hipGetLastError();
}

hipError_t launch_gemm_mid(int tile, const Operand& a, const Operand& w, int64_t M, int64_t N, int64_t K, void* y,
                           bool out_bf16, int64_t ldy, hipStream_t s) {
    const mid::Variant& v = (mid_gemm_pairs(tile, a.tiled && w.tiled, K) ? mid::pairs : mid::singles)[tile];
    const int64_t tm = (M + 64 * v.mb - 1) / (64 * v.mb), tn = (N + 64 * v.na - 1) / (64 * v.na), T = tm * tn;
    const int lines = on_half_lines(y, N, ldy, out_bf16);
    hipLaunchKernelGGL((out_bf16 ? v.bf16 : v.f32), dim3((uint32_t)((T + 7) / 8 * 8)), dim3(256), mid::lds_bytes(v.na, v.mb, v.dw, v.da), s,
                       a.codes, a.scales, w.codes, w.scales, (int)M, (int)N, (int)K, y, ldy, (int)a.tiled, (int)w.tiled, lines);
    return hipGetLastError();
}

}  // namespace brq
