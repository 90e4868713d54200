// Reduction of the per-block statistics to what the paper's analysis reports (Sec. 4.1, 4.2 and the
// Appendix "Rotation Comparison"): the distribution of the block-wise scales, and the quantization loss and
// the growth of the scales split into regular and outlier blocks.  Input: the per-block arrays that
// brq_block_stats writes (one fp32 per block of 32).  HBM bound and small: 8 to 12 bytes per block.
#include "brq_device.h"
#include "brq_launch.h"

namespace brq {

struct SummaryArgs {
    const float* amax;              // [n] block-wise scales after the transformation under study
    const float* sqerr;             // [n] or null: per-block MXFP4 loss after it
    const float* ref;               // [n] or null: block-wise scales of the reference (untransformed) activations
    unsigned long long n;
    float outlier;                  // a block is an outlier block when its reference scale exceeds this
    int nedges;                     // 0..32
    float edges[32];
    unsigned long long* hist;       // [nedges + 1] or null, added to
    unsigned long long* counts;     // [4] or null, added to
    double* sums;                   // [4] or null, added to
};

// Eight blocks per lane and pass, 16 bytes of each array per load (VEC; arrays that are not 16-byte aligned are read
// 4 bytes at a time), the next pass's loads issued before this pass's blocks are looked at.  Histogram: the edges
// ascend, so a scale that exceeds edge e exceeds every edge below it; per edge the wavefront counts its lanes above it
// with one comparison and the scalar unit's bit count, and bin j follows as (count above edge j - 1) - (count above
// edge j).  Class counts the same way.  The outlier sums are touched only where the wavefront has an outlier block.
// The fp64 sums are added across a wavefront's lanes in a fixed butterfly, across the workgroup's
// wavefronts in index order, and across workgroups by the hardware's fp64 atomic add (the generic atomicAdd on a
// double is a compare-and-swap loop): the result depends on the order in which workgroups finish, to a few units
// of 2^-53 times their number.
// 4.19 M blocks with seven edges (50 MB): 19.4 -> 15.9 us; with 4-byte loads, and every one of 32 possible edges looked
// at by the compiler's own choice, the scalar registers' contents went through vector registers (56 spilled).
// NE: edges that are looked at, 0 (no histogram), 8, 16 or 32; those beyond nedges are +inf.  With the number known to
// the compiler the edges and their counters stay in scalar registers, up to 8 of them (16 edges spill 6 registers, 32 edges 48).
template <int NE>
struct SummaryAcc {
    unsigned int cnt[4], nlive, gt[NE ? NE : 1];     // wavefront-uniform, held by the scalar unit
    double sum[4];
};
// One block per lane; `live` = this lane has one.
template <int NE>
__device__ __forceinline__ void summary_block(SummaryAcc<NE>& s, const SummaryArgs& a, float am, float rf, float sq, bool live, bool has_sq, bool has_ref) {
    const unsigned long long lm = __builtin_amdgcn_ballot_w64(live);
    const unsigned long long mo = __builtin_amdgcn_ballot_w64(rf > a.outlier) & lm;
    const unsigned long long mr = lm & ~mo;
    const unsigned long long mg = has_ref ? __builtin_amdgcn_ballot_w64(am > rf) : 0ull;
    s.cnt[0] += (unsigned int)__builtin_popcountll(mr);
    s.cnt[2] += (unsigned int)__builtin_popcountll(mr & mg);
    const bool isr = (mr >> (threadIdx.x & 63u)) & 1ull;
    s.sum[0] += (double)((isr && has_sq) ? sq : 0.0f);
    s.sum[2] += (double)(isr ? am : 0.0f);
    if (mo) {   // uniform
        s.cnt[1] += (unsigned int)__builtin_popcountll(mo);
        s.cnt[3] += (unsigned int)__builtin_popcountll(mo & mg);
        const bool iso = (mo >> (threadIdx.x & 63u)) & 1ull;
        s.sum[1] += (double)((iso && has_sq) ? sq : 0.0f);
        s.sum[3] += (double)(iso ? am : 0.0f);
    }
    if constexpr (NE > 0) {
        s.nlive += (unsigned int)__builtin_popcountll(lm);
        const float v = live ? am : -__builtin_inff();     // above no edge
#pragma unroll
        for (int e = 0; e < NE; ++e) count_above<false>(s.gt[e], v, a.edges[e]);
    }
}
template <bool VEC, int NE>
__global__ void __launch_bounds__(1024) k_block_summary(SummaryArgs a) {
    __shared__ unsigned int s_gt[33];        // [e]: blocks above edge e; [32]: all blocks of the workgroup
    __shared__ unsigned int s_cnt[4];
    __shared__ double s_wsum[16][4];
    if (threadIdx.x < 33) s_gt[threadIdx.x] = 0;
    if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const float* const refp = a.ref ? a.ref : a.amax;
    const float* const sqp = a.sqerr ? a.sqerr : a.amax;
    const bool has_sq = a.sqerr != nullptr, has_ref = a.ref != nullptr, lane0 = (threadIdx.x & 63u) == 0;
    SummaryAcc<NE> s;
    s.nlive = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e) s.gt[e] = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) { s.cnt[k] = 0; s.sum[k] = 0.0; }
    constexpr unsigned int U = 8, SPAN = 1024 * U;
    const unsigned long long step = (unsigned long long)gridDim.x * SPAN;
    unsigned long long i0 = (unsigned long long)blockIdx.x * SPAN;
    // (every load is unconditional - an absent array is replaced by the scales themselves - because a load behind a
    // branch makes the compiler wait for all earlier ones)
    struct Batch { v4f am[2], rf[2], sq[2]; };
    auto load = [&](unsigned long long at, Batch& b) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if constexpr (VEC) {
                const unsigned long long i = at + q * 4096u + threadIdx.x * 4u;
                b.am[q] = *reinterpret_cast<const v4f*>(a.amax + i);
                b.rf[q] = *reinterpret_cast<const v4f*>(refp + i);
                b.sq[q] = *reinterpret_cast<const v4f*>(sqp + i);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned long long i = at + q * 4096u + u * 1024u + threadIdx.x;
                    b.am[q][u] = a.amax[i];
                    b.rf[q][u] = refp[i];
                    b.sq[q][u] = sqp[i];
                }
            }
        }
    };
    Batch cur;
    if (i0 + SPAN <= a.n) load(i0, cur);
    for (; i0 + SPAN <= a.n; i0 += step) {
        Batch nxt;
        load(i0 + step + SPAN <= a.n ? i0 + step : i0, nxt);       // (nothing follows: this one again)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) summary_block(s, a, cur.am[q][u], cur.rf[q][u], cur.sq[q][u], true, has_sq, has_ref);
        cur = nxt;
    }
    if (i0 < a.n) {   // the ragged end: one workgroup
        for (unsigned int u = 0; u < U; ++u) {
            const unsigned long long i = i0 + u * 1024u + threadIdx.x;
            const bool live = i < a.n;
            const unsigned long long ic = live ? i : a.n - 1;
            summary_block(s, a, a.amax[ic], refp[ic], sqp[ic], live, has_sq, has_ref);
        }
    }
    unsigned int (&cnt)[4] = s.cnt;
    double (&sum)[4] = s.sum;
    const unsigned int nlive = s.nlive;
    const unsigned int wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double v = sum[k];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
        if (lane0) {
            s_wsum[wave][k] = v;
            if (cnt[k]) atomicAdd(&s_cnt[k], cnt[k]);
        }
    }
    if (lane0 && NE > 0) {
        atomicAdd(&s_gt[32], nlive);
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if (s.gt[e]) atomicAdd(&s_gt[e], s.gt[e]);
    }
    __syncthreads();
    if (NE > 0 && threadIdx.x <= (unsigned)a.nedges) {
        const unsigned int above_prev = threadIdx.x == 0 ? s_gt[32] : s_gt[threadIdx.x - 1];
        const unsigned int above_this = threadIdx.x == (unsigned)a.nedges ? 0u : s_gt[threadIdx.x];
        if (above_prev != above_this) atomicAdd(&a.hist[threadIdx.x], (unsigned long long)(above_prev - above_this));
    }
    if (threadIdx.x < 4) {
        if (a.counts && s_cnt[threadIdx.x]) atomicAdd(&a.counts[threadIdx.x], (unsigned long long)s_cnt[threadIdx.x]);
        double t = 0.0;
        for (unsigned int w = 0; w < blockDim.x / 64u; ++w) t += s_wsum[w][threadIdx.x];
        if (a.sums && t != 0.0) __builtin_amdgcn_global_atomic_fadd_f64(&a.sums[threadIdx.x], t);
    }
}

hipError_t launch_block_summary(const float* amax, const float* sqerr, const float* ref, int64_t n, float outlier,
                                const float* edges, int nedges, unsigned long long* hist, unsigned long long* counts,
                                double* sums, hipStream_t s) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
    SummaryArgs a;
    a.amax = amax; a.sqerr = sqerr; a.ref = ref; a.n = (unsigned long long)n; a.outlier = outlier; a.nedges = nedges;
    for (int e = 0; e < 32; ++e) a.edges[e] = e < nedges ? edges[e] : __builtin_inff();   // beyond nedges: exceeded by nothing
    a.hist = hist; a.counts = counts; a.sums = sums;
    // One workgroup of 16 wavefronts per compute unit at most: every workgroup ends with an atomic per output
    // word, and atomics on the same few words from thousands of workgroups would take longer than the pass
    // over the data.
    const int64_t want = (n + 8191) / 8192;
    const int64_t cap = (int64_t)cus;
    const dim3 grid((uint32_t)(want < cap ? (want < 1 ? 1 : want) : cap));
    const bool vec = ((reinterpret_cast<uintptr_t>(amax) | reinterpret_cast<uintptr_t>(sqerr) | reinterpret_cast<uintptr_t>(ref)) & 15u) == 0;
    using Kern = void (*)(SummaryArgs);
    static const Kern kern[2][4] = {{k_block_summary<false, 0>, k_block_summary<false, 8>, k_block_summary<false, 16>, k_block_summary<false, 32>},
                                    {k_block_summary<true, 0>, k_block_summary<true, 8>, k_block_summary<true, 16>, k_block_summary<true, 32>}};
    const Kern k = kern[vec][!hist ? 0 : nedges <= 8 ? 1 : nedges <= 16 ? 2 : 3];
    hipLaunchKernelGGL(k, grid, dim3(1024), 0, s, a);
    return hipGetLastError();
}

}  // namespace brq
