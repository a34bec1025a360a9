// Quality diagnostic of libdhsa: per-row recall of the routed key sets against
// exact top-k attention (App. "Theoretical Analysis", Setup and Notation:
// Recall_i = |I*_i n I_hat_i| / |I*_i|, I*_i = the k keys j <= i with the largest
// attention scores, k = min(N_b, i + 1), equal scores by lower index).
//
// Two kernels:
//   k_recall_logits  logits q_i . k_j, j <= i, in fp64, summed in the order d = 0, 1, ... by one
//      thread per key (the products of bf16 / fp32 values are exact in fp64, so the
//      value is the same on any machine that sums in that order), stored as
//      order-preserving 64-bit integers in the caller's workspace;
//   k_recall_count  one workgroup per sampled row: the k-th largest of them by a
//      most-significant-digit radix select, then the row's selected keys (walked from
//      the plan like the attention kernels do) are counted if their logit is above that
//      threshold, or equal to it and among the lowest-indexed equal ones that still fit
//      into the top k.
// Measured (48 rows of L = 32768, D = 128): 550 us when one workgroup per row did all of it
// (a thread read its key row two bytes at a time and the plan entries were walked one by
// one); what the two kernels take now is at each of them.
#include <algorithm>

#include "dhsa_internal.h"

namespace dhsa {

constexpr int kRecallRows = 512;        // rows per launch: their numbers travel as kernel arguments
struct RecallRows {
    int32_t n;
    int32_t row[kRecallRows];
};

// A thread owns kLgKeys keys and kLgRows of the sampled rows, so that an element of q read from LDS
// (a broadcast) serves kLgKeys products and a converted element of K serves kLgRows.  Bound by
// the fp64 rate of the vector unit and the LDS reads of q, about equally.  A key row is
// read 64 bytes at a time by its thread.  48 rows of L = 32768, D = 128: 24 us.
constexpr int kLgKeys = 2, kLgRows = 8;

template <typename T> struct RecallElem;
template <> struct RecallElem<float> {
    static constexpr int kPerWord = 1;
    __device__ static double get(uint32_t w, int) { return (double)__uint_as_float(w); }
    __device__ static double load(const float *p) { return (double)*p; }
};
template <> struct RecallElem<bf16_t> {
    static constexpr int kPerWord = 2;
    __device__ static double get(uint32_t w, int half) {
        return (double)__uint_as_float(half ? w & 0xffff0000u : w << 16);
    }
    __device__ static double load(const bf16_t *p) { return (double)__uint_as_float((uint32_t)p->bits << 16); }
};

template <typename T, int D>
__global__ __launch_bounds__(256) void k_recall_logits(PlanView pv, const T *__restrict__ Q, const T *__restrict__ K,
                                                       int G, int head, RecallRows rows, int64_t L,
                                                       unsigned long long *__restrict__ ws, int64_t qs_h, int64_t qs_l,
                                                       int64_t ks_h, int64_t ks_l) {
    __shared__ double s_q[kLgRows][D];
    if (!plan_matches(pv)) return;   // not this problem's plan: nothing is written
    const int tid = threadIdx.x;
    const int t0 = blockIdx.y * kLgRows;
    const int nr = rows.n - t0 < kLgRows ? rows.n - t0 : kLgRows;
    int last = 0;                    // last row of the group
    for (int r = 0; r < nr; ++r) last = rows.row[t0 + r] > last ? rows.row[t0 + r] : last;
    const int j0 = blockIdx.x * 256 * kLgKeys;
    if (j0 > last) return;           // no row sees these keys (block-uniform)
    for (int x = tid; x < kLgRows * D; x += 256) {
        const int r = x / D < nr ? x / D : 0;
        s_q[x / D][x % D] = RecallElem<T>::load(Q + (int64_t)head * qs_h + (int64_t)rows.row[t0 + r] * qs_l + x % D);
    }
    __syncthreads();
    const T *kr[kLgKeys];
#pragma unroll
    for (int k = 0; k < kLgKeys; ++k) {
        const int j = j0 + k * 256 + tid;
        kr[k] = K + (int64_t)(head / G) * ks_h + (int64_t)(j < last ? j : last) * ks_l;   // a row that exists
    }
    double acc[kLgKeys][kLgRows];
#pragma unroll
    for (int k = 0; k < kLgKeys; ++k)
#pragma unroll
        for (int r = 0; r < kLgRows; ++r) acc[k][r] = 0.0;
    constexpr int kEl = 64 / (int)sizeof(T);            // elements per 64 bytes
#pragma unroll 1   // all of D at once makes <float, 64> spill 774 registers: 426 us at that size, 39 us so
    for (int d0 = 0; d0 < D; d0 += kEl) {
        uint4 u[kLgKeys][4];
#pragma unroll
        for (int k = 0; k < kLgKeys; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) u[k][c] = reinterpret_cast<const uint4 *>(kr[k] + d0)[c];
#pragma unroll
        for (int w = 0; w < 16; ++w)
#pragma unroll
            for (int half = 0; half < RecallElem<T>::kPerWord; ++half) {
                double kx[kLgKeys];
#pragma unroll
                for (int k = 0; k < kLgKeys; ++k) {
                    const uint4 &v = u[k][w / 4];
                    const uint32_t word = (w & 3) == 0 ? v.x : (w & 3) == 1 ? v.y : (w & 3) == 2 ? v.z : v.w;
                    kx[k] = RecallElem<T>::get(word, half);
                }
                const int d = d0 + w * RecallElem<T>::kPerWord + half;
#pragma unroll
                for (int r = 0; r < kLgRows; ++r)
#pragma unroll
                    for (int k = 0; k < kLgKeys; ++k) acc[k][r] = __builtin_fma(s_q[r][d], kx[k], acc[k][r]);
            }
    }
#pragma unroll
    for (int r = 0; r < kLgRows; ++r) {
        if (r >= nr) break;
        const int i = rows.row[t0 + r];
#pragma unroll
        for (int k = 0; k < kLgKeys; ++k) {
            const int j = j0 + k * 256 + tid;
            double x = acc[k][r];
            if (x == 0.0) x = 0.0;                       // -0.0 ties with +0.0
            const unsigned long long u = (unsigned long long)__double_as_longlong(x);
            if (j <= i) ws[(int64_t)(t0 + r) * L + j] = (u >> 63) ? ~u : (u | 0x8000000000000000ull);
        }
    }
}

// ---------------------------------------------------------------------------
// Radix select and count of one row.  The first digits are 14 bits wide (sign, exponent and two bits of
// the mantissa: narrower ones would put most logits into two or three counters) and are
// counted from memory; a region of at most kRcCand keys moves into LDS and is finished there
// with 8-bit digits.  The select ends early when every key of the region belongs to the
// top set.  Bound by latency: one CU reads the row's keys twice (256 KB each time at n = 32768;
// 21 us for 48 rows).  Ties at the threshold: where the last equal key of the top set lies is found once, by counting.
// ---------------------------------------------------------------------------
constexpr int kRcThreads = 1024;
constexpr int kRcBits = 14;
constexpr int kRcCand = 4096;

__global__ __launch_bounds__(kRcThreads) void k_recall_count(PlanView pv, int N_b, int head, RecallRows rows, int64_t L,
                                                             const unsigned long long *__restrict__ ws,
                                                             int32_t *__restrict__ hits_out,
                                                             int32_t *__restrict__ size_out) {
    __shared__ int s_hist[1 << kRcBits];
    __shared__ unsigned long long s_cand[kRcCand];
    __shared__ int s_wave[kRcThreads / 64];
    __shared__ unsigned long long s_bits[kRcThreads / 64][2];
    __shared__ int s_digit, s_above, s_equal, s_n, s_l, s_cut;
    if (!plan_matches(pv)) return;   // not this problem's plan: nothing is written
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = rows.row[t];
    const int n = i + 1;
    const int k_top = N_b < n ? N_b : n;
    const unsigned long long *key = ws + (int64_t)t * L;
    for (int x = tid; x < pv.N_q; x += kRcThreads)       // the row's query group
        if (pv.RB[x] <= i && i < pv.RB[x + 1]) s_l = x;

    // ---- threshold: the k_top-th largest key is the want-th largest of the region, the keys whose bits from
    // `shift` up equal `prefix`; above = keys larger than the region's, equal = keys of the region ----
    unsigned long long prefix = 0ull;
    int above = 0, equal = n, shift = 64;
    bool in_lds = false, stuck = false;
    while (shift > 0 && above + equal != k_top) {
        if (!in_lds && equal <= kRcCand) {
            if (tid == 0) s_n = 0;
            __syncthreads();
            for (int j0 = tid; j0 < n; j0 += 8 * kRcThreads) {
                unsigned long long u[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) u[e] = j0 + e * kRcThreads < n ? key[j0 + e * kRcThreads] : 0ull;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (j0 + e * kRcThreads < n && (shift == 64 || (u[e] >> shift) == prefix)) s_cand[atomicAdd(&s_n, 1)] = u[e];
            }
            in_lds = true;
            __syncthreads();
        }
        if (stuck) {                 // the last digit was the same in the whole region: on to the first bit that is not
            unsigned long long ones = 0ull, zeros = 0ull;
            for (int x = tid; x < s_n; x += kRcThreads) {
                const unsigned long long u = s_cand[x];
                if ((u >> shift) == prefix) { ones |= u; zeros |= ~u; }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                ones |= __shfl_xor(ones, off);
                zeros |= __shfl_xor(zeros, off);
            }
            if (lane == 0) { s_bits[wave][0] = ones; s_bits[wave][1] = zeros; }
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kRcThreads / 64; ++w) { ones |= s_bits[w][0]; zeros |= s_bits[w][1]; }
            const unsigned long long low = (1ull << shift) - 1ull, diff = ones & zeros & low;
            const int first = diff ? 64 - __builtin_clzll(diff) : 0;
            prefix = (prefix << (shift - first)) | ((ones & low) >> first);
            shift = first;
            if (shift == 0) break;
        }
        const int bits = in_lds ? (shift < 8 ? shift : 8) : (shift < kRcBits ? shift : kRcBits);
        const int bins = 1 << bits, lower = shift - bits;
        for (int x = tid; x < bins; x += kRcThreads) s_hist[x] = 0;
        __syncthreads();
        if (in_lds) {
            for (int x = tid; x < s_n; x += kRcThreads) {
                const unsigned long long u = s_cand[x];
                if (shift == 64 || (u >> shift) == prefix) atomicAdd(&s_hist[(int)(u >> lower) & (bins - 1)], 1);
            }
        } else {
            for (int j0 = tid; j0 < n; j0 += 8 * kRcThreads) {
                unsigned long long u[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) u[e] = j0 + e * kRcThreads < n ? key[j0 + e * kRcThreads] : 0ull;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (j0 + e * kRcThreads < n && (shift == 64 || (u[e] >> shift) == prefix))
                        atomicAdd(&s_hist[(int)(u[e] >> lower) & (bins - 1)], 1);
            }
        }
        __syncthreads();
        // counts from the largest digit down: thread t holds the digits below bins - per t
        const int per = bins > kRcThreads ? bins / kRcThreads : 1;
        const int want = k_top - above;                  // 1 <= want < equal
        int local = 0;
        if (tid * per < bins)
            for (int e = 0; e < per; ++e) local += s_hist[bins - 1 - tid * per - e];
        const int inc = wave_incl_scan(local);
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        int gt = inc - local;                            // keys of the region with a larger digit
#pragma unroll
        for (int w = 0; w < kRcThreads / 64; ++w) gt += w < wave ? s_wave[w] : 0;
        if (gt < want && gt + local >= want) {           // one thread
            int d = bins - 1 - tid * per;
            while (gt + s_hist[d] < want) gt += s_hist[d--];
            s_digit = d; s_above = gt; s_equal = s_hist[d];
        }
        __syncthreads();
        stuck = in_lds && s_equal == equal;
        above += s_above;
        equal = s_equal;
        prefix = (prefix << bits) | (unsigned long long)s_digit;
        shift = lower;
    }
    // A key belongs to the top set if its bits from `shift` up are above `prefix`, or equal to it and there is room:
    // for the whole region, or (then shift = 0: equal keys) for the lowest-indexed need_eq of it.
    const int need_eq = k_top - above;
    const bool all_eq = need_eq >= equal;
    __syncthreads();                                     // s_l, where the loop did not run
    int cut = n;                                         // the last of them; equal keys from there on are not in the top set
    if (!all_eq) {                                       // a tie cut by the budget
        constexpr int kPer = 8, kW = kRcThreads / 64;    // slabs of kPer rounds of kRcThreads keys; counts of a (round, wave)
        for (int j0 = 0, before = 0; before < need_eq; j0 += kPer * kRcThreads) {   // ends: the region holds more than need_eq
            unsigned long long m[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                const int j = j0 + e * kRcThreads + tid;
                m[e] = __ballot(j < n && key[j < n ? j : 0] == prefix);
                if (lane == 0) s_hist[e * kW + wave] = __popcll(m[e]);
            }
            __syncthreads();
            int run = before;
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                for (int w = 0; w < kW; ++w) {
                    if (w == wave && ((m[e] >> lane) & 1ull) &&
                        run + __popcll(m[e] & ((1ull << lane) - 1ull)) == need_eq - 1)
                        s_cut = j0 + e * kRcThreads + tid;
                    run += s_hist[e * kW + w];
                }
            }
            before = run;
            __syncthreads();
        }
        cut = s_cut;
    }

    // ---- the row's selected keys: one wave per plan entry ----
    const int l = s_l;
    const int v = i + 1 - pv.RB[l];
    const int E = pv.count[(int64_t)head * pv.N_q + l];
    const int32_t *ent = pv.entries + ((int64_t)head * pv.N_q + l) * pv.stride * 2;
    int hits = 0;
    for (int e = wave; e < E; e += kRcThreads / 64) {
        const int w0 = ent[2 * e], rem = ent[2 * e + 1];
        const int k = w0 & kChunkMask, pos = w0 >> kPosShift;
        const int b0 = pv.B[k];
        int take = entry_take(pos, rem, pv.B[k + 1] - b0, v);
        if (pos == 3) {                                  // row-block form: listed keys above the row are masked
            const int vis = i + 1 - b0;
            if (vis < take) take = vis > 0 ? vis : 0;
        }
        for (int x = lane; x < take; x += 64) {
            const int j = b0 + x;
            const unsigned long long u = shift == 64 ? 0ull : key[j] >> shift;   // shift 64: every key is in the top set
            hits += u > prefix || (u == prefix && j <= cut);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) hits += __shfl_xor(hits, off);
    if (lane == 0) s_wave[wave] = hits;
    __syncthreads();
    if (tid == 0) {
        int total = 0;
        for (int w = 0; w < kRcThreads / 64; ++w) total += s_wave[w];
        hits_out[t] = total;
        size_out[t] = k_top;
    }
}

hipError_t launch_recall(const Prob &p, const PlanView &pv, const void *Q, const void *K, int head,
                         const int64_t *rows_host, int n_rows, unsigned long long *ws, int32_t *hits, int32_t *size,
                         hipStream_t s) {
    RecallRows rr;
    for (int t0 = 0; t0 < n_rows; t0 += kRecallRows) {
        rr.n = std::min(kRecallRows, n_rows - t0);
        int last = 0;
        for (int t = 0; t < rr.n; ++t) last = std::max(last, rr.row[t] = (int32_t)rows_host[t0 + t]);
        for (int t = rr.n; t < kRecallRows; ++t) rr.row[t] = 0;
        unsigned long long *w = ws + (int64_t)t0 * p.L;
        const dim3 grid((last + 256 * kLgKeys) / (256 * kLgKeys), (rr.n + kLgRows - 1) / kLgRows), block(256);
#define DHSA_LOGITS(T, DD)                                                                                       \
    hipLaunchKernelGGL((k_recall_logits<T, DD>), grid, block, 0, s, pv, (const T *)Q, (const T *)K, p.G, head, rr, \
                       p.L, w, p.qs_h, p.qs_l, p.ks_h, p.ks_l)
        if (p.dtype == DHSA_F32) {
            if (p.D == 64) DHSA_LOGITS(float, 64); else DHSA_LOGITS(float, 128);
        } else {
            if (p.D == 64) DHSA_LOGITS(bf16_t, 64); else DHSA_LOGITS(bf16_t, 128);
        }
#undef DHSA_LOGITS
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_recall_count, dim3(rr.n), dim3(kRcThreads), 0, s, pv, p.N_b, head, rr, p.L, w, hits + t0,
                           size + t0);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace dhsa
