// Quality diagnostic of libdhsa: per-row recall of the routed key sets against
// exact top-k attention (App. "Theoretical Analysis", Setup and Notation:
// Recall_i = |I*_i n I_hat_i| / |I*_i|, I*_i = the k keys j <= i with the largest
// attention scores, k = min(N_b, i + 1), equal scores by lower index).
//
// Two kernels:
//   k_recall_logits  logits q_i . k_j, j <= i, in fp64, summed in the order d = 0, 1, ...
//      (the products of bf16 / fp32 values are exact in fp64, so the
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

// Logits by the fp64 matrix unit, 16 sampled rows x 16 keys a product: v_mfma_f64_16x16x4_f64 adds the products of its four
// d to the sum one after the other, d ascending, each rounded once -- the fused multiply-adds of the order above, bit for
// bit (checked against them over 650000 sums of bf16 and fp32 values; infinities and NaN included).  Lane 16 q + n supplies
// d = 4 s + q of row n and of key n to product s.  A wave takes 16 keys; the four lanes of a key read a quarter of its row
// each and deal the elements out among them.  Bound by the rate of the unit (a product of 1024 multiply-adds takes 64
// cycles) and the memory latency in front of it: 48 rows of L = 32768, D = 128 16 us; 24.6 us on the vector unit, with the
// rows' elements broadcast from LDS, whose reads were what took the time; 26 us when every lane read all of its key's row.
// fp32, D = 128, 82 rows of L = 50760: 30 us; 85 us when a lane read its elements one by one, 16 bytes of a row to an
// instruction; 58 us on the vector unit.  With 32 or 64 keys a wave 48 rows of L = 32768 take 1.3 and 5.2 us longer.
constexpr int kLgRows = 16, kLgKeys = 4 * 16;   // rows, keys of a workgroup

typedef double f64x4 __attribute__((ext_vector_type(4)));

// This lane's elements d = 4 s + q of a row, in fp64
template <typename T, int D> struct RecallRow;
template <int D> struct RecallRow<float, D> {
    unsigned v[D / 4];       // the 16-byte pieces 4 m + q of the row, four words each; dealt: v[s] is the element of product s
    __device__ void load(const float *row, int q) {
#pragma unroll
        for (int m = 0; m < D / 16; ++m) {
            const uint4 u = reinterpret_cast<const uint4 *>(row)[4 * m + q];
            v[4 * m] = u.x; v[4 * m + 1] = u.y; v[4 * m + 2] = u.z; v[4 * m + 3] = u.w;
        }
    }
    // Product 4 m + i takes word q of piece 4 m + i: words against pieces, of two halves of the wave, then of two 16s of each
    __device__ void deal() {
#pragma unroll
        for (int m = 0; m < D / 16; ++m) {
            const auto a = __builtin_amdgcn_permlane32_swap(v[4 * m], v[4 * m + 2], false, false);
            const auto b = __builtin_amdgcn_permlane32_swap(v[4 * m + 1], v[4 * m + 3], false, false);
            const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
            const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
            v[4 * m] = c[0]; v[4 * m + 1] = c[1]; v[4 * m + 2] = d[0]; v[4 * m + 3] = d[1];
        }
    }
    __device__ double get(int s, int) const { return (double)__uint_as_float(v[s]); }
};
template <int D> struct RecallRow<bf16_t, D> {
    // w: the 16-byte pieces 4 m + q of the row; v[m][i]: two elements, one of them this lane's, of product 8 m + i
    unsigned w[D / 32][4], v[D / 32][8];
    __device__ void load(const bf16_t *row, int q) {
#pragma unroll
        for (int m = 0; m < D / 32; ++m) {
            const uint4 u = reinterpret_cast<const uint4 *>(row)[4 * m + q];
            w[m][0] = u.x; w[m][1] = u.y; w[m][2] = u.z; w[m][3] = u.w;
        }
    }
    // Product 2 P + half takes element q of four from word 2 half + (q >> 1) of piece P: words 0 and 2 of all four pieces go to
    // the lower half of the wave, 1 and 3 to the upper one, then the two 16s of a half give one another theirs.
    __device__ void deal() {
#pragma unroll
        for (int m = 0; m < D / 32; ++m)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const auto a = __builtin_amdgcn_permlane32_swap(w[m][2 * half], w[m][2 * half + 1], false, false);
                const auto b = __builtin_amdgcn_permlane16_swap(a[0], a[0], false, false);   // pieces 0 and 1 of four
                const auto c = __builtin_amdgcn_permlane16_swap(a[1], a[1], false, false);   // 2 and 3
                v[m][half] = b[0]; v[m][2 + half] = b[1]; v[m][4 + half] = c[0]; v[m][6 + half] = c[1];
            }
    }
    __device__ double get(int s, int q) const {          // the 16 bits of the lane's element, above zeros
        const unsigned x = v[s / 8][s % 8];
        return (double)__uint_as_float(q & 1 ? x & 0xffff0000u : x << 16);
    }
};

template <typename T, int D>
__global__ __launch_bounds__(256, 2) void k_recall_logits(PlanView pv, const T *__restrict__ Q, const T *__restrict__ K,
                                                          int G, int head, RecallRows rows, int64_t L,
                                                          unsigned long long *__restrict__ ws, int64_t qs_h, int64_t qs_l,
                                                          int64_t ks_h, int64_t ks_l) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n16 = lane & 15, q = lane >> 4;
    const int t0 = blockIdx.y * kLgRows;
    const int nr = rows.n - t0 < kLgRows ? rows.n - t0 : kLgRows;
    int my_row = rows.row[t0], last = my_row;   // the lane's row; the last of the group
#pragma unroll
    for (int r = 1; r < kLgRows; ++r) {         // (scalar loads: the vector unit reads kernel arguments from far away)
        const int i = rows.row[t0 + (r < nr ? r : 0)];
        my_row = n16 == r ? i : my_row;
        last = i > last ? i : last;
    }
    const int j0 = blockIdx.x * kLgKeys + wave * 16, j = j0 + n16;   // the lane's key
    if (!plan_matches(pv)) return;   // not this problem's plan: nothing is written
    if (j0 > last) return;           // no row sees these keys
    RecallRow<T, D> kr, qr;
    qr.load(Q + (int64_t)head * qs_h + (int64_t)my_row * qs_l, q);
    kr.load(K + (int64_t)(head / G) * ks_h + (int64_t)(j < last ? j : last) * ks_l, q);   // a row that exists
    __builtin_amdgcn_sched_barrier(0);   // left alone, the scheduler moves the loads next to their use
    qr.deal();
    kr.deal();
    f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < D / 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qr.get(s, q), kr.get(s, q), acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {    // element v of a lane: row 4 v + q, key n
        const int r = 4 * v + q, i = __shfl(my_row, r);
        double x = acc[v];
        if (x == 0.0) x = 0.0;                       // -0.0 ties with +0.0
        const unsigned long long u = (unsigned long long)__double_as_longlong(x);
        if (r < nr && j <= i) ws[(int64_t)(t0 + r) * L + j] = (u >> 63) ? ~u : (u | 0x8000000000000000ull);
    }
}

// ---------------------------------------------------------------------------
// Radix select and count of one row.  The first digits are 14 bits wide (sign, exponent and two bits of
// the mantissa: narrower ones would put most logits into two or three counters) and are
// counted from memory; a region of at most kRcCand keys moves into LDS and is finished there
// with 8-bit digits.  The select ends early when every key of the region belongs to the
// top set.  Bound by the instructions of one CU, which goes through the row's keys twice (256 KB each time at n = 32768;
// 17 us for 48 rows).  Ties at the threshold: where the last equal key of the top set lies is found once, by counting.
// ---------------------------------------------------------------------------
constexpr int kRcThreads = 1024;
constexpr int kRcBits = 14;
constexpr int kRcCand = 4096;

__global__ __launch_bounds__(kRcThreads) void k_recall_count(PlanView pv, int N_b, int head, RecallRows rows, int64_t L,
                                                             const unsigned long long *__restrict__ ws,
                                                             int32_t *__restrict__ hits_out,
                                                             int32_t *__restrict__ size_out) {
    __shared__ __align__(16) int s_hist[1 << kRcBits];
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
    // All keys of a row, eight requested at a time
    const auto for_keys = [&](const auto &get, const auto &body) {
        for (int j0 = tid; j0 < n; j0 += 8 * kRcThreads) {
            decltype(get(0)) u[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) u[e] = get(j0 + e * kRcThreads < n ? j0 + e * kRcThreads : 0);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (j0 + e * kRcThreads < n) body(u[e]);
        }
    };
    const auto whole = [&](int j) { return key[j]; };
    const auto upper = [&](int j) { return reinterpret_cast<const uint2 *>(key)[j].y; };   // (2 j may not fit in 32 bits)
    __syncthreads();
    // Lane x of a wave has plan entry 16 x + wave of every 1024: its chunk's first token and the tokens the row takes
    const int l = s_l;
    const int v = i + 1 - pv.RB[l];
    const int E = pv.count[(int64_t)head * pv.N_q + l];
    const int2 *ent = reinterpret_cast<const int2 *>(pv.entries) + ((int64_t)head * pv.N_q + l) * pv.stride;
    const auto entry = [&](int e, int &b0, int &take) {
        const int2 w = e < E ? ent[e] : int2{0, 0};
        const int k = w.x & kChunkMask, pos = w.x >> kPosShift;
        b0 = pv.B[k];
        take = e < E ? entry_take(pos, w.y, pv.B[k + 1] - b0, v) : 0;
        if (pos == 3) {                                  // row-block form: listed keys above the row are masked
            const int vis = i + 1 - b0;
            if (vis < take) take = vis > 0 ? vis : 0;
        }
    };
    int b0_e, take_e;                                    // of the first 1024: their loads do not wait for the threshold
    entry(lane * (kRcThreads / 64) + wave, b0_e, take_e);

    // ---- threshold: the k_top-th largest key is the want-th largest of the region, the keys whose bits from
    // `shift` up equal `prefix`; above = keys larger than the region's, equal = keys of the region ----
    unsigned long long prefix = 0ull;
    int above = 0, equal = n, shift = 64;
    bool in_lds = false, stuck = false;
    while (shift > 0 && above + equal != k_top) {
        if (!in_lds && equal <= kRcCand) {
            if (tid == 0) s_n = 0;
            __syncthreads();
            const auto take = [&](unsigned long long u) { s_cand[atomicAdd(&s_n, 1)] = u; };
            if (shift == 64) for_keys(whole, take);
            else if (shift >= 32)        // (one CU goes through all keys of the row: 32-bit instructions where they do)
                for_keys(whole, [&](unsigned long long u) { if ((unsigned)(u >> 32) >> (shift - 32) == (unsigned)prefix) take(u); });
            else for_keys(whole, [&](unsigned long long u) { if ((u >> shift) == prefix) take(u); });
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
            if (shift == 64) for_keys(upper, [&](unsigned u) { atomicAdd(&s_hist[u >> (32 - kRcBits)], 1); });
            else for_keys(whole, [&](unsigned long long u) { if ((u >> shift) == prefix) atomicAdd(&s_hist[(int)(u >> lower) & (bins - 1)], 1); });
        }
        __syncthreads();
        // counts from the largest digit down
        const int want = k_top - above;                  // 1 <= want < equal
        if (bins <= kRcThreads) {                        // thread t holds digit bins - 1 - t
            const int local = tid < bins ? s_hist[bins - 1 - tid] : 0;
            const int inc = wave_incl_scan(local);
            if (lane == 63) s_wave[wave] = inc;
            __syncthreads();
            int gt = inc - local;                        // keys of the region with a larger digit
#pragma unroll
            for (int w = 0; w < kRcThreads / 64; ++w) gt += w < wave ? s_wave[w] : 0;
            if (gt < want && gt + local >= want) { s_digit = bins - 1 - tid; s_above = gt; s_equal = local; }   // one thread
        } else {
            // A wave adds up 1024 digits, 16 bytes a lane from one place to the next (16 digits a thread, 16 words apart, met on
            // few banks: 8700 of the kernel's 45000 cycles), then the one that holds the digit looks for it.
            static_assert(1 << kRcBits == kRcThreads / 64 * 1024, "all digits");
            const int4 *top = reinterpret_cast<const int4 *>(s_hist) + (bins - 1024 * wave) / 4 - 1 - lane;   // the lane's largest four
            int4 c[4];
            int sum[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                c[x] = top[-64 * x];
                sum[x] = (c[x].x + c[x].y) + (c[x].z + c[x].w);
            }
            const int all = wave_incl_scan((sum[0] + sum[1]) + (sum[2] + sum[3]));
            if (lane == 63) s_wave[wave] = all;
            __syncthreads();
            int gt = 0;
#pragma unroll
            for (int w = 0; w < kRcThreads / 64; ++w) gt += w < wave ? s_wave[w] : 0;
            if (gt < want && gt + s_wave[wave] >= want) {    // one wave
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int inc = wave_incl_scan(sum[x]);
                    int before = gt + inc - sum[x];
                    if (before < want && before + sum[x] >= want) {
                        const int four[4] = {c[x].w, c[x].z, c[x].y, c[x].x};
                        int d = bins - 1024 * wave - 256 * x - 4 * lane - 1;
                        bool found = false;
#pragma unroll
                        for (int y = 0; y < 4; ++y) {
                            if (!found && before + four[y] >= want) { found = true; s_digit = d - y; s_above = before; s_equal = four[y]; }
                            before += four[y];
                        }
                    }
                    gt += __builtin_amdgcn_readlane(inc, 63);
                }
            }
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

    // ---- the row's selected keys: a wave takes its entries four at a time, 64 keys of each ----
    int hits = 0;
    const auto hit = [&](int j, unsigned long long u64) {
        const unsigned long long u = shift == 64 ? 0ull : u64 >> shift;   // shift 64: every key is in the top set
        return (int)(u > prefix || (u == prefix && j <= cut));
    };
    for (int e0 = 0; e0 < E; e0 += kRcThreads) {
        if (e0 > 0) entry(e0 + lane * (kRcThreads / 64) + wave, b0_e, take_e);
        const int n_e = E - e0 - wave <= 0 ? 0 : (E - e0 - wave + kRcThreads / 64 - 1) / (kRcThreads / 64);   // of this wave
        for (int x = 0; x < n_e && x < 64; x += 4) {
            int b0[4], take[4];
            unsigned long long u[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {                // (lanes past the wave's last entry take nothing)
                b0[c] = __builtin_amdgcn_readlane(b0_e, (x + c) & 63);
                take[c] = x + c < 64 ? __builtin_amdgcn_readlane(take_e, (x + c) & 63) : 0;
                u[c] = lane < take[c] ? key[b0[c] + lane] : 0ull;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (lane < take[c]) hits += hit(b0[c] + lane, u[c]);
                for (int y = lane + 64; y < take[c]; y += 64) hits += hit(b0[c] + y, key[b0[c] + y]);
            }
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
        hipError_t e;
        // rows and keys counted from key0: a later launch gets Q, K and the keys' places moved by as much, and rows above it below 0
        constexpr int64_t step = (int64_t)kGridMax * kLgKeys;
        for (int64_t key0 = 0; key0 <= last; key0 += step) {
            if (key0 > 0)
                for (int t = 0; t < kRecallRows; ++t) rr.row[t] -= (int32_t)step;
            const dim3 grid((unsigned)std::min<int64_t>(kGridMax, (last - key0) / kLgKeys + 1), (rr.n + kLgRows - 1) / kLgRows), block(256);
#define DHSA_LOGITS(T, DD)                                                                                               \
    hipLaunchKernelGGL((k_recall_logits<T, DD>), grid, block, 0, s, pv, (const T *)Q + key0 * p.qs_l,                    \
                       (const T *)K + key0 * p.ks_l, p.G, head, rr, p.L, w + key0, p.qs_h, p.qs_l, p.ks_h, p.ks_l)
            if (p.dtype == DHSA_F32) {
                if (p.D == 64) DHSA_LOGITS(float, 64); else DHSA_LOGITS(float, 128);
            } else {
                if (p.D == 64) DHSA_LOGITS(bf16_t, 64); else DHSA_LOGITS(bf16_t, 128);
            }
#undef DHSA_LOGITS
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        for (int t = 0; last >= step && t < kRecallRows; ++t) rr.row[t] += (int32_t)(last / step * step);
        hipLaunchKernelGGL(k_recall_count, dim3(rr.n), dim3(kRcThreads), 0, s, pv, p.N_b, head, rr, p.L, w, hits + t0,
                           size + t0);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace dhsa
