// Ranking of the chunks for one (head, query group), and its scores where they are made beside it: device code that the
// kernels of several translation units share.
#pragma once
#include "dhsa_internal.h"

namespace dhsa {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Ranking + per-row budget for one (head, query group): Alg. 1's Argsort and walk, done
// once for all rows of the group.  An entry of the plan is a chunk that some row takes
// a token of, with rem = N_b - (tokens of the other chunks ranked before it; the group's own chunk
// left out).  Row-block form (B_r > 0, Alg. 1 as printed): the candidates are the chunks that
// start before the block's end q_max, their lengths are clipped to q_max, there is no "own chunk", and
// an entry records how many tokens of the chunk the block's list holds (pos = 3).
// ---------------------------------------------------------------------------

// order-preserving image of a score and back; -0.0 ties with +0.0
__device__ __forceinline__ unsigned long long score_key(double s) {
    if (s == 0.0) s = 0.0;
    const unsigned long long u = (unsigned long long)__double_as_longlong(s);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
// The score rounded to fp32, in the order of score_key: a NaN lies outside all other scores, on the side of its sign.
__device__ __forceinline__ float score_f32(double s) {
    const float f = (float)s;
    return f == f ? f : __builtin_copysignf(INFINITY, f);
}
__device__ __forceinline__ double key_score(unsigned long long k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

// LDS traffic between the lanes of one wave: the LDS executes a wave's operations in order, so only the
// compiler has to be kept from moving them
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Wider sums and extrema with the steps of wave_incl_scan.
__device__ __forceinline__ unsigned long long wave_incl_scan(unsigned long long x) {
#define DHSA_STEP(CTRL, ROWS)                                                               \
    x += ((unsigned long long)(unsigned)dpp_or<CTRL, ROWS>(0, (int)(unsigned)(x >> 32)) << 32) | \
         (unsigned long long)(unsigned)dpp_or<CTRL, ROWS>(0, (int)(unsigned)x);
    DHSA_DPP_STEPS(DHSA_STEP)
#undef DHSA_STEP
    return x;
}
__device__ __forceinline__ float wave_max(float x) {
#define DHSA_STEP(CTRL, ROWS) x = fmaxf(x, __int_as_float(dpp_or<CTRL, ROWS>(__float_as_int(x), __float_as_int(x))));
    DHSA_DPP_STEPS(DHSA_STEP)
#undef DHSA_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ unsigned long long wave_read(unsigned long long x, int src) {   // src: wave-uniform
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), src) << 32) |
           (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, src);
}

// ---------------------------------------------------------------------------
// NW waves per (head, query group).  Only chunks that some row takes a token of need a
// rank, and the tokens ranked before such a chunk are all that is wanted of it:
//   1. scores of the visible chunks into registers (eight per lane at a time), their range;
//   2. tokens and chunks per score bin (256 bins over the range, best first; packed tokens << 16 | chunks,
//      LDS atomics): the bin where the tokens reach N_b is the last one that can hold a listed
//      chunk, whatever the order inside it, so the chunks up to that bin are the candidates.  If
//      they are more than the list holds, the last bin is cut again over its own range (outliers
//      far from the rest), and at last by digits of the keys and ids (ties);
//   3. candidates into LDS, grouped by bin (the bins' counts are their places);
//   4. tokens before a candidate = tokens of better bins + of the better candidates of its own bin (a few; with a
//      bin of many, a prefix sum over the sorted candidates);
//   5. the listed chunks set their bit, and go into the plan at the number of bits below theirs
//      (ascending chunk id).
// Bins are taken from the scores rounded to fp32 (which keeps their order), the order inside a bin from the fp64
// scores.  Bound by instruction issue and by the scores' way from memory (342 MB for 1634 chunks x 32 heads).  That
// case takes 256 us; it took 480 us with a radix select by 8-bit digits (whose first digit counts nearly all
// scores in two or three LDS words), a bitonic sort and two scans, with ~40 block barriers.
// ---------------------------------------------------------------------------
constexpr int kSelBins = 256;
constexpr int kSelPer = 8;           // scores per lane in registers
constexpr int kSelCrowd = 32;        // candidates in one bin that are still compared with one another
constexpr int kSelMaxStride = 1024;  // listed chunks this kernel can hold; with more the whole row is sorted (below)

inline int select_cap(int stride) { return (stride + 2 + 32 + 63) / 64 * 64; }   // some to spare before a bin is cut again
inline int select_row_bytes(int NW, int cap, int N_c) {   // cap: a multiple of 64
    return kSelBins * (NW == 1 ? 8 : 16) + cap * 20 + (N_c + 63) / 64 * 8;
}

// Launch arguments.
struct SelectArgs {
    int32_t *plan;
    PlanLayout pl;
    int N_c, N_b, B_r;
    int l_first, n_groups;   // the groups of the launch, laid out from 0: l indexes Sc, RB and the plan, l_first + l is the group's number
    int r_first, n_rows, cap, row_bytes;
};

// The chunks a query group ranks: own = the group's own chunk, q_max = the clip of the chunk lengths, n = visible chunks 0..n-1
struct Visible {
    int own, q_max, n;
};
__device__ __forceinline__ Visible visible_chunks(const SelectArgs &a, const int32_t *B, int l) {
    const int lane = threadIdx.x & 63, N_c = a.N_c;
    const bool blocks = a.B_r > 0;
    const int q_max = blocks ? (a.plan + a.pl.off_RB)[l + 1] : 0x7fffffff;
    const int own = blocks ? -1 : a.l_first + l;
    int n = own + 1;
    if (blocks) {                        // the chunks that start before q_max: B ascends, 64-ary search
        int step = (N_c + 63) >> 6;
        n = (__popcll(__ballot(lane * step < N_c && B[lane * step < N_c ? lane * step : 0] < q_max)) - 1) * step;   // B[0] = 0 < q_max
        int got = 0;
        for (int k0 = 0; k0 < step; k0 += 64) {
            const int k = n + k0 + lane;
            got += __popcll(__ballot(k0 + lane < step && k < N_c && B[k < N_c ? k : 0] < q_max));
        }
        n = __builtin_amdgcn_readfirstlane(n + got);
    }
    return {own, q_max, n};
}

// Ranks the scores row[0 .. vis.n) of a group and calls put(i, first word, second word) for the entries of its list, in any
// order; returns their number.  mine8: row_bytes of LDS, s_red: NW words of it.  row and B in memory or LDS.
template <int NW, typename PUT>
__device__ __forceinline__ int select_row(const SelectArgs &a, const double *row, const int32_t *B, const Visible vis,
                                          unsigned char *mine8, unsigned long long *s_red, const PUT &put) {
    constexpr int NT = 64 * NW, PER = kSelPer, kSlab = PER * NT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = NW == 1 ? lane : (int)threadIdx.x;                     // thread of the row
    const int N_c = a.N_c, N_b = a.N_b, cap = a.cap;
    const int stride = a.pl.stride;
    const auto sync = [] { if constexpr (NW == 1) wave_lds_fence(); else __syncthreads(); };
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(mine8);              // [kSelBins]
    unsigned long long *place = NW == 1 ? hist : hist + kSelBins;                          // [kSelBins] (one wave: in place)
    unsigned long long *ckey = place + kSelBins;                                           // [cap]
    unsigned long long *kept = ckey + cap;                                                 // [ceil(N_c / 64)]
    int *cid = reinterpret_cast<int *>(kept + ((N_c + 63) >> 6));                          // [cap]  id | pos << kPosShift
    int *clen = cid + cap, *crem = clen + cap;                                             // [cap]
    const bool blocks = a.B_r > 0;
    const int own = vis.own, q_max = vis.q_max, n = vis.n;
    // (an unsigned offset: a 64-bit address per lane that lives through the rare passes has no registers)
    const auto score_at = [&](int x) { return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(row) + 8u * (unsigned)x); };
    const auto len_at = [&](int x) {
        const int b0 = B[x], b1 = B[x + 1];
        return x == own ? 0 : (b1 < q_max ? b1 : q_max) - b0;
    };

    double v[PER];
    int len[PER];
    const auto load = [&](int x0) {      // a thread past the end repeats the last chunk
#pragma unroll
        for (int e = 0; e < PER; ++e)
            if (x0 + e * NT < n) {
                const int x = x0 + e * NT + t < n ? x0 + e * NT + t : n - 1;
                v[e] = score_at(x);
                len[e] = len_at(x);
            }
    };
// BODY for every visible chunk x (in: it exists) with score s and length n_tok, whole waves; rows longer than the
// registers hold are read again in every pass
#define DHSA_SEL_FOR(...)                                                                    \
    for (int x0_ = 0; x0_ < n; x0_ += kSlab) {                                               \
        if (n > kSlab) load(x0_);                                                            \
        _Pragma("unroll") for (int e_ = 0; e_ < PER; ++e_) {                             \
            if (x0_ + e_ * NT < n) {                                                         \
                const int x = x0_ + e_ * NT + t;                                             \
                const bool in = x < n;                                                       \
                const double s = v[e_];                                                      \
                const int n_tok = len[e_];                                                   \
                __VA_ARGS__                                                                  \
            }                                                                                \
        }                                                                                    \
    }
// the same for the rare passes, always from memory
#define DHSA_SEL_AGAIN(...)                                                                  \
    _Pragma("unroll 1") for (int x0_ = 0; x0_ < n; x0_ += NT) {                              \
        const int x = x0_ + t;                                                               \
        const bool in = x < n;                                                               \
        const double s = score_at(in ? x : n - 1);                                                \
        const int n_tok = len_at(in ? x : n - 1);                                            \
        __VA_ARGS__                                                                          \
    }
    // over the threads of the row (NW > 1: two barriers)
    const auto row_range = [&](float &lo_, float &hi_) {
        hi_ = wave_max(hi_);
        lo_ = -wave_max(-lo_);
        if constexpr (NW > 1) {
            __syncthreads();
            if (lane == 0)
                s_red[wave] = ((unsigned long long)__float_as_uint(lo_) << 32) | __float_as_uint(hi_);
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const unsigned long long x = s_red[w];
                lo_ = fminf(lo_, __uint_as_float((unsigned)(x >> 32)));
                hi_ = fmaxf(hi_, __uint_as_float((unsigned)x));
            }
            lo_ = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(lo_)));   // the same in all lanes:
            hi_ = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(hi_)));   // no vector registers
        }
    };
    const auto row_min = [&](unsigned long long x) {     // NW > 1: two barriers
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(x, off);
            x = o < x ? o : x;
        }
        if constexpr (NW > 1) {
            __syncthreads();
            if (lane == 0) s_red[wave] = x;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) x = s_red[w] < x ? s_red[w] : x;
        }
        return wave_read(x, 0);          // a wave-uniform value needs no vector registers
    };
    const auto clear_hist = [&] {
        sync();                          // everybody has read the last counts
        for (int b = t; b < kSelBins; b += NT) hist[b] = 0ull;
        sync();
    };

    for (int b = t; b < kSelBins; b += NT) hist[b] = 0ull;
    if (n <= kSlab) load(0);
    const unsigned long long k_own = score_key(own >= 0 ? row[own] : 0.0);
    float lo = INFINITY, hi = -INFINITY, inv;
    DHSA_SEL_FOR({ (void)x; (void)in; (void)n_tok; lo = fminf(lo, score_f32(s)); hi = fmaxf(hi, score_f32(s)); })
    row_range(lo, hi);
    if constexpr (NW == 1) wave_lds_fence();   // hist is clear (NW > 1: row_range has a barrier)
    const float best = hi;
    const auto bin_of = [&](double s) {  // never decreasing as s falls
        return (int)fminf(fmaxf((hi - score_f32(s)) * inv, 0.f), (float)(kSelBins - 1));   // inf - inf: bin 0
    };

    // candidates: chunks ranked at or before (cut_key, cut_id) once that is known (cut), or those of the bins up to tbin
    bool cut = false;
    unsigned long long cut_key = 0ull;
    int cut_id = 0x7fffffff, tbin;
    const auto is_cand = [&](double s, int x) {
        const unsigned long long k = score_key(s);
        return k > cut_key || (k == cut_key && x <= cut_id);
    };
    unsigned long long above = 0ull;     // tokens << 16 | chunks with a score above hi
    unsigned long long before, upto;     // ranked before the last bin, and up to it
    bool crowded;                        // some bin of candidates holds more than kSelCrowd of them
    // From the counts in hist, every wave for itself: what is ranked before each bin (tokens, and chunks = the place of
    // its first) goes to place; the last bin is the one in which the tokens reach N_b (none does: the worst of all)
    const auto find_last = [&] {
        sync();
        unsigned long long c[4];         // bins 4 lane .. 4 lane + 3
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = hist[4 * lane + i];
        const unsigned long long mine = c[0] + c[1] + c[2] + c[3];
        unsigned long long run = above + wave_incl_scan(mine) - mine;
        int my_bin = kSelBins;           // the bin of this lane in which the tokens reach N_b
        before = upto = 0ull;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (NW == 1 || wave == 0) place[4 * lane + i] = run;
            if ((run >> 16) < (unsigned long long)N_b && ((run + c[i]) >> 16) >= (unsigned long long)N_b) {
                my_bin = 4 * lane + i;
                before = run;
                upto = run + c[i];
            }
            run += c[i];
        }
        const unsigned long long found = __ballot(my_bin < kSelBins);
        const int src = found ? __builtin_ctzll(found) : 63;
        tbin = found ? __builtin_amdgcn_readlane(my_bin, src) : kSelBins - 1;
        before = wave_read(before, src);
        upto = wave_read(found ? upto : run, src);
        crowded = false;
        if ((int)(upto & 0xffffull) > kSelCrowd) {
            int most = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n_bin = (int)c[i] & 0xffff;
                most = (cut || 4 * lane + i <= tbin) && n_bin > most ? n_bin : most;
            }
            crowded = __ballot(most > kSelCrowd) != 0ull;
        }
    };
    for (int level = 0;; ++level) {
        inv = hi > lo ? fminf((float)kSelBins / (hi - lo), 1e30f) : 0.f;
        if (level == 0) {
            DHSA_SEL_FOR({ (void)x; if (in) atomicAdd(&hist[bin_of(s)], ((unsigned long long)n_tok << 16) | 1ull); })
        } else {
            clear_hist();
            DHSA_SEL_AGAIN({
                if (in && (cut ? is_cand(s, x) : (score_f32(s) >= lo && score_f32(s) <= hi)))
                    atomicAdd(&hist[bin_of(s)], ((unsigned long long)n_tok << 16) | 1ull);
            })
        }
        find_last();
        if (cut) {
            tbin = kSelBins - 1;
            break;
        }
        int n_upto = (int)(upto & 0xffffull);                    // chunks up to the last bin
        if (n_upto <= cap && level == 0) break;                  // the usual end
        if (n_upto <= cap) {             // group all candidates over one range: from the worst of them to the best
            float worst = INFINITY, none = -INFINITY;
            DHSA_SEL_AGAIN({
                (void)x; (void)n_tok;
                if (in && (score_f32(s) > hi || (score_f32(s) >= lo && bin_of(s) <= tbin))) worst = fminf(worst, score_f32(s));
            })
            row_range(worst, none);
            lo = worst;
            // every score that rounds to `worst` or more: the smallest such key
            unsigned long long key_lo = ~0ull;
            DHSA_SEL_AGAIN({
                (void)x; (void)n_tok;
                const unsigned long long k = score_key(s);
                if (in && score_f32(s) >= worst && k < key_lo) key_lo = k;
            })
            cut_key = row_min(key_lo);
        } else if (level < 3 && hi > lo) {   // cut the last bin again, over its own range
            float a = INFINITY, z = -INFINITY;
            DHSA_SEL_AGAIN({
                (void)x; (void)n_tok;
                if (in && score_f32(s) >= lo && score_f32(s) <= hi && bin_of(s) == tbin) { a = fminf(a, score_f32(s)); z = fmaxf(z, score_f32(s)); }
            })
            above = before;
            row_range(a, z);
            lo = a;
            hi = z;
            continue;
        } else {
            // (Nearly) equal scores: the last bin holds the keys k_lo .. k_hi.  It is cut by 8-bit digits of the keys from
            // the first one they differ in, then, where all keys left are equal, by the id: no more digits than it takes
            // to be left with `cap` chunks.  Keys all zero, 8 heads: routing of 820 chunks 131 us (358 us bit by bit, 78 passes
            // over the row; a radix select of the whole row 330 us), of 205 chunks 33 us (92; 30), of 1570 chunks 457 us.
            unsigned long long k_lo = ~0ull, k_hi = ~0ull;       // k_hi: complemented
            DHSA_SEL_AGAIN({
                (void)x; (void)n_tok;
                if (in && score_f32(s) >= lo && score_f32(s) <= hi && bin_of(s) == tbin) {
                    const unsigned long long k = score_key(s);
                    k_lo = k < k_lo ? k : k_lo;
                    k_hi = ~k < k_hi ? ~k : k_hi;
                }
            })
            k_lo = row_min(k_lo);
            k_hi = ~row_min(k_hi);
            for (int d = 0; d < 8 && n_upto > cap && k_lo != k_hi; ++d) {
                const int top = 64 - __builtin_clzll(k_lo ^ k_hi), low = top > 8 ? top - 8 : 0;   // the digit: bits low .. top - 1
                above = before;
                clear_hist();
                DHSA_SEL_AGAIN({
                    (void)x;
                    const unsigned long long k = score_key(s);
                    if (in && k >= k_lo && k <= k_hi)
                        atomicAdd(&hist[kSelBins - 1 - (int)((k >> low) & (kSelBins - 1))], ((unsigned long long)n_tok << 16) | 1ull);
                })
                find_last();
                n_upto = (int)(upto & 0xffffull);
                const unsigned long long rest = (1ull << low) - 1ull;
                const unsigned long long first = (((k_hi >> low) & ~(kSelBins - 1ull)) | (unsigned long long)(kSelBins - 1 - tbin)) << low;
                k_lo = first > k_lo ? first : k_lo;
                k_hi = (first | rest) < k_hi ? first | rest : k_hi;
            }
            cut_key = k_lo;
            for (int i = 1; n_upto > cap && i >= 0; --i) {       // 64 ids a bin, then each
                above = before;
                clear_hist();
                DHSA_SEL_AGAIN({
                    if (in && score_key(s) == cut_key && (i == 1 || x >> 6 == cut_id >> 6))
                        atomicAdd(&hist[i == 1 ? x >> 6 : x & 63], ((unsigned long long)n_tok << 16) | 1ull);
                })
                find_last();
                n_upto = (int)(upto & 0xffffull);
                cut_id = i == 1 ? tbin * 64 + 63 : (cut_id & ~63) + tbin;
            }
            lo = score_f32(key_score(cut_key));
        }
        cut = true;                      // one more level: the bins of the candidates alone
        above = 0ull;
        hi = best;
    }
    for (int w = t; w < ((n + 63) >> 6); w += NT) kept[w] = 0ull;
    sync();

    // ---- candidates, grouped by bin: the chunk count in place[bin] moves from the place of its first to its end ----
    DHSA_SEL_FOR({
        const int bin = bin_of(s);
        if (in && (cut ? is_cand(s, x) : bin <= tbin)) {
            const int at = (int)(atomicAdd(&place[bin], 1ull) & 0xffffull);
            const unsigned long long k = score_key(s);
            const int pos = blocks ? 3 : x == own ? 1 : (k > k_own || (k == k_own && x < own)) ? 0 : 2;
            if (at < cap) { ckey[at] = k; cid[at] = x | (pos << kPosShift); clen[at] = n_tok; }
        }
    })
#undef DHSA_SEL_FOR
#undef DHSA_SEL_AGAIN
    sync();
    int n_c = __builtin_amdgcn_readfirstlane((int)(place[tbin] & 0xffffull));
    n_c = n_c < cap ? n_c : cap;

    // A bin that holds many (ties; all scores but an outlier's) would cost their number squared: the list is sorted
    // instead, by a network whose comparisons all put the better one first, so that nothing is moved past its end,
    // and the tokens before each candidate are a prefix sum.  Routing of 820 chunks, 32 heads, keys all zero: 1070 ->
    // 223 us; 500 chunks of one token, 12 heads, with outliers: 874 -> 160 us (ordinary scores: 78 us)
    if (__builtin_expect(crowded, 0)) {
        const auto first = [&](unsigned long long ka, int wa, unsigned long long kb, int wb) {
            return ka > kb || (ka == kb && (wa & kChunkMask) < (wb & kChunkMask));
        };
        bool any = false;                // equal scores, taken in ascending order of the ids, are in order already
        for (int c = t; c + 1 < n_c; c += NT) any |= first(ckey[c + 1], cid[c + 1], ckey[c], cid[c]);
        any = __any(any);
        if constexpr (NW > 1) {
            if (lane == 0) s_red[wave] = any;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) any |= s_red[w] != 0ull;
        }
        int half = any ? 1 : 0;
        while (any && 2 * half < n_c) half *= 2;
#pragma unroll 1
        for (int size = 1; size <= half; size *= 2) {    // runs of `size` are in order: join two, the second one reversed
#pragma unroll 1
            for (int step = size; step > 0; step >>= 1) {
#pragma unroll 1
                for (int p = t; p < half; p += NT) {
                    const int in_run = p & (step - 1), lo_at = 2 * p - in_run;
                    const int hi_at = step == size ? lo_at + 2 * (step - in_run) - 1 : lo_at + step;
                    if (hi_at >= n_c) continue;
                    const unsigned long long ka = ckey[lo_at], kb = ckey[hi_at];
                    const int wa = cid[lo_at], wb = cid[hi_at];
                    if (first(kb, wb, ka, wa)) {
                        ckey[lo_at] = kb;
                        ckey[hi_at] = ka;
                        cid[lo_at] = wb;
                        cid[hi_at] = wa;
                    }
                }
                sync();
            }
        }
        for (int c = t; c < n_c; c += NT) clen[c] = len_at(cid[c] & kChunkMask);   // (the lengths were left where they were)
        sync();
        if (NW == 1 || wave == 0) {
            const int per = (n_c + 63) >> 6, c0 = lane * per, c1 = c0 + per < n_c ? c0 + per : n_c;
            int mine = 0;
            for (int c = c0; c < c1; ++c) mine += clen[c];
            int run = wave_incl_scan(mine) - mine;
            for (int c = c0; c < c1; ++c) {
                crem[c] = run;
                run += clen[c];
            }
        }
        sync();
    }
    // ---- tokens ranked before each candidate, and whether some row takes a token of it ----
    for (int c = t; c < n_c; c += NT) {
        const unsigned long long k = ckey[c];
        const int w = cid[c], x = w & kChunkMask, pos = w >> kPosShift;
        int run;
        if (crowded) {
            run = crem[c];
        } else {
            const int bin = bin_of(key_score(k));
            const unsigned long long pb = place[bin];
            const int j1 = (int)(pb & 0xffffull) < n_c ? (int)(pb & 0xffffull) : n_c;
            run = (int)(pb >> 16);
            for (int j = bin > 0 ? (int)(place[bin - 1] & 0xffffull) : 0; j < j1; ++j) {
                const unsigned long long kj = ckey[j];
                const int lj = clen[j];
                if (kj > k || (kj == k && (cid[j] & kChunkMask) < x)) run += lj;
            }
        }
        int rem = N_b - run;
        const bool need = (pos == 2) ? (rem > 1) : (rem > 0);
        if (blocks && rem > clen[c]) rem = clen[c];     // tokens of the chunk in the block's list
        crem[c] = need ? rem : 0;
        if (need) atomicOr(&kept[x >> 6], 1ull << (x & 63));
    }
    sync();

    // ---- into the plan in ascending chunk id: listed chunks below word 2 lane + {0, 1} of `kept` ----
    const int nw = (n + 63) >> 6;                       // at most 128
    const int c0 = 2 * lane < nw ? __popcll(kept[2 * lane]) : 0, c1 = 2 * lane + 1 < nw ? __popcll(kept[2 * lane + 1]) : 0;
    const int listed = wave_incl_scan(c0 + c1);
    const int total = __builtin_amdgcn_readlane(listed, 63);
    for (int cb = 0; cb < n_c; cb += NT) {              // whole waves: the shuffles need their lanes
        const int c = cb + t < n_c ? cb + t : n_c - 1;
        const int rem = cb + t < n_c ? crem[c] : 0, w = cid[c], x = w & kChunkMask, word = x >> 6;
        const int even = __shfl(listed - c0 - c1, word >> 1), odd = __shfl(listed - c1, word >> 1);   // all lanes read
        const int below = (word & 1) ? odd : even;
        const int slot = below + __popcll(kept[word] & ((1ull << (x & 63)) - 1ull));
        if (rem > 0 && slot < stride) put(slot, w, rem);
    }
    return total < stride ? total : stride;
}

// ---------------------------------------------------------------------------
// The same for at most X chunks (a multiple of 64) by a workgroup of NT threads: every chunk is compared with every other one,
// chunk x by the threads x, x + X, .. which share the others: no bins, two barriers.  Of a decoding step of 38 chunks the
// ranking had been 8000 of 27500 cycles; with this one, and pooled keys that are requested first, 15.1 -> 13.0 us a step.  The number of entries is returned to the first wave only.
// ---------------------------------------------------------------------------
template <int NT, int X>
struct FewSmem {
    unsigned long long key[X];
    int len[X];
    int run[NT / X][X];
};
template <int NT, int X, typename PUT>
__device__ __forceinline__ int select_few(const SelectArgs &a, const double *row, const int32_t *B, const Visible vis,
                                          FewSmem<NT, X> &sm, const PUT &put) {
    static_assert(X % 64 == 0 && NT % X == 0, "the threads of a wave share their part of the chunks");
    constexpr int PARTS = NT / X;
    const int n = vis.n, x = threadIdx.x % X, part = __builtin_amdgcn_readfirstlane(threadIdx.x / X);
    const unsigned long long k = x < n ? score_key(row[x]) : 0ull;
    if (part == 0 && x < n) {
        const int b0 = B[x], b1 = B[x + 1];
        sm.key[x] = k;
        sm.len[x] = x == vis.own ? 0 : (b1 < vis.q_max ? b1 : vis.q_max) - b0;
    }
    __syncthreads();
    int run = 0;
#pragma unroll 4
    for (int j = part; j < n; j += PARTS) {
        const unsigned long long kj = sm.key[j];
        const int lj = sm.len[j];
        run += (kj > k || (kj == k && j < x)) ? lj : 0;
    }
    sm.run[part][x] = run;
    __syncthreads();
    if (threadIdx.x >= 64) return 0;
    const unsigned long long k_own = vis.own >= 0 ? sm.key[vis.own] : 0ull;
    int total = 0;
#pragma unroll
    for (int x0 = 0; x0 < X; x0 += 64) {             // into the list in ascending chunk id
        const int c = x0 + threadIdx.x;
        int before = 0;
#pragma unroll
        for (int p = 0; p < PARTS; ++p) before += sm.run[p][c];
        const unsigned long long kc = sm.key[c < n ? c : n - 1];
        const int pos = a.B_r > 0 ? 3 : c == vis.own ? 1 : (kc > k_own || (kc == k_own && c < vis.own)) ? 0 : 2;
        int rem = a.N_b - before;
        const bool need = c < n && ((pos == 2) ? (rem > 1) : (rem > 0));
        if (a.B_r > 0 && c < n && rem > sm.len[c]) rem = sm.len[c];   // tokens of the chunk in the block's list
        const unsigned long long all = __ballot(need);
        const int i = total + __builtin_amdgcn_mbcnt_hi((unsigned)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)all, 0));
        if (need && i < a.pl.stride) put(i, c | (pos << kPosShift), rem);
        total += __popcll(all);
    }
    return total < a.pl.stride ? total : a.pl.stride;
}

// ---------------------------------------------------------------------------
// Scores of one query group against 16 chunks, one of them per lane & 15, by a wave: the group's vector is repeated as all 16
// rows, so that a score is made of the same products in the same order as in k_scores.  b: this lane's pieces of its chunk's
// pooled vector.  The result is in all lanes of a chunk.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void load_pooled(f64x2 (&to)[D / 8], const double *pooled) {
    const int q = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int s = 0; s < D / 8; ++s) to[s] = *reinterpret_cast<const f64x2 *>(pooled + 2 * q + 8 * s);
}
template <int D>
__device__ __forceinline__ double score_16(const f64x2 (&a)[D / 8], const f64x2 (&b)[D / 8]) {
    f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < D / 8; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][j], b[s][j], acc, 0, 0, 0);
    return acc[0];
}

// Plan entries of a query group and the boundaries, in memory or LDS.
struct TileList {
    const int2 *ent;
    int E;
    const int32_t *B;
};
__device__ __forceinline__ TileList plan_list(const PlanView &pv, int h, int l) {
    const int64_t group = (int64_t)h * pv.N_q + l;
    return {reinterpret_cast<const int2 *>(pv.entries) + group * pv.stride, pv.count[group], pv.B};
}

// ---------------------------------------------------------------------------
// Scores and ranking for a row tile of group l of head h by its own workgroup of 256 threads, as k_score_select makes them; the
// list stays in LDS, and the first tile of a group (`first`) also writes it, and the scores, where they always are.
// ---------------------------------------------------------------------------
constexpr int kRouteAttendMax = 64;   // chunks: 16 for each wave
struct RouteScratch {
    double row[kRouteAttendMax];
    FewSmem<256, kRouteAttendMax> few;
    int2 ent[kRouteAttendMax];
    int32_t B[kRouteAttendMax + 1];
    int count;
};

template <int D>
__device__ __forceinline__ TileList route_tile(RouteScratch &rs, const PlanView &pv, const SelectArgs &sel, const double *Qc,
                                               const double *Kc, double *Sc, int G, int h, int l, bool first) {
    const int64_t group = (int64_t)h * pv.N_q + l;
    const int tid = threadIdx.x, lane = tid & 63, k0 = (tid >> 6) * 16, k = k0 + (lane & 15);
    const Visible vis = visible_chunks(sel, pv.B, l);
    if (tid <= sel.N_c) rs.B[tid] = pv.B[tid];
    if (k0 < vis.n) {
        f64x2 q[D / 8], b[D / 8];
        load_pooled<D>(b, Kc + ((int64_t)(h / G) * sel.N_c + (k < vis.n ? k : vis.n - 1)) * D);
        load_pooled<D>(q, Qc + group * D);
        __builtin_amdgcn_sched_barrier(0);   // left alone, the scheduler moves the loads next to their use
        const double score = score_16<D>(q, b);
        if (lane < 16 && k < vis.n) {
            rs.row[k] = score;
            if (first) Sc[group * sel.N_c + k] = score;
        }
    }
    __syncthreads();
    int2 *entries = reinterpret_cast<int2 *>(sel.plan + sel.pl.off_entries) + group * sel.pl.stride;
    const int n = select_few<256, kRouteAttendMax>(sel, rs.row, rs.B, vis, rs.few, [&](int i, int w, int rem) {
        rs.ent[i] = make_int2(w, rem);
        if (first) entries[i] = make_int2(w, rem);
    });
    if (tid == 0) {
        rs.count = n;
        if (first) sel.plan[sel.pl.off_count + group] = n;
    }
    __syncthreads();
    return {rs.ent, __builtin_amdgcn_readfirstlane(rs.count), rs.B};
}

}  // namespace dhsa
