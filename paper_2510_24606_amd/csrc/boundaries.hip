// Boundary finalisation of libdhsa: boundary scores -> chunk boundaries B
// (Sec. 3.2 "Inference Pipeline"; App. "Inference of the Boundary Predictor":
// drop the positions whose score does not exceed a threshold, visit the rest by
// descending score, keep a position and remove every other candidate within W
// tokens of it).
//
// The greedy is sequential as stated; its result is the unique set in which a
// candidate is kept iff no better candidate within W tokens of it is kept
// ("better" = higher score, equal scores: lower position).  Two kernels build it:
//
//   k_nms_windows (one workgroup per 512 positions) decides in LDS what a window
//     of those positions and a halo on each side can decide.  A decision needs
//     only final facts -- removed: a neighbour is kept; kept: no better neighbour
//     is left -- so it holds whatever the rest of the sequence looks like, and the
//     threads may take their decisions in any order.  A detector's scores (and
//     noise) leave nothing undecided: the chain of candidates a decision hangs on
//     has to rise in score all the way to leave the halo.
//   k_nms_finish (one workgroup) decides what is left in rounds over the whole
//     sequence -- long monotone runs, windows of more tokens than the halo has --
//     and compacts the kept positions into B.
//
// Bound by latency (0.5 MB of scores at L = 131072): 6.4 + 6.2 us, against 1.1 ms when one
// workgroup did all of it in rounds from memory.
//
// Rounds of k_nms_finish: a still undecided candidate that is
// better than every undecided candidate within W tokens is kept (nothing can
// remove it any more), then every undecided candidate within W tokens of a
// newly kept one is removed.  The best undecided candidate of the whole
// sequence is decided in every round, so the loop ends.  A round only visits the 64-position
// blocks in which something can change: a candidate can become the best of its
// neighbourhood only after a better neighbour was removed, so the blocks within W
// of a removal are the next round's work list (three bitmaps in the workspace);
// a long monotone run then costs one cheap round per chunk end instead of a pass
// over the sequence.
#include <algorithm>

#include "dhsa_internal.h"

namespace dhsa {

constexpr int kNmsThreads = 1024;
constexpr int kNmsWaves = kNmsThreads / 64;
enum : uint8_t { kOut = 0, kUndecided = 1, kKept = 2, kNewKept = 3 };

// set the bits of the 64-position blocks that intersect positions [lo, hi]
__device__ __forceinline__ void nms_mark(unsigned *bits, int64_t lo, int64_t hi) {
    for (int64_t b = lo >> 6; b <= (hi >> 6); ++b) atomicOr(&bits[b >> 5], 1u << (b & 31));
}

// Calls body(block) for every block whose bit is set, a whole wave per block, the
// waves sharing the blocks in groups of 64.
#define DHSA_NMS_FOR_BLOCKS(bits, ...)                                                           \
    for (int64_t g0_ = (int64_t)wave * 64; g0_ < NB; g0_ += (int64_t)kNmsWaves * 64) {           \
        const int64_t mine_ = g0_ + lane;                                                        \
        const bool set_ = mine_ < NB && ((bits[mine_ >> 5] >> (mine_ & 31)) & 1u);               \
        unsigned long long m_ = __ballot(set_);                                                  \
        while (m_) {                                                                             \
            const int64_t blk = g0_ + __builtin_ctzll(m_);                                       \
            m_ &= m_ - 1;                                                                        \
            __VA_ARGS__                                                                          \
        }                                                                                        \
    }

// ---------------------------------------------------------------------------
// Local decisions.  The window of workgroup b is [512 b - H, 512 b + 512 + H)
// clipped to the sequence; only its 512 positions are written to st.  `und` and
// `kept` are bitmaps over the window.  A position is marked kept before it stops
// being undecided, and `und` is read before `kept`, so a neighbour on its way
// from one to the other is never missed.
// ---------------------------------------------------------------------------
constexpr int kNmsSeg = 512;                          // positions decided by one workgroup
constexpr int kNmsHaloMax = 512;                      // positions looked at on each side (a multiple of 64)
constexpr int kNmsWinMax = kNmsSeg + 2 * kNmsHaloMax;
// A thread for each position of the smallest window: a round is a chain of LDS reads, which a thread with three positions
// goes through three times: 131072 positions 9.7 -> 6.4 us.
constexpr int kNmsWinThreads = kNmsSeg + 2 * 128;
static_assert(kNmsWinMax % kNmsWinThreads == 0, "whole passes");

__global__ __launch_bounds__(kNmsWinThreads) void k_nms_windows(const float *__restrict__ p, int64_t L, float tau, int W, int H,
                                                     uint8_t *__restrict__ st) {
    __shared__ float s_p[kNmsWinMax];
    __shared__ unsigned long long s_und[kNmsWinMax / 64], s_kept[kNmsWinMax / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t seg0 = (int64_t)blockIdx.x * kNmsSeg;
    const int64_t win0 = seg0 - H > 0 ? seg0 - H : 0;
    const int64_t win1 = seg0 + kNmsSeg + H < L ? seg0 + kNmsSeg + H : L;
    const int n = (int)(win1 - win0);                 // H and kNmsSeg are multiples of 64: so is win0
    const bool open_lo = win0 > 0, open_hi = win1 < L;   // unseen positions on that side
    volatile unsigned long long *und = s_und, *kept = s_kept;

    // candidates: score strictly above the threshold (a NaN never is)
    float pr[kNmsWinMax / kNmsWinThreads];
#pragma unroll
    for (int e = 0; e < kNmsWinMax / kNmsWinThreads; ++e) {
        const int x = e * kNmsWinThreads + tid;
        pr[e] = x < n ? p[win0 + x] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < kNmsWinMax / kNmsWinThreads; ++e) {
        const int x = e * kNmsWinThreads + tid;
        const unsigned long long c = __ballot(x < n && pr[e] > tau);
        s_p[x] = pr[e];
        if (lane == 0) { s_und[x >> 6] = c; s_kept[x >> 6] = 0ull; }
    }
    __syncthreads();
    for (;;) {   // every round but the last decides a candidate
        int decided = 0;
#pragma unroll
        for (int e = 0; e < kNmsWinMax / kNmsWinThreads; ++e) {
            const int x = e * kNmsWinThreads + tid;
            if (x >= n || !((und[x >> 6] >> lane) & 1ull)) continue;
            const float px = pr[e];
            bool blocked = (W > x && open_lo) || (W >= n - x && open_hi);   // an unseen neighbour may be better
            bool removed = false;
            const int lo = x > W ? x - W : 0, hi = W < n - 1 - x ? x + W : n - 1;
            for (int w = lo >> 6; w <= hi >> 6 && !removed; ++w) {
                unsigned long long m = ~0ull;
                if (w == lo >> 6) m &= ~0ull << (lo & 63);
                if (w == hi >> 6) m &= ~0ull >> (63 - (hi & 63));
                unsigned long long u = und[w] & m;
                removed = (kept[w] & m) != 0ull;      // x is undecided, so a kept neighbour is a better one
                while (u && !blocked) {
                    const int y = w * 64 + __builtin_ctzll(u);
                    u &= u - 1;
                    const float py = s_p[y];
                    blocked = py > px || (py == px && y < x);
                }
            }
            if (removed || !blocked) {
                unsigned *k32 = reinterpret_cast<unsigned *>(s_kept), *u32 = reinterpret_cast<unsigned *>(s_und);
                if (!removed) atomicOr(&k32[x >> 5], 1u << (x & 31));
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // kept before no longer undecided
                atomicAnd(&u32[x >> 5], ~(1u << (x & 31)));
                decided = 1;
            }
        }
        if (!__syncthreads_or(decided)) break;
    }
    // states of the segment, four positions per thread; the state array is padded to 256 bytes
    const int64_t at = seg0 + 4 * tid, st_end = (L + 255) / 256 * 256;
    if (tid < kNmsSeg / 4 && at < st_end) {
        const int x = (int)(at - win0);
        unsigned word = 0u;
        if (x < n) {                                  // bits past n are clear
            const unsigned u4 = (unsigned)(s_und[x >> 6] >> (x & 63)) & 15u, k4 = (unsigned)(s_kept[x >> 6] >> (x & 63)) & 15u;
#pragma unroll
            for (int j = 0; j < 4; ++j) word |= (((u4 >> j) & 1u) * kUndecided | ((k4 >> j) & 1u) * kKept) << (8 * j);
        }
        *reinterpret_cast<unsigned *>(st + at) = word;
    }
}

constexpr int kNmsPer = 128;                          // positions per thread and slab in the compaction
constexpr int kNmsStage = 8192;                       // boundaries staged in LDS for coalesced stores

__global__ __launch_bounds__(kNmsThreads) void k_nms_finish(const float *__restrict__ p, int64_t L, int W, uint8_t *st,
                                                            unsigned *bits0, unsigned *bits1, unsigned *bits2,
                                                            int32_t *__restrict__ B_out,
                                                            int32_t *__restrict__ N_c_out) {
    __shared__ int s_cnt[kNmsWaves];
    __shared__ int s_und;          // candidates still undecided
    __shared__ int s_any;          // does the next round have a block to visit?
    __shared__ int s_stage[kNmsStage];
    __shared__ __align__(16) uint16_t s_kept[kNmsThreads * kNmsPer / 16];   // bits of kept positions: a slab, or all of a short sequence
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t NB = (L + 63) >> 6, NW = (NB + 31) >> 5;   // 64-position blocks, bitmap words
    const int64_t n16 = (L + 255) / 256 * 16;                // 16-byte pieces of the state array
    unsigned *dirtyA = bits0, *dirtyB = bits1, *dirtyN = bits2;   // visit now / near a new chunk end / visit next

    // how many candidates the windows left undecided (state kUndecided; no other state has been written yet
    // with its low bit set)
    // A sequence of one slab leaves its kept positions in LDS by the way: with the states read again, 128 bytes in a row for a
    // thread, the kernel took 10.0 us at L = 131072 instead of 6.2.
    const bool once = n16 <= (int64_t)kNmsThreads * 8;
    const auto kept_bits = [](const uint4 &v) {   // kKept is bit 1 of a state byte: gather the bits of 16
        const unsigned w[4] = {(v.x >> 1) & 0x01010101u, (v.y >> 1) & 0x01010101u, (v.z >> 1) & 0x01010101u, (v.w >> 1) & 0x01010101u};
        unsigned bits = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) bits |= ((w[j] * 0x10204080u) >> 28) << (4 * j);
        return (uint16_t)bits;
    };
    int und = 0;
    for (int64_t i = tid; i < n16; i += kNmsThreads * 8) {
        uint4 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t at = i + (int64_t)e * kNmsThreads;
            v[e] = at < n16 ? reinterpret_cast<const uint4 *>(st)[at] : uint4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            und += __popc(v[e].x & 0x01010101u) + __popc(v[e].y & 0x01010101u) + __popc(v[e].z & 0x01010101u) +
                   __popc(v[e].w & 0x01010101u);
            if (once) s_kept[tid + e * kNmsThreads] = kept_bits(v[e]);
        }
    }
    int und_now = __syncthreads_count(und > 0);
    const bool in_lds = once && und_now == 0;
    if (und_now > 0) {             // (the bitmaps serve the rounds only)
        for (int64_t w = tid; w < NW; w += kNmsThreads) { dirtyA[w] = 0xffffffffu; dirtyB[w] = 0u; dirtyN[w] = 0u; }
        // A candidate next to a segment's border may be undecided although the window on the other side of the border
        // has kept a neighbour of it (a better one): it goes first.  From the kept positions, which are more than W
        // apart, to the few candidates beyond their own segment: two passes over the sequence at most, whatever W
        // (from the candidates, 2 W + 1 states each in search of a kept one: 20 of 93 ms at W = 1024, L = 131072).
        for (int64_t g0 = (int64_t)wave * 256; g0 < L; g0 += (int64_t)kNmsWaves * 256) {
            const int64_t i4 = g0 + 4 * lane;
            const unsigned w4 = i4 < n16 * 16 ? *reinterpret_cast<const unsigned *>(st + i4) : 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t seg = (i4 + j) / kNmsSeg * kNmsSeg;
                unsigned long long m = __ballot(((w4 >> (8 * j)) & 255u) == kKept &&
                                                (i4 + j - W < seg || i4 + j + W >= seg + kNmsSeg));
                while (m) {
                    const int64_t i = g0 + 4 * __builtin_ctzll(m) + j, seg0 = i / kNmsSeg * kNmsSeg;
                    m &= m - 1;
                    const int64_t lo = i - W < 0 ? 0 : i - W, hi = i + W > L - 1 ? L - 1 : i + W;
                    for (int64_t x = lo + lane; x < seg0; x += 64)
                        if (st[x] == kUndecided) st[x] = kOut;
                    for (int64_t x = seg0 + kNmsSeg + lane; x <= hi; x += 64)
                        if (st[x] == kUndecided) st[x] = kOut;
                }
            }
        }
        __threadfence_block();
        __syncthreads();
        und = 0;
        for (int64_t i = tid; i < n16; i += kNmsThreads) {
            const uint4 v = reinterpret_cast<const uint4 *>(st)[i];
            und += __popc(v.x & 0x01010101u) + __popc(v.y & 0x01010101u) + __popc(v.z & 0x01010101u) +
                   __popc(v.w & 0x01010101u);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) und += __shfl_xor(und, off);
        if (lane == 0) s_cnt[wave] = und;
        __syncthreads();
        if (tid == 0) {
            int t = 0;
            for (int w = 0; w < kNmsWaves; ++w) t += s_cnt[w];
            s_und = t;
        }
        __syncthreads();
        und_now = s_und;           // read between two barriers: nobody changes s_und before the second one,
        __syncthreads();           // so every thread takes the same decision at the loop head
    }

    while (und_now > 0) {
        if (tid == 0) s_any = 0;   // set again only in phase 2, behind the next barrier
        // ---- phase 1: an undecided candidate that beats every undecided neighbour becomes a chunk end ----
        DHSA_NMS_FOR_BLOCKS(dirtyA, {
            const int64_t i = blk * 64 + lane;
            bool best = false;
            if (i < L && st[i] == kUndecided) {
                const float pi = p[i];
                const int64_t lo = i - W < 0 ? 0 : i - W, hi = i + W > L - 1 ? L - 1 : i + W;
                best = true;
                for (int64_t j = lo; j <= hi && best; ++j) {
                    if (j == i) continue;
                    const uint8_t sj = st[j];   // a neighbour marked in this phase still counts as a rival
                    if (sj != kUndecided && sj != kNewKept) continue;
                    const float pj = p[j];
                    if (pj > pi || (pj == pi && j < i)) best = false;
                }
                if (best) {
                    st[i] = kNewKept;
                    nms_mark(dirtyB, lo, hi);
                }
            }
            const int n_ = __popcll(__ballot(best));
            if (lane == 0 && n_) atomicSub(&s_und, n_);
        })
        __threadfence_block();
        __syncthreads();
        // ---- phase 2: undecided candidates within W tokens of a new chunk end are removed ----
        DHSA_NMS_FOR_BLOCKS(dirtyB, {
            const int64_t j = blk * 64 + lane;
            bool hit = false;
            if (j < L && st[j] == kUndecided) {
                const int64_t lo = j - W < 0 ? 0 : j - W, hi = j + W > L - 1 ? L - 1 : j + W;
                for (int64_t x = lo; x <= hi && !hit; ++x) hit = st[x] == kNewKept;
                if (hit) {
                    st[j] = kOut;
                    nms_mark(dirtyN, lo, hi);   // its neighbours may now be the best of their neighbourhood
                }
            }
            const int n_ = __popcll(__ballot(hit));
            if (lane == 0 && n_) { atomicSub(&s_und, n_); s_any = 1; }
        })
        __threadfence_block();
        __syncthreads();
        // ---- phase 3: the new chunk ends become plain ones; rotate the work lists ----
        DHSA_NMS_FOR_BLOCKS(dirtyA, {
            const int64_t i = blk * 64 + lane;
            if (i < L && st[i] == kNewKept) st[i] = kKept;
        })
        __threadfence_block();
        __syncthreads();
        {
            unsigned *t_ = dirtyA;
            dirtyA = dirtyN;
            dirtyN = t_;
        }
        // no removal but candidates left cannot happen (the best undecided candidate is always
        // visited); should it, every block is visited again rather than looping forever
        und_now = s_und;
        const unsigned fill = (s_any || und_now == 0) ? 0u : 0xffffffffu;
        for (int64_t w = tid; w < NW; w += kNmsThreads) {
            dirtyB[w] = 0u;
            dirtyN[w] = 0u;
            if (fill) dirtyA[w] = fill;
        }
        __threadfence_block();
        __syncthreads();
    }

    // ---- boundaries in the half-open convention: 0, (kept end + 1) ..., L; ascending ----
    // A thread takes kNmsPer consecutive positions of a slab as one bit each; position L-1 is the end
    // of the sequence anyway.
    int base = 1;                              // B_out[0] = 0
    for (int64_t s0 = 0; s0 < L - 1; s0 += (int64_t)kNmsThreads * kNmsPer) {
        const int64_t i0 = s0 + (int64_t)tid * kNmsPer;
        int mine = 0;
        if (!in_lds) {
            __syncthreads();                   // the slab before is done with
#pragma unroll
            for (int e = 0; e < kNmsPer / 16; ++e) {
                const int64_t at = (s0 >> 4) + e * kNmsThreads + tid;
                s_kept[e * kNmsThreads + tid] = kept_bits(at < n16 ? reinterpret_cast<const uint4 *>(st)[at] : uint4{0u, 0u, 0u, 0u});
            }
            __syncthreads();
        }
        const uint4 k4 = *reinterpret_cast<const uint4 *>(&s_kept[tid * (kNmsPer / 16)]);
        unsigned kb[kNmsPer / 32] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
        for (int e = 0; e < kNmsPer / 32; ++e) {
            const int64_t r0 = i0 + 32 * e;
            if (r0 + 32 > L - 1) kb[e] = r0 < L - 1 ? kb[e] & ((1u << (unsigned)(L - 1 - r0)) - 1u) : 0u;
            mine += __popc(kb[e]);
        }
        const int inc = wave_incl_scan(mine);
        __syncthreads();
        if (lane == 63) s_cnt[wave] = inc;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kNmsWaves; ++w) {
            const int x = s_cnt[w];
            if (w < wave) before += x;
            total += x;
        }
        const bool stage = total <= kNmsStage;  // through LDS: B_out may be host memory, where scattered stores cost most
        int at = before + inc - mine;
#pragma unroll
        for (int e = 0; e < kNmsPer / 32; ++e)
            for (unsigned m = kb[e]; m; m &= m - 1u, ++at) {
                const int32_t b = (int32_t)(i0 + 32 * e + __builtin_ctz(m) + 1);
                if (stage) s_stage[at] = b; else B_out[base + at] = b;
            }
        __syncthreads();
        if (stage)
            for (int x = tid; x < total; x += kNmsThreads) B_out[base + x] = s_stage[x];
        base += total;
    }
    if (tid == 0) {
        B_out[0] = 0;
        B_out[base] = (int32_t)L;
        *N_c_out = base;
    }
}

}  // namespace dhsa

namespace {
// workspace: one state byte per position, then three bitmaps with one bit per 64 positions
int64_t nms_state_bytes(int64_t L) { return (L + 255) / 256 * 256; }
int64_t nms_bitmap_bytes(int64_t L) { return (((((L + 63) >> 6) + 31) >> 5) * 4 + 255) / 256 * 256; }
}  // namespace

extern "C" __attribute__((visibility("default"))) size_t dhsa_finalize_boundaries_workspace_bytes(int64_t L) {
    return L >= 1 && L < ((int64_t)1 << 31) ? (size_t)(nms_state_bytes(L) + 3 * nms_bitmap_bytes(L)) : 0;
}

extern "C" __attribute__((visibility("default"))) dhsa_status dhsa_finalize_boundaries(
    const float *scores_dev, int64_t L, float threshold, int32_t window, int32_t *B_dev, int32_t *N_c_dev,
    void *ws_dev, size_t ws_bytes, void *stream) {
    using namespace dhsa;
    if (!scores_dev || !B_dev || !N_c_dev || !ws_dev) return DHSA_ERR_NULL;
    if (L < 1 || L >= ((int64_t)1 << 31) || window < 0 || threshold != threshold) return DHSA_ERR_SHAPE;
    if (ws_bytes < dhsa_finalize_boundaries_workspace_bytes(L)) return DHSA_ERR_WORKSPACE;
    uint8_t *st = (uint8_t *)ws_dev;
    unsigned *bits = (unsigned *)(st + nms_state_bytes(L));
    const int64_t bw = nms_bitmap_bytes(L) / 4;
    // halo: sixteen windows of tokens, where a decision has long been taken in scores that do not rise
    // monotonically; at least 128 positions (cheap), at most what the LDS arrays hold
    const int H = (int)std::min<int64_t>(kNmsHaloMax, std::max<int64_t>(128, ((int64_t)window * 16 + 63) / 64 * 64));
    hipLaunchKernelGGL(k_nms_windows, dim3((unsigned)((L + kNmsSeg - 1) / kNmsSeg)), dim3(kNmsWinThreads), 0, (hipStream_t)stream,
                       scores_dev, L, threshold, (int)window, H, st);
    if (hipGetLastError() != hipSuccess) return DHSA_ERR_HIP;
    hipLaunchKernelGGL(k_nms_finish, dim3(1), dim3(kNmsThreads), 0, (hipStream_t)stream, scores_dev, L, (int)window, st,
                       bits, bits + bw, bits + 2 * bw, B_dev, N_c_dev);
    return hipGetLastError() == hipSuccess ? DHSA_OK : DHSA_ERR_HIP;
}
