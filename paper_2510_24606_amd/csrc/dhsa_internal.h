// Internal declarations shared by the HIP translation units of libdhsa.
// Nothing here is part of the C ABI (see include/dhsa.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dhsa.h"

namespace dhsa {

constexpr int kRowTile = DHSA_ROW_TILE;  // query rows per attention workgroup
constexpr int kMaxChunks = 8192;         // N_c limit (LDS ranking of one query chunk)
constexpr int kPosShift = 28;            // plan entry word 0 = chunk id | pos << 28
constexpr int kChunkMask = (1 << kPosShift) - 1;

// Resolved problem: strides filled in, budget clamped, scale chosen.
struct Prob {
    int64_t L;
    int H_q, H_kv, G, D, N_c, N_b;  // N_b already clamped to L
    int B_r, N_q;                   // row-block size (0 = query groups are the chunks), query groups
    int pooling;                    // dhsa_pooling
    int dtype;
    float scale;
    int64_t qs_h, qs_l, ks_h, ks_l, vs_h, vs_l, os_h, os_l;
};

constexpr int kPlanHeaderWords = DHSA_PLAN_HEADER_WORDS;

// Word offsets inside the plan buffer (see the layout comment in dhsa.h).
struct PlanLayout {
    int stride;       // entries per (h, l)
    int T1;           // row tiles per head
    int T_big;        // ... of which have more than 64 rows (listed first)
    int T_cls[4];     // tiles of > 96, 65..96, 33..64 and <= 32 rows: the order of the tile table
    int N_q;          // query groups (chunks, or row blocks)
    int b_sum;        // checksum of the boundaries (header word 17)
    int64_t off_B, off_RB, off_count, off_entries, off_tiles, words;
};

// What the caller's problem says a plan must have been built for.  Every kernel that reads a plan
// compares this with the plan's header first and leaves without writing anything if they differ
// (a plan routed for another budget, row-block size, representation or boundary array of equal
// size would otherwise be used silently).
struct PlanSig {
    int32_t H_q, N_c, N_b, L, B_r, N_q, pooling, b_sum, stride, T1;
};

// Device-side view of a plan.
struct PlanView {
    const int32_t *hdr;      // [kPlanHeaderWords]
    PlanSig sig;
    const int32_t *B;        // [N_c + 1] key chunk boundaries
    const int32_t *RB;       // [N_q + 1] query group boundaries (== B when the groups are the chunks)
    const int32_t *count;    // [H_q][N_q]
    const int32_t *entries;  // [H_q][N_q][stride][2]
    const int32_t *tiles;    // [T1][2]: tiles of > 96 rows, then 65..96, 33..64, <= 32 rows (T_cls of each)
    int stride, T1, T_big, N_q;
    int T_cls[4];
};

// Workspace layout in doubles.
struct WsLayout {
    int64_t off_Qc, off_Kc, off_Sc, doubles;
};

// Decode workspace (byte offsets).  Kc persists between steps; the rest is scratch of one step.
// The "plan" is a one-group plan: B [N_c_cap + 1], RB [2], count [H_q], entries [H_q][stride][2]
// (room for stride = N_c_cap), laid out by `pl` in words from off_plan.
struct DecodeLayout {
    int64_t off_Kc, off_Qc, off_Sc, off_plan, off_done, off_part, bytes;
    PlanLayout pl;
    int S_cap;   // most key slices (workgroups per head) of the attention step
};
// Selected keys per workgroup of the decode attention step.  While workgroups are few, a chain of loads takes the time and
// short slices run side by side, merged by the last workgroup of a head: 32 keys up to 128 workgroups, 64 up to 256.  More
// of them wait for one another's stores, and a head's merge gets long: one head, N_b = 8192 29.9 us with 32, 25.6 us with
// 64, 27.1 us with 128 keys; 6 heads, N_b = 4096 32.6, 27.1, 26.1 us; 8 heads, N_b = 512 20.9, 21.4, 23.4 us.  Else 128 and
// more (merged by a kernel), so many that there are at most five workgroups per CU.  That is what a CU holds of the bf16 kernel at D = 128; it would hold
// seven at D = 64 and eight in fp32, but shorter slices gain nothing there: 32 heads of D = 64, N_b = 8192 35.5 us with
// five, 36.6 us with seven; 16 fp32 heads of D = 64 32.8 us with five, 33.7 us with eight (128: 45.4, 45.5 us).
constexpr int kDecSlice = 128, kDecSliceMax = 512;
constexpr int kDecSliceFew = 32, kDecWgFew = 128;      // shortest slices, and the most workgroups they make
constexpr int kDecSliceSome = 64, kDecWgSome = 256;    // the same of middling ones
inline int decode_slice(int H_q, int64_t N_b) {
    if (H_q * ((N_b + kDecSliceFew - 1) / kDecSliceFew) <= kDecWgFew) return kDecSliceFew;
    if (H_q * ((N_b + kDecSliceSome - 1) / kDecSliceSome) <= kDecWgSome) return kDecSliceSome;
    const int64_t at_once = 5 * 256 / H_q > 0 ? 5 * 256 / H_q : 1, slice = ((N_b + at_once - 1) / at_once + 15) / 16 * 16;
    return (int)(slice < kDecSlice ? kDecSlice : slice > kDecSliceMax ? kDecSliceMax : slice);
}
// Boundaries B[kc_valid .. kc_valid + n] of the chunks a decoding step pools anew, passed by
// value when they are few (n = 0: the kernels read all boundaries from the workspace).
constexpr int kBoundaryTailMax = 6;
struct BoundaryTail {
    int n;
    int32_t b[kBoundaryTailMax + 1];
};

// Up to kBoundaryBlockMax boundaries passed by value to a kernel (a launch argument block
// holds at most 4 KiB), for callers whose boundary array must not go through a host copy.
constexpr int kBoundaryBlockMax = 960;

struct BoundaryBlock {
    int32_t first, n;
    int32_t b[kBoundaryBlockMax];
};

// Workgroups of at most 256 threads in one dimension of a launch: a dimension holds fewer than 2^32 threads, and a
// row-block problem can have 2^20 groups per head.
constexpr int kGridMax = 1 << 23;

// ---- launchers (each enqueues on `s` and returns the launch status) ----
// B_host[0 .. n) -> B_dev, carried by kernel arguments (no copy engine, no staging buffer)
hipError_t launch_put_boundaries(const int32_t *B_host, int n, int32_t *B_dev, hipStream_t s);
// boundaries and plan set-up, pooled vectors; ev (may be null): an event recorded before the pooling kernel
hipError_t launch_setup_pool(const Prob &p, const PlanLayout &pl, const void *Q, const void *K, const int32_t *B_host,
                             int32_t *plan, double *Qc, double *Kc, hipStream_t s, hipEvent_t *ev);
hipError_t launch_scores(const Prob &p, const double *Qc, const double *Kc, const int32_t *B_dev,
                         const int32_t *RB_dev, double *Sc, hipStream_t s);
hipError_t launch_select(const Prob &p, const PlanLayout &pl, const double *Sc, int32_t *plan, hipStream_t s);
// the two in one launch, for problems that score_select_ok takes
bool score_select_ok(const Prob &p);
hipError_t launch_score_select(const Prob &p, const PlanLayout &pl, const double *Qc, const double *Kc, double *Sc, int32_t *plan,
                               hipStream_t s);
// query groups [l_first, l_first + n_groups) only; `pl`, `Sc` and `plan` are indexed by group - l_first
hipError_t launch_select_groups(const Prob &p, const PlanLayout &pl, const double *Sc, int32_t *plan, int l_first,
                                int n_groups, hipStream_t s);
// one decoding step (decode.hip).  rb0 = first row of the open query group; boundaries that are not in `tail` are already in
// the step's plan
hipError_t launch_decode_step(const Prob &p, const DecodeLayout &dl, int N_c_cap, int kc_valid, int rb0, const BoundaryTail &tail,
                              const void *Q, const void *K, const void *V, void *ws, void *O_row, int32_t *idx, int32_t *cnt,
                              hipStream_t s);
hipError_t launch_expand(const Prob &p, const PlanView &pv, int head, const int64_t *rows_dev, int n_rows,
                         int32_t *idx, int cap, int32_t *cnt, hipStream_t s);
hipError_t launch_recall(const Prob &p, const PlanView &pv, const void *Q, const void *K, int head,
                         const int64_t *rows_host, int n_rows, unsigned long long *ws, int32_t *hits, int32_t *size,
                         hipStream_t s);
hipError_t launch_attn_f32(const Prob &p, const PlanView &pv, const void *Q, const void *K, const void *V,
                               void *O, hipStream_t s);
// ev (may be null): three events recorded after the launches of the tiles of more than 64 rows, of
// 33..64 rows and of at most 32 rows
hipError_t launch_attn_mfma(const Prob &p, const PlanView &pv, const void *Q, const void *K, const void *V,
                            void *O, hipStream_t s, hipEvent_t *ev = nullptr);
// scores, ranking and attention in one launch, behind launch_setup_pool, for problems that route_attend_ok takes (T_cls row tiles a head)
bool route_attend_ok(const Prob &p, const int32_t *T_cls);
hipError_t launch_route_attend(const Prob &p, const PlanLayout &pl, const PlanView &pv, const double *Qc, const double *Kc, double *Sc,
                               int32_t *plan, const void *Q, const void *K, const void *V, void *O, hipStream_t s);
bool f32_route_attend_ok(const Prob &p, const int32_t *T_cls);   // of fp32 problems (attn.hip)
hipError_t launch_f32_route_attend(const Prob &p, const PlanLayout &pl, const PlanView &pv, const double *Qc, const double *Kc,
                                   double *Sc, int32_t *plan, const void *Q, const void *K, const void *V, void *O, hipStream_t s);
// the kernels and events of launch_attn_mfma by height class (dhsa_attention_kernels)
void attn_mfma_kernels(const Prob &p, const int32_t *T_cls, int32_t *kernel, int32_t *slot);

// ---- small device helpers ----
// bf16 storage type (a bare 16-bit pattern; the kernels convert by hand)
struct bf16_t { uint16_t bits; };

// 16 bytes of a row as fp64 addends (the pooling kernels accumulate in fp64)
template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int kPer16 = 4;
    __device__ static void unpack(const uint4 &u, double *acc) {
        acc[0] += (double)__uint_as_float(u.x);
        acc[1] += (double)__uint_as_float(u.y);
        acc[2] += (double)__uint_as_float(u.z);
        acc[3] += (double)__uint_as_float(u.w);
    }
};
template <> struct Elem<bf16_t> {
    static constexpr int kPer16 = 8;
    __device__ static void unpack(const uint4 &u, double *acc) {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] += (double)__uint_as_float(w[i] << 16);
            acc[2 * i + 1] += (double)__uint_as_float(w[i] & 0xffff0000u);
        }
    }
};

__device__ __forceinline__ int chunk_of_row(const int32_t *__restrict__ B, int N_c, int64_t i) {
    int lo = 0, hi = N_c;  // B[lo] <= i < B[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if ((int64_t)B[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

// One batch of scalar loads: with a branch per word (&&) the second line of the header was requested only when the first
// one was there, most of a microsecond of each workgroup's prologue.
__device__ __forceinline__ bool plan_matches(const PlanView &pv) {
    const int32_t *w = pv.hdr;
    return (w[0] == DHSA_PLAN_MAGIC) & (w[1] == DHSA_PLAN_VERSION) & (w[2] == pv.sig.H_q) & (w[3] == pv.sig.N_c) &
           (w[4] == pv.sig.N_b) & (w[5] == pv.sig.stride) & (w[6] == pv.sig.L) & (w[7] == pv.sig.T1) &
           (w[14] == pv.sig.N_q) & (w[15] == pv.sig.B_r) & (w[16] == pv.sig.pooling) & (w[17] == pv.sig.b_sum);
}

// Class of a row tile by its number of rows (1..128): the attention kernels give each class its
// own arrangement of waves.  0: more than 96 rows, 1: 65..96, 2: 33..64, 3: at most 32.
__host__ __device__ __forceinline__ int tile_class(int rows) {
    return rows > 96 ? 0 : rows > 64 ? 1 : rows > 32 ? 2 : 3;
}

// Tokens row (visible own-chunk count v) takes from a plan entry.  For pos = 3
// (row-block form) rem is the number of listed tokens, never above len_k; the
// causal mask is applied per token by the caller.
__device__ __forceinline__ int entry_take(int pos, int rem, int len_k, int v) {
    int lim = (pos == 1) ? v : len_k;
    int room = (pos == 2) ? rem - v : rem;
    int t = room < lim ? room : lim;
    return t > 0 ? t : 0;
}

// Lane-crossing sums of a wave on the vector unit (DPP: shifts inside rows of 16 lanes, then the last lane of a row or
// half to the ones above it); lane 63 ends up with all 64 lanes.  A step is one instruction; through the LDS (__shfl_up)
// it is a round trip of about a hundred cycles.  With this in the prologues of the attention kernels and the header read at
// once: fp32 prefill of 1059 tokens, 8 heads 35.0 -> 34.0 us, attention of 3007 tokens, 187 keys 31.2 -> 30.1 us.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
#define DHSA_DPP_STEPS(STEP) STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)
__device__ __forceinline__ int wave_incl_scan(int x) {
#define DHSA_STEP(CTRL, ROWS) x += dpp_or<CTRL, ROWS>(0, x);
    DHSA_DPP_STEPS(DHSA_STEP)
#undef DHSA_STEP
    return x;
}

// Exclusive prefix sum of one int per thread over a 256-thread block (wave
// scans + one LDS slot per wave).  `total` receives the block sum.  Contains
// two block barriers; s_wave is an int[4] in LDS.
__device__ __forceinline__ int block_excl_scan(int val, int *s_wave, int *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = wave_incl_scan(val);
    __syncthreads();  // protects s_wave from its previous use
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        int x = s_wave[w];
        if (w < wave) base += x;
        tot += x;
    }
    *total = tot;
    return base + inc - val;
}

// Two exclusive prefix sums at once (same barriers as one).
__device__ __forceinline__ void block_excl_scan2(int a, int b, int *s_wave8, int *excl_a, int *excl_b, int *total_a,
                                                 int *total_b) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ia = wave_incl_scan(a), ib = wave_incl_scan(b);
    __syncthreads();  // protects s_wave8 from its previous use
    if (lane == 63) { s_wave8[wave] = ia; s_wave8[4 + wave] = ib; }
    __syncthreads();
    int base_a = 0, base_b = 0, tot_a = 0, tot_b = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int xa = s_wave8[w], xb = s_wave8[4 + w];
        if (w < wave) { base_a += xa; base_b += xb; }
        tot_a += xa; tot_b += xb;
    }
    *total_a = tot_a; *total_b = tot_b;
    *excl_a = base_a + ia - a;
    *excl_b = base_b + ib - b;
}

}  // namespace dhsa
