// Routing kernels of libdhsa: plan set-up, chunk pooling (Sec. 3.3 Eq. 4),
// chunk similarity S_c = Q_c K_c^T (Sec. 3.3), ranking and per-row budget
// (Sec. 3.1 Step 2, Alg. 1), and the plan -> index-set expansion hook.
//
// All routing arithmetic is fp64: pooled sums of bf16 inputs are then exact
// (order-free), and S_c carries ~1e-14 absolute error, so the ranking does not
// hinge on summation order.
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "dhsa_internal.h"

namespace dhsa {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Boundaries into the plan without a copy from host memory: each launch carries
// up to kBoundaryBlockMax of them as kernel arguments.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_put_boundaries(int32_t *__restrict__ dst, BoundaryBlock blk) {
    for (int i = threadIdx.x; i < blk.n; i += 256) dst[blk.first + i] = blk.b[i];
}

static void fill_block(BoundaryBlock &blk, const int32_t *B_host, int first, int n) {
    blk.first = first;
    blk.n = std::min(kBoundaryBlockMax, n - first);
    memcpy(blk.b, B_host + first, sizeof(int32_t) * (size_t)blk.n);
    memset(blk.b + blk.n, 0, sizeof(int32_t) * (size_t)(kBoundaryBlockMax - blk.n));
}

hipError_t launch_put_boundaries(const int32_t *B_host, int n, int32_t *B_dev, hipStream_t s) {
    BoundaryBlock blk;
    for (int first = 0; first < n; first += kBoundaryBlockMax) {
        fill_block(blk, B_host, first, n);
        hipLaunchKernelGGL(k_put_boundaries, dim3(1), dim3(256), 0, s, B_dev, blk);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// What the set-up block writes beside the boundaries.
struct SetupArgs {
    int32_t *plan;
    PlanLayout pl;
    int H_q, H_kv, D, N_c, N_b, B_r, pooling;
    int64_t L;
};

// ---------------------------------------------------------------------------
// Plan header, query-group boundaries and row-tile table, by one block.  The query
// groups are the chunks themselves, or (Alg. 1 as printed) row blocks of B_r rows,
// RB[i] = min(i B_r, L).  Tiles are the <= 128-row pieces of the query groups; the
// table lists them by class -- more than 96 rows, 65..96, 33..64, at most 32 --
// each class ordered by row.  B: the key chunk boundaries, wherever they are.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void setup_block(const SetupArgs &a, const int32_t *B) {
    __shared__ int s_wave8[8];
    const int tid = threadIdx.x;
    const PlanLayout &pl = a.pl;
    const int N_q = pl.N_q;
    int32_t *tiles = a.plan + pl.off_tiles;
    int32_t *RBw = a.plan + pl.off_RB;
    if (tid < kPlanHeaderWords) {
        int32_t w = 0;
        switch (tid) {
            case 0: w = DHSA_PLAN_MAGIC; break;
            case 1: w = DHSA_PLAN_VERSION; break;
            case 2: w = a.H_q; break;
            case 3: w = a.N_c; break;
            case 4: w = a.N_b; break;
            case 5: w = pl.stride; break;
            case 6: w = (int32_t)a.L; break;
            case 7: w = pl.T1; break;
            case 8: w = (int32_t)pl.off_B; break;
            case 9: w = (int32_t)pl.off_count; break;
            case 10: w = (int32_t)pl.off_entries; break;
            case 11: w = (int32_t)pl.off_tiles; break;
            case 12: w = pl.T_big; break;
            case 13: w = (int32_t)pl.off_RB; break;
            case 14: w = N_q; break;
            case 15: w = a.B_r; break;
            case 16: w = a.pooling; break;
            case 17: w = pl.b_sum; break;
            case 18: w = a.H_kv; break;
            case 19: w = a.D; break;
            case 20: case 21: case 22: case 23: w = pl.T_cls[tid - 20]; break;
            default: break;
        }
        a.plan[tid] = w;
    }
    // where each class continues in the table (the same in every thread)
    int at[4] = {0, pl.T_cls[0], pl.T_cls[0] + pl.T_cls[1], pl.T_cls[0] + pl.T_cls[1] + pl.T_cls[2]};
    for (int base = 0; base < N_q; base += 256) {
        const int l = base + tid;
        int b0 = 0, nfull = 0, rem = 0;
        if (l < N_q) {
            int b1;
            if (a.B_r > 0) {
                const int64_t x0 = (int64_t)l * a.B_r, x1 = x0 + a.B_r;
                b0 = (int32_t)x0;
                b1 = (int32_t)(x1 < a.L ? x1 : a.L);
                if (l == 0) RBw[0] = 0;
                RBw[l + 1] = b1;
            } else {
                b0 = B[l];
                b1 = B[l + 1];
            }
            nfull = (b1 - b0) / kRowTile;
            rem = (b1 - b0) % kRowTile;
        }
        const int rem_cls = rem > 0 ? tile_class(rem) : -1;
        int mine[4], before[4], total[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) mine[c] = (c == 0 ? nfull : 0) + (rem_cls == c);
        block_excl_scan2(mine[0], mine[1], s_wave8, &before[0], &before[1], &total[0], &total[1]);
        block_excl_scan2(mine[2], mine[3], s_wave8, &before[2], &before[3], &total[2], &total[3]);
        for (int t = 0; t < nfull; ++t) {
            tiles[2 * (at[0] + before[0] + t)] = l;
            tiles[2 * (at[0] + before[0] + t) + 1] = b0 + t * kRowTile;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (rem_cls == c) {   // the remainder follows the group's full tiles
                const int x = at[c] + before[c] + mine[c] - 1;
                tiles[2 * x] = l;
                tiles[2 * x + 1] = b0 + nfull * kRowTile;
            }
            at[c] += total[c];
        }
    }
}

// ---------------------------------------------------------------------------
// Chunk pooling, Eq. 4: X_c[h, k, :] = (sqrt(len)/len) * sum_{i in chunk k} X[h, i, :],
// and the plan's set-up beside it.
// One block per (chunk, head); a row of D elements is read by D*sizeof(T)/16
// threads with 16-byte loads, row groups are summed through LDS.  HBM-bound.
// Keys are pooled over the chunks B; queries over the query groups RB (the
// chunks again, or with B_r > 0 the row blocks of Alg. 1, whose representation
// is sqrt(B_r) * mean of the block's rows).
// grid (1 + max(N_q, N_c), H_q + H_kv): x = 0 holds the set-up block (y = 0), started first.
// BLK: the boundaries, all of them, come as kernel arguments and the set-up block writes them
// into the plan, so a short prompt needs one launch where boundaries, set-up and pooling took three (7.2 us of a
// 1K-token prefill, now 4 us); otherwise they are in the plan already.
// ---------------------------------------------------------------------------
struct NoBlock {};

template <typename T, int D, typename BLK>
__global__ __launch_bounds__(256) void k_pool(const T *__restrict__ Q, const T *__restrict__ K, SetupArgs a,
                                              double *__restrict__ Qc, double *__restrict__ Kc, int64_t qs_h,
                                              int64_t qs_l, int64_t ks_h, int64_t ks_l, BLK blk) {
    constexpr int EPT = Elem<T>::kPer16;   // elements per thread per row
    constexpr int TPR = D / EPT;           // threads per row
    constexpr int RG = 256 / TPR;          // rows in flight
    constexpr bool kInline = !std::is_same<BLK, NoBlock>::value;
    __shared__ double s_sum[RG][D];
    const int tid = threadIdx.x;
    const int32_t *B;
    if constexpr (kInline) B = blk.b; else B = a.plan + a.pl.off_B;
    if (blockIdx.x == 0) {
        if (blockIdx.y != 0) return;
        if constexpr (kInline)
            for (int i = tid; i < blk.n; i += 256) a.plan[a.pl.off_B + i] = blk.b[i];
        setup_block(a, B);
        return;
    }
    const int k = blockIdx.x - 1, N_q = a.pl.N_q;
    int h = blockIdx.y;
    const T *X;
    double *Xc;
    int64_t s_l;
    const bool is_q = h < a.H_q;
    if (k >= (is_q ? N_q : a.N_c)) return;   // block-uniform: the grid spans max(N_q, N_c)
    if (is_q) {
        X = Q + (int64_t)h * qs_h; s_l = qs_l; Xc = Qc + ((int64_t)h * N_q + k) * D;
    } else {
        h -= a.H_q;
        X = K + (int64_t)h * ks_h; s_l = ks_l; Xc = Kc + ((int64_t)h * a.N_c + k) * D;
    }
    int b0, b1;
    if (is_q && a.B_r > 0) {
        const int64_t x0 = (int64_t)k * a.B_r, x1 = x0 + a.B_r;
        b0 = (int)x0;
        b1 = (int)(x1 < a.L ? x1 : a.L);
    } else {
        b0 = B[k];
        b1 = B[k + 1];
    }
    const int rg = tid / TPR, col = (tid % TPR) * EPT;
    double acc[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) acc[e] = 0.0;
    for (int i = b0 + rg; i < b1; i += RG) {
        uint4 u = *reinterpret_cast<const uint4 *>(X + (int64_t)i * s_l + col);
        Elem<T>::unpack(u, acc);
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) s_sum[rg][col + e] = acc[e];
    __syncthreads();
    if (tid < D) {
        double sum = 0.0;
#pragma unroll 4
        for (int r = 0; r < RG; ++r) sum += s_sum[r][tid];
        const double len = (double)(b1 - b0);
        Xc[tid] = a.pooling == DHSA_POOL_MEAN ? sum / len                                // plain average (ablation)
                  : (is_q && a.B_r > 0)    ? sqrt((double)a.B_r) * (sum / len)          // Alg. 1 row blocks
                                           : (sqrt(len) / len) * sum;                   // Eq. 4
    }
}

hipError_t launch_setup_pool(const Prob &p, const PlanLayout &pl, const void *Q, const void *K, const int32_t *B_host,
                             int32_t *plan, double *Qc, double *Kc, hipStream_t s, hipEvent_t *ev) {
    const bool inl = p.N_c + 1 <= kBoundaryBlockMax;
    if (!inl) {
        hipError_t e = launch_put_boundaries(B_host, p.N_c + 1, plan + pl.off_B, s);
        if (e != hipSuccess) return e;
    }
    if (ev && hipEventRecord(ev[0], s) != hipSuccess) return hipErrorUnknown;
    const SetupArgs a = {plan, pl, p.H_q, p.H_kv, p.D, p.N_c, p.N_b, p.B_r, p.pooling, p.L};
    const dim3 grid(1 + (p.N_q > p.N_c ? p.N_q : p.N_c), p.H_q + p.H_kv), block(256);
#define DHSA_POOL(T, DD)                                                                                             \
    do {                                                                                                             \
        if (inl) {                                                                                                   \
            BoundaryBlock blk;                                                                                       \
            fill_block(blk, B_host, 0, p.N_c + 1);                                                                   \
            hipLaunchKernelGGL((k_pool<T, DD, BoundaryBlock>), grid, block, 0, s, (const T *)Q, (const T *)K, a, Qc, \
                               Kc, p.qs_h, p.qs_l, p.ks_h, p.ks_l, blk);                                             \
        } else                                                                                                       \
            hipLaunchKernelGGL((k_pool<T, DD, NoBlock>), grid, block, 0, s, (const T *)Q, (const T *)K, a, Qc, Kc,   \
                               p.qs_h, p.qs_l, p.ks_h, p.ks_l, NoBlock{});                                           \
    } while (0)
    if (p.dtype == DHSA_F32) {
        if (p.D == 64) DHSA_POOL(float, 64); else DHSA_POOL(float, 128);
    } else {
        if (p.D == 64) DHSA_POOL(bf16_t, 64); else DHSA_POOL(bf16_t, 128);
    }
#undef DHSA_POOL
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Chunk similarity S_c[h, l, k] = <Q_c[h, l], K_c[h / G, k]> for the key chunks
// k that some row of query group l can see (B[k] < RB[l+1]; with the chunks as
// query groups that is k <= l), fp64 MFMA (16x16x4).  Four waves in a 2 x 2
// arrangement; tiles none of whose pairs is visible are skipped.
//
// Lane 16 q + n of a wave holds d = 8 s + 2 q + {0, 1} of row n of each operand block (16 bytes) and
// supplies one of the two to each of two products, which contract over the d the four q hold.
//
// k_scores (64 x 64 tiles, a wave 2 x 2 blocks): operands staged through registers into LDS in
// slabs of 32 d, the next slab requested before the current one is multiplied; the 16-byte pieces of a row are
// XOR-swizzled by its number, so that the 16 rows x 4 pieces of a read spread over all banks.
// 1634 chunks x 32 heads of D = 128: 242 us (150 us of products at the fp64 rate of the matrix unit); the form with
// 8-byte reads and padded rows took 332 us, bound by bank conflicts, one that reads its operands from memory in
// this layout, 383 us.
// k_scores_few (32 x 32 tiles, a wave one block, operands straight from memory, all of D
// requested at once): fewer than 512 tiles, where the chain of one wave is what takes the time (one
// tile of 64 x 64: 10 us in the other form, 5 us).
//
// Workgroups are dealt to the 8 XCDs round-robin: an XCD gets whole heads, one after the other, so that
// its L2 holds the pooled vectors of one or two heads at a time.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void score_tile(int b, int H_q, int per, int *h, int *t) {
    if ((H_q & 7) == 0) { *t = (b >> 3) % per; *h = (b & 7) * (H_q >> 3) + (b >> 3) / per; }
    else { *t = b % per; *h = b / per; }
}

constexpr int kScTile = 64;
constexpr int kScSlab = 32;   // d staged in LDS at a time: 16 pieces of 16 bytes per row

template <int D>
__global__ __launch_bounds__(256, 4) void k_scores(const double *__restrict__ Qc, const double *__restrict__ Kc,
                                                   const int32_t *__restrict__ B, const int32_t *__restrict__ RB,
                                                   double *__restrict__ Sc, int N_c, int N_q, int H_q, int G, int ntk,
                                                   int ntl, int blocks) {
    __shared__ f64x2 sA[kScTile][kScSlab / 2], sB[kScTile][kScSlab / 2];
    int h, t;
    score_tile(blockIdx.x, H_q, ntk * ntl, &h, &t);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = (t % ntk) * kScTile, l0 = (t / ntk) * kScTile;
    const int l_last = (l0 + kScTile < N_q ? l0 + kScTile : N_q) - 1;   // last query group of the tile
    if (blocks ? B[k0] >= RB[l_last + 1] : k0 > l_last) return;         // its first chunk starts past every row
    const int n16 = lane & 15, q = lane >> 4;
    const int wl = (wave >> 1) * 32, wk = (wave & 1) * 32;

    // staging: thread -> row tid / 16 (+ 16 i), piece tid % 16; rows past the end repeat the last one (not stored)
    const int sr = tid >> 4, sp = tid & 15;
    const double *A[4], *Bm[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int l = l0 + sr + 16 * i, k = k0 + sr + 16 * i;
        A[i] = Qc + ((int64_t)h * N_q + (l < N_q ? l : N_q - 1)) * D + 2 * sp;
        Bm[i] = Kc + ((int64_t)(h / G) * N_c + (k < N_c ? k : N_c - 1)) * D + 2 * sp;
    }
    f64x4 acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = (f64x4){0.0, 0.0, 0.0, 0.0};
    f64x2 ra[4], rb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        ra[i] = *reinterpret_cast<const f64x2 *>(A[i]);
        rb[i] = *reinterpret_cast<const f64x2 *>(Bm[i]);
    }
#pragma unroll
    for (int d0 = 0; d0 < D; d0 += kScSlab) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sA[sr + 16 * i][sp ^ sr] = ra[i];   // row & 15 == sr
            sB[sr + 16 * i][sp ^ sr] = rb[i];
        }
        __syncthreads();
        if (d0 + kScSlab < D) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ra[i] = *reinterpret_cast<const f64x2 *>(A[i] + d0 + kScSlab);
                rb[i] = *reinterpret_cast<const f64x2 *>(Bm[i] + d0 + kScSlab);
            }
            __builtin_amdgcn_sched_barrier(0);   // left alone, the scheduler moves the loads next to their use
        }
#pragma unroll
        for (int s = 0; s < kScSlab / 8; ++s) {
            f64x2 a[2], b[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                a[m] = sA[wl + 16 * m + n16][(4 * s + q) ^ n16];
                b[m] = sB[wk + 16 * m + n16][(4 * s + q) ^ n16];
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int n = 0; n < 2; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m][j], b[n][j], acc[m][n], 0, 0, 0);
        }
        __syncthreads();
    }
    // D[i][j]: accumulator element v of a lane is row 4*v + lane/16, column lane % 16
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int l = l0 + wl + 16 * m + 4 * v + q, k = k0 + wk + 16 * n + n16;
                if (l < N_q && k < N_c) Sc[((int64_t)h * N_q + l) * N_c + k] = acc[m][n][v];
            }
}

template <int D>
__global__ __launch_bounds__(256) void k_scores_few(const double *__restrict__ Qc, const double *__restrict__ Kc,
                                                    const int32_t *__restrict__ B, const int32_t *__restrict__ RB,
                                                    double *__restrict__ Sc, int N_c, int N_q, int H_q, int G, int ntk,
                                                    int ntl, int blocks) {
    int h, t;
    score_tile(blockIdx.x, H_q, ntk * ntl, &h, &t);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = (t % ntk) * 32 + (wave & 1) * 16, l0 = (t / ntk) * 32 + (wave >> 1) * 16;
    if (k0 >= N_c || l0 >= N_q) return;
    const int l_last = (l0 + 16 < N_q ? l0 + 16 : N_q) - 1;        // last query group of the wave
    if (blocks ? B[k0] >= RB[l_last + 1] : k0 > l_last) return;
    const int n16 = lane & 15, q = lane >> 4;
    const double *A = Qc + ((int64_t)h * N_q + (l0 + n16 < N_q ? l0 + n16 : N_q - 1)) * D + 2 * q;
    const double *Bm = Kc + ((int64_t)(h / G) * N_c + (k0 + n16 < N_c ? k0 + n16 : N_c - 1)) * D + 2 * q;
    f64x2 a[D / 8], b[D / 8];
#pragma unroll
    for (int s = 0; s < D / 8; ++s) {
        a[s] = *reinterpret_cast<const f64x2 *>(A + 8 * s);
        b[s] = *reinterpret_cast<const f64x2 *>(Bm + 8 * s);
    }
    __builtin_amdgcn_sched_barrier(0);
    f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < D / 8; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][j], b[s][j], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int l = l0 + 4 * v + q, k = k0 + n16;
        if (l < N_q && k < N_c) Sc[((int64_t)h * N_q + l) * N_c + k] = acc[v];
    }
}

hipError_t launch_scores(const Prob &p, const double *Qc, const double *Kc, const int32_t *B_dev,
                         const int32_t *RB_dev, double *Sc, hipStream_t s) {
    const bool few = ((int64_t)(p.N_c + 63) / 64) * ((p.N_q + 63) / 64) * p.H_q < 512;
    const int T = few ? 32 : kScTile;
    const int ntk = (p.N_c + T - 1) / T, ntl = (p.N_q + T - 1) / T;
    const dim3 grid((unsigned)((int64_t)ntk * ntl * p.H_q)), block(256);
#define DHSA_SCORES(KERNEL)                                                                                      \
    hipLaunchKernelGGL(KERNEL, grid, block, 0, s, Qc, Kc, B_dev, RB_dev, Sc, p.N_c, p.N_q, p.H_q, p.G, ntk, ntl, \
                       p.B_r > 0 ? 1 : 0)
    if (p.D == 64) {
        if (few) DHSA_SCORES(k_scores_few<64>); else DHSA_SCORES(k_scores<64>);
    } else {
        if (few) DHSA_SCORES(k_scores_few<128>); else DHSA_SCORES(k_scores<128>);
    }
#undef DHSA_SCORES
    return hipGetLastError();
}

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

static int select_cap(int stride) { return (stride + 2 + 32 + 63) / 64 * 64; }   // some to spare before a bin is cut again
static int select_row_bytes(int NW, int cap, int N_c) {   // cap: a multiple of 64
    return kSelBins * (NW == 1 ? 8 : 16) + cap * 20 + (N_c + 63) / 64 * 8;
}

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

// Ranks the scores row[0 .. vis.n) of group l of head h; mine8: row_bytes of LDS, s_red: NW words of it.  row and B in
// memory or LDS.
template <int NW>
__device__ __forceinline__ void select_row(const SelectArgs &a, const double *row, const int32_t *B, const Visible vis,
                                           const int h, const int l, unsigned char *mine8, unsigned long long *s_red) {
    constexpr int NT = 64 * NW, PER = kSelPer, kSlab = PER * NT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = NW == 1 ? lane : (int)threadIdx.x;                     // thread of the row
    const int N_c = a.N_c, N_b = a.N_b, cap = a.cap;
    int32_t *const plan = a.plan;
    const PlanLayout &pl = a.pl;
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
    int32_t *entries = plan + pl.off_entries + ((int64_t)h * pl.N_q + l) * pl.stride * 2;
    for (int cb = 0; cb < n_c; cb += NT) {              // whole waves: the shuffles need their lanes
        const int c = cb + t < n_c ? cb + t : n_c - 1;
        const int rem = cb + t < n_c ? crem[c] : 0, w = cid[c], x = w & kChunkMask, word = x >> 6;
        const int even = __shfl(listed - c0 - c1, word >> 1), odd = __shfl(listed - c1, word >> 1);   // all lanes read
        const int below = (word & 1) ? odd : even;
        const int slot = below + __popcll(kept[word] & ((1ull << (x & 63)) - 1ull));
        if (rem > 0 && slot < pl.stride) *reinterpret_cast<int2 *>(entries + 2 * slot) = make_int2(w, rem);
    }
    if (t == 0) plan[pl.off_count + (int64_t)h * pl.N_q + l] = total < pl.stride ? total : pl.stride;
}

template <int NW>
__global__ __launch_bounds__(256, 7) void k_select(const double *__restrict__ Sc, SelectArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned long long s_red[NW];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = a.r_first + (int)(NW == 1 ? blockIdx.x * (blockDim.x >> 6) + wave : blockIdx.x);
    if (r >= a.n_rows) return;           // NW == 1: waves do not wait for each other
    const int h = r / a.n_groups, l = r % a.n_groups;
    const int32_t *B = a.plan + a.pl.off_B;
    select_row<NW>(a, Sc + ((int64_t)h * a.pl.N_q + l) * a.N_c, B, visible_chunks(a, B, l), h, l,
                   smem + (size_t)(NW == 1 ? wave : 0) * a.row_bytes, s_red);
}

// ---------------------------------------------------------------------------
// Scores of one query group against the chunks 0 .. n-1 by the NW waves of a workgroup: a wave takes 16 chunks at a time, as
// columns, and repeats the group's vector as all 16 rows, so that a score is made of the same products in the same
// order as in k_scores.  key(k): the pooled vector of chunk k.
// ---------------------------------------------------------------------------
template <int D, int NW, typename KEY>
__device__ __forceinline__ void score_row(const double *q_c, const KEY &key, int n, double *s_row) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n16 = lane & 15, q = lane >> 4;
    f64x2 a[D / 8], b[2][D / 8];
    const auto load = [&](int k0, f64x2 (&to)[D / 8]) {
        const double *Bm = key(k0 + n16 < n ? k0 + n16 : n - 1) + 2 * q;
#pragma unroll
        for (int s = 0; s < D / 8; ++s) to[s] = *reinterpret_cast<const f64x2 *>(Bm + 8 * s);
    };
    const auto block = [&](int k0, const f64x2 (&b_)[D / 8]) {
        f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < D / 8; ++s)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][j], b_[s][j], acc, 0, 0, 0);
        if (q == 0 && k0 + n16 < n) s_row[k0 + n16] = acc[0];
    };
    int k0 = wave * 16;
    if (k0 >= n) return;
    load(k0, b[0]);
#pragma unroll
    for (int s = 0; s < D / 8; ++s) a[s] = *reinterpret_cast<const f64x2 *>(q_c + 2 * q + 8 * s);
    __builtin_amdgcn_sched_barrier(0);
    for (;; k0 += 32 * NW) {             // the next 16 chunks are requested before these are multiplied
        if (k0 + 16 * NW < n) load(k0 + 16 * NW, b[1]);
        __builtin_amdgcn_sched_barrier(0);
        block(k0, b[0]);
        if (k0 + 16 * NW >= n) break;
        if (k0 + 32 * NW < n) load(k0 + 32 * NW, b[0]);
        __builtin_amdgcn_sched_barrier(0);
        block(k0 + 16 * NW, b[1]);
        if (k0 + 32 * NW >= n) break;
    }
}

// Scores and ranking of one (head, query group) by a workgroup of four waves, for problems of few groups and few chunks,
// where a launch takes longer than the scores of a group.  Bound by a chain: one memory latency, 32 products in a row, the ranking.
template <int D>
__global__ __launch_bounds__(256, 2) void k_score_select(const double *__restrict__ Qc, const double *__restrict__ Kc,
                                                         double *__restrict__ Sc, int G, SelectArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned long long s_red[4];
    const int h = blockIdx.x / a.n_groups, l = blockIdx.x % a.n_groups;
    const int32_t *B = a.plan + a.pl.off_B;
    const Visible vis = visible_chunks(a, B, l);
    double *s_row = reinterpret_cast<double *>(smem + a.row_bytes);
    const double *K = Kc + (int64_t)(h / G) * a.N_c * D;
    score_row<D, 4>(Qc + ((int64_t)h * a.pl.N_q + l) * D, [&](int k) { return K + (int64_t)k * D; }, vis.n, s_row);
    __syncthreads();
    double *row = Sc + ((int64_t)h * a.pl.N_q + l) * a.N_c;
    for (int x = threadIdx.x; x < vis.n; x += 256) row[x] = s_row[x];
    select_row<4>(a, s_row, B, vis, h, l, smem, s_red);
}

// ---------------------------------------------------------------------------
// Routing of one decoding step, all of it, by one workgroup of eight waves per query head: the open group's queries and the
// new key chunks are pooled (the first four waves and the others side by side, in k_pool_decode's order), then scored and
// ranked.  The heads of a kv-group pool the same key chunks; the first of them stores them for later steps.  Boundaries and
// pooled keys that come with the step are taken from LDS, the others from the workspace.
// ---------------------------------------------------------------------------
constexpr int kRouteDecodeNew = 3;   // key chunks to pool: with the group's queries two rounds of the workgroup's halves

template <typename T, int D>
__global__ __launch_bounds__(512, 2) void k_route_decode(const T *__restrict__ Q, const T *__restrict__ K, BoundaryTail tail,
                                                         int32_t *__restrict__ done, double *__restrict__ Kc, SelectArgs a,
                                                         int H_kv, int G, int N_c_cap, int kc_valid, int rb0, int L,
                                                         int pooling, int64_t qs_h, int64_t qs_l, int64_t ks_h, int64_t ks_l) {
    constexpr int EPT = Elem<T>::kPer16, TPR = D / EPT, RG = 256 / TPR;   // as in k_pool_decode
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_sum[2][RG][D];
    __shared__ double s_pool[1 + kRouteDecodeNew][D];       // the queries, then the new chunks
    __shared__ unsigned long long s_red[8];
    const int h = blockIdx.x, g = h / G, tid = threadIdx.x, half = __builtin_amdgcn_readfirstlane(tid >> 8), th = tid & 255;
    double *s_row = reinterpret_cast<double *>(smem + a.row_bytes);
    int32_t *s_B = reinterpret_cast<int32_t *>(s_row + a.N_c);
    int32_t *B = a.plan + a.pl.off_B, *RBw = a.plan + a.pl.off_RB;
    for (int k = tid; k < kc_valid; k += 512) s_B[k] = B[k];
    if (tid <= tail.n) s_B[kc_valid + tid] = tail.b[tid];
    if (tid == 0) done[h] = 0;                              // slices of the head finished so far (k_attn_decode)
    if (h == 0) {                                           // for the kernels after this one
        if (tid <= tail.n) B[kc_valid + tid] = tail.b[tid];
        if (tid == 0) { RBw[0] = rb0; RBw[1] = L; }
    }
    const int rg = th / TPR, col = (th % TPR) * EPT;
    for (int x0 = 0; x0 <= tail.n; x0 += 2) {
        const int x = x0 + half;
        const bool is_q = x == 0;
        const T *X = is_q ? Q + (int64_t)h * qs_h : K + (int64_t)g * ks_h;
        const int64_t s_l = is_q ? qs_l : ks_l;
        int b0 = rb0, b1 = L;
        if (!is_q) { b0 = x <= tail.n ? tail.b[x - 1] : 0; b1 = x <= tail.n ? tail.b[x] : 0; }
        double acc[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) acc[e] = 0.0;
        for (int i = b0 + rg; i < b1; i += RG) {
            const uint4 u = *reinterpret_cast<const uint4 *>(X + (int64_t)i * s_l + col);
            Elem<T>::unpack(u, acc);
        }
        if (x0 > 0) __syncthreads();
#pragma unroll
        for (int e = 0; e < EPT; ++e) s_sum[half][rg][col + e] = acc[e];
        __syncthreads();
        if (th < D && x <= tail.n) {
            double sum = 0.0;
#pragma unroll 4
            for (int r = 0; r < RG; ++r) sum += s_sum[half][r][th];
            const double len = (double)(b1 - b0);
            const double pooled = pooling == DHSA_POOL_MEAN ? sum / len                        // plain average (ablation)
                                  : (is_q && a.B_r > 0)    ? sqrt((double)a.B_r) * (sum / len)  // Alg. 1 row blocks
                                                           : (sqrt(len) / len) * sum;           // Eq. 4
            s_pool[x][th] = pooled;
            if (!is_q && h == g * G) Kc[((int64_t)g * N_c_cap + kc_valid + x - 1) * D + th] = pooled;
        }
    }
    __syncthreads();
    const double *Kg = Kc + (int64_t)g * N_c_cap * D;
    score_row<D, 8>(s_pool[0], [&](int k) { return k < kc_valid ? Kg + (int64_t)k * D : s_pool[1 + k - kc_valid]; }, a.N_c, s_row);
    __syncthreads();
    const Visible vis = {a.B_r > 0 ? -1 : a.N_c - 1, L, a.N_c};   // the last group sees all chunks
    select_row<8>(a, s_row, s_B, vis, h, 0, smem, s_red);
}

// ---------------------------------------------------------------------------
// The same for groups that can list more than kSelMaxStride chunks (many chunks of a few tokens): one
// workgroup per (head, query group) sorts the whole row in LDS.
//   1. scores of the visible chunks -> LDS as order-preserving 64-bit integers;
//   2. bitonic sort, larger score first, equal scores lower id first;
//   3. exclusive prefix sum of chunk lengths along the ranking, chunk l left out
//      -> rem = N_b - (tokens of other chunks before this rank);
//   4. a chunk is kept if some row takes a token of it; kept chunks are
//      compacted in ascending chunk id (prefix sum of flags) into the plan.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_select_sorted(const double *__restrict__ Sc, int32_t *__restrict__ plan,
                                                       PlanLayout pl, int N_c, int N_b, int B_r, int l_first) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_wave[4];
    __shared__ int s_p;
    const int l = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const int32_t *B = plan + pl.off_B;
    const bool blocks = B_r > 0;
    const int q_max = blocks ? (plan + pl.off_RB)[l + 1] : 0x7fffffff;   // clip of the chunk lengths
    const int own = blocks ? -1 : l_first + l;                            // the query group's own chunk
    const int n = blocks ? chunk_of_row(B, N_c, (int64_t)q_max - 1) + 1 : l_first + l + 1;   // visible chunks 0..n-1
    int P = 64;
    while (P < n) P <<= 1;
    unsigned long long *key = reinterpret_cast<unsigned long long *>(smem);  // [P]
    int *id = reinterpret_cast<int *>(smem + (size_t)P * 8);                 // [P]
    const double *row = Sc + ((int64_t)h * pl.N_q + l) * N_c;

    // eight scores per thread are requested before the first is used (one memory latency per
    // 2048 scores instead of one per 256)
    for (int x0 = tid; x0 < P; x0 += 8 * 256) {
        double sc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int x = x0 + e * 256;
            sc[e] = (x < n) ? row[x] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int x = x0 + e * 256;
            if (x >= P) break;
            key[x] = x < n ? score_key(sc[e]) : 0ull;
            id[x] = x < n ? x : 0x7fffffff;
        }
    }
    if (tid == 0) s_p = 0x7fffffff;
    __syncthreads();

    // ---- bitonic network; "a goes first" iff key larger, or equal and id smaller ----
    for (int size = 2; size <= P; size <<= 1) {
        for (int j = size >> 1, lj = 31 - __clz(size >> 1); j > 0; j >>= 1, --lj) {   // j = 1 << lj
            for (int t = tid; t < (P >> 1); t += 256) {
                int lo = ((t >> lj) << (lj + 1)) + (t & (j - 1));
                int hi = lo + j;
                bool up = (lo & size) == 0;
                unsigned long long ka = key[lo], kb = key[hi];
                int ia = id[lo], ib = id[hi];
                bool a_first = (ka > kb) || (ka == kb && ia < ib);
                if (a_first != up) {
                    key[lo] = kb; key[hi] = ka;
                    id[lo] = ib; id[hi] = ia;
                }
            }
            __syncthreads();
        }
    }
    for (int x = tid; x < n; x += 256)       // rank of the own chunk
        if (id[x] == own) s_p = x;
    __syncthreads();
    const int p = s_p;
    // chunk lengths along the ranking (chunk l left out) and their exclusive prefix sum
    int lens[32];
    const int per = P / 256 > 0 ? P / 256 : 1;           // consecutive ranks per thread
    int local = 0;
    for (int e = 0; e < per; ++e) {
        int r = tid * per + e;
        int len = 0;
        if (r < n) {
            int k = id[r];
            const int end = B[k + 1] < q_max ? B[k + 1] : q_max;
            len = (k == own) ? 0 : end - B[k];
        }
        lens[e] = len;
        local += len;
    }
    int total;
    int run = block_excl_scan(local, s_wave, &total);
    // the row's key array is dead now: reuse it as rem_by_id / pos_by_id
    int *rem_by_id = reinterpret_cast<int *>(smem);        // [P]
    int *pos_by_id = rem_by_id + P;                        // [P]
    __syncthreads();
    for (int e = 0; e < per; ++e) {
        int r = tid * per + e;
        if (r < n) {
            int k = id[r];
            int pos = blocks ? 3 : ((r < p) ? 0 : (r == p ? 1 : 2));
            int rem = N_b - run;                      // may be <= 0: not needed
            bool need = (pos == 2) ? (rem > 1) : (rem > 0);
            if (blocks && rem > lens[e]) rem = lens[e];   // tokens of the chunk in the block's list
            rem_by_id[k] = need ? rem : 0;
            pos_by_id[k] = pos;
        }
        run += lens[e];
    }
    __syncthreads();
    // compact in ascending chunk id
    int32_t *entries = plan + pl.off_entries + ((int64_t)h * pl.N_q + l) * pl.stride * 2;
    local = 0;
    for (int e = 0; e < per; ++e) {
        int k = tid * per + e;
        if (k < n && rem_by_id[k] != 0) ++local;
    }
    int slot = block_excl_scan(local, s_wave, &total);
    for (int e = 0; e < per; ++e) {
        int k = tid * per + e;
        if (k < n && rem_by_id[k] != 0) {
            if (slot < pl.stride) {
                entries[2 * slot] = k | (pos_by_id[k] << kPosShift);
                entries[2 * slot + 1] = rem_by_id[k];
            }
            ++slot;
        }
    }
    if (tid == 0) plan[pl.off_count + (int64_t)h * pl.N_q + l] = total < pl.stride ? total : pl.stride;
}

hipError_t launch_select(const Prob &p, const PlanLayout &pl, const double *Sc, int32_t *plan, hipStream_t s) {
    return launch_select_groups(p, pl, Sc, plan, 0, p.N_q, s);
}

// A launch (and its scores' way through memory) costs more than scoring every group by itself while a workgroup's four waves
// score all chunks in one go; from then on fifteen of sixteen rows of each product are what it pays for.  Routing in us,
// two launches -> one: 8 heads of 25 chunks 13.3 -> 10.4, of 60 chunks 15.2 -> 13.8 (row blocks 15.5 -> 13.1), 4 heads of 100
// chunks 15.2 -> 15.3, of 127 chunks 15.5 -> 18.9.  prefill of 1021 tokens 24.5 -> 21.8, of 2048 tokens in fp32 29.8 -> 27.4.
constexpr int kScoreSelectMax = 64;
bool score_select_ok(const Prob &p, const PlanLayout &pl) {
    return (int64_t)p.H_q * p.N_q < 512 && p.N_c <= kScoreSelectMax && pl.stride <= kSelMaxStride;
}

hipError_t launch_score_select(const Prob &p, const PlanLayout &pl, const double *Qc, const double *Kc, double *Sc, int32_t *plan,
                               hipStream_t s) {
    const int cap = select_cap(pl.stride), n_rows = p.H_q * p.N_q, row_bytes = (select_row_bytes(4, cap, p.N_c) + 15) / 16 * 16;
    const SelectArgs a = {plan, pl, p.N_c, p.N_b, p.B_r, 0, p.N_q, 0, n_rows, cap, row_bytes};
    const size_t shmem = row_bytes + 8 * (size_t)p.N_c;
    if (p.D == 64) hipLaunchKernelGGL(k_score_select<64>, dim3(n_rows), dim3(256), shmem, s, Qc, Kc, Sc, p.G, a);
    else hipLaunchKernelGGL(k_score_select<128>, dim3(n_rows), dim3(256), shmem, s, Qc, Kc, Sc, p.G, a);
    return hipGetLastError();
}

// One launch instead of three while scoring all chunks by eight waves and pooling side by side take no longer than a launch.
// A step in us, apart -> joined: 8 heads of 38 chunks 18.9 -> 16.2, with two chunks to pool 19.3 -> 18.0, 100 chunks 19.4 -> 17.8
// and 19.8 -> 19.5, 128 chunks 19.4 -> 18.5 and 19.7 -> 20.2, 200 chunks 19.6 -> 21.6; 32 heads of 128 chunks 20.0 -> 18.9.
// Long chunks, pooled by every head, would make the pooling the longest part.
bool route_decode_ok(const Prob &p, const PlanLayout &pl, int rb0, const BoundaryTail &tail) {
    int64_t longest = p.L - rb0;
    for (int j = 0; j < tail.n; ++j) longest = std::max<int64_t>(longest, tail.b[j + 1] - tail.b[j]);
    return tail.n > 0 && tail.n <= kRouteDecodeNew && p.N_c * tail.n <= 128 && longest <= 512 && pl.stride <= kSelMaxStride;
}

hipError_t launch_route_decode(const Prob &p, const PlanLayout &pl, int N_c_cap, int kc_valid, int rb0, const BoundaryTail &tail,
                               const void *Q, const void *K, double *Kc, int32_t *plan, int32_t *done, hipStream_t s) {
    const int cap = select_cap(pl.stride), row_bytes = (select_row_bytes(8, cap, p.N_c) + 15) / 16 * 16;
    const SelectArgs a = {plan, pl, p.N_c, p.N_b, p.B_r, p.N_q - 1, 1, 0, p.H_q, cap, row_bytes};
    const size_t shmem = row_bytes + 8 * (size_t)p.N_c + 4 * (size_t)(p.N_c + 1);
#define DHSA_ROUTED(T, DD)                                                                                              \
    hipLaunchKernelGGL((k_route_decode<T, DD>), dim3(p.H_q), dim3(512), shmem, s, (const T *)Q, (const T *)K, tail, done, Kc, a, \
                       p.H_kv, p.G, N_c_cap, kc_valid, rb0, (int)p.L, p.pooling, p.qs_h, p.qs_l, p.ks_h, p.ks_l)
    if (p.dtype == DHSA_F32) {
        if (p.D == 64) DHSA_ROUTED(float, 64); else DHSA_ROUTED(float, 128);
    } else {
        if (p.D == 64) DHSA_ROUTED(bf16_t, 64); else DHSA_ROUTED(bf16_t, 128);
    }
#undef DHSA_ROUTED
    return hipGetLastError();
}

hipError_t launch_select_groups(const Prob &p, const PlanLayout &pl, const double *Sc, int32_t *plan, int l_first,
                                int n_groups, hipStream_t s) {
    const int n_rows = n_groups * p.H_q;
    if (pl.stride > kSelMaxStride) {
        int P = 64;
        while (P < p.N_c) P <<= 1;
        const size_t shmem = (size_t)P * 12;
        if (shmem > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_select_sorted),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_select_sorted, dim3(n_groups, p.H_q), dim3(256), shmem, s, Sc, plan, pl, p.N_c, p.N_b,
                           p.B_r, l_first);
        return hipGetLastError();
    }
    // Waves per row: as many as hold its scores in eight registers a lane, and four where rows are few (a decoding
    // step).  Fewer waves with more scores each repeat less, but leave fewer rows in flight: 1634 chunks x 32
    // heads take 250 us with four waves, 315 us with one of 32 scores a lane.
    const int cap = select_cap(pl.stride);
    const int nw = n_rows < 512 ? 4 : p.N_c <= 512 ? 1 : p.N_c <= 1024 ? 2 : 4;
    const int row_bytes = select_row_bytes(nw, cap, p.N_c);
    const size_t shmem = nw == 1 ? (size_t)4 * row_bytes : row_bytes;
    const int per = nw == 1 ? 4 : 1;                     // rows per workgroup
    const dim3 block(nw == 1 ? 256 : 64 * nw);
#define DHSA_SELECT(NW)                                                                                            \
    do {                                                                                                           \
        if (shmem > 48 * 1024) {                                                                                   \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_select<NW>),                       \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);            \
            if (e != hipSuccess) return e;                                                                         \
        }                                                                                                          \
        for (int64_t r0 = 0; r0 < n_rows; r0 += (int64_t)kGridMax * per) {                                         \
            const dim3 grid((unsigned)std::min<int64_t>(kGridMax, (n_rows - r0 + per - 1) / per));                 \
            const SelectArgs a = {plan, pl, p.N_c, p.N_b, p.B_r, l_first, n_groups, (int)r0, n_rows, cap, row_bytes}; \
            hipLaunchKernelGGL(k_select<NW>, grid, block, shmem, s, Sc, a);                                        \
            const hipError_t e = hipGetLastError();                                                                \
            if (e != hipSuccess) return e;                                                                         \
        }                                                                                                          \
    } while (0)
    if (nw == 1) DHSA_SELECT(1);
    else if (nw == 2) DHSA_SELECT(2);
    else DHSA_SELECT(4);
#undef DHSA_SELECT
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Plan -> explicit index sets (Alg. 1's output) for a list of rows of one head.
// One wave per row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_expand(PlanView pv, int N_c, int head, const int64_t *__restrict__ rows,
                                               int32_t *__restrict__ idx, int cap, int32_t *__restrict__ cnt) {
    if (!plan_matches(pv)) return;   // not this problem's plan: nothing is written
    const int t = blockIdx.x, lane = threadIdx.x;
    const int64_t i = rows[t];
    const int l = chunk_of_row(pv.RB, pv.N_q, i);
    const int v = (int)(i + 1 - pv.RB[l]);
    const int E = pv.count[(int64_t)head * pv.N_q + l];
    const int32_t *ent = pv.entries + ((int64_t)head * pv.N_q + l) * pv.stride * 2;
    int32_t *out = idx + (int64_t)t * cap;
    int n = 0;
    for (int e = 0; e < E; ++e) {
        int w0 = ent[2 * e], rem = ent[2 * e + 1];
        int k = w0 & kChunkMask, pos = w0 >> kPosShift;
        int b0 = pv.B[k];
        int take = entry_take(pos, rem, pv.B[k + 1] - b0, v);
        for (int x = lane; x < take; x += 64)
            if (n + x < cap) out[n + x] = b0 + x;
        n += take;
    }
    for (int x = n + lane; x < cap; x += 64) out[x] = -1;
    if (lane == 0) cnt[t] = n;
}

hipError_t launch_expand(const Prob &p, const PlanView &pv, int head, const int64_t *rows_dev, int n_rows,
                         int32_t *idx, int cap, int32_t *cnt, hipStream_t s) {
    if (n_rows == 0) return hipSuccess;
    hipLaunchKernelGGL(k_expand, dim3(n_rows), dim3(64), 0, s, pv, p.N_c, head, rows_dev, idx, cap, cnt);
    return hipGetLastError();
}

}  // namespace dhsa
