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

#include "select.h"

namespace dhsa {

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

template <int NW>
__global__ __launch_bounds__(NW <= 4 ? 256 : 64 * NW, NW <= 4 ? 7 : 4) void k_select(const double *__restrict__ Sc, SelectArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned long long s_red[NW];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = a.r_first + (int)(NW == 1 ? blockIdx.x * (blockDim.x >> 6) + wave : blockIdx.x);
    if (r >= a.n_rows) return;           // NW == 1: waves do not wait for each other
    const int h = r / a.n_groups, l = r % a.n_groups;
    const int32_t *B = a.plan + a.pl.off_B;
    const int64_t group = (int64_t)h * a.pl.N_q + l;
    int2 *entries = reinterpret_cast<int2 *>(a.plan + a.pl.off_entries) + group * a.pl.stride;
    const int n = select_row<NW>(a, Sc + group * a.N_c, B, visible_chunks(a, B, l), smem + (size_t)(NW == 1 ? wave : 0) * a.row_bytes,
                                 s_red, [&](int i, int w, int rem) { entries[i] = make_int2(w, rem); });
    if ((NW == 1 ? threadIdx.x & 63 : threadIdx.x) == 0) a.plan[a.pl.off_count + group] = n;
}

// Scores and ranking of one (head, query group) by a workgroup, for problems of few groups and few chunks,
// where a launch takes longer than the scores of a group.  Bound by a chain: one memory latency, 32 products in a row, the ranking.
template <int D, int X>   // at most X chunks, 16 for each wave
__global__ __launch_bounds__(4 * X, X == 64 ? 2 : 1) void k_score_select(const double *__restrict__ Qc, const double *__restrict__ Kc,
                                                         double *__restrict__ Sc, int G, SelectArgs a) {
    __shared__ double s_row[X];
    __shared__ FewSmem<4 * X, X> sm;
    const int h = blockIdx.x / a.n_groups, l = blockIdx.x % a.n_groups;
    const int64_t group = (int64_t)h * a.pl.N_q + l;
    const int32_t *B = a.plan + a.pl.off_B;
    const Visible vis = visible_chunks(a, B, l);
    const int lane = threadIdx.x & 63, k0 = (int)(threadIdx.x >> 6) * 16, k = k0 + (lane & 15);
    if (k0 < vis.n) {
        f64x2 q[D / 8], b[D / 8];
        load_pooled<D>(b, Kc + ((int64_t)(h / G) * a.N_c + (k < vis.n ? k : vis.n - 1)) * D);
        load_pooled<D>(q, Qc + group * D);
        __builtin_amdgcn_sched_barrier(0);   // left alone, the scheduler moves the loads next to their use
        const double score = score_16<D>(q, b);
        if (lane < 16 && k < vis.n) {
            s_row[k] = score;
            Sc[group * a.N_c + k] = score;
        }
    }
    __syncthreads();
    int2 *entries = reinterpret_cast<int2 *>(a.plan + a.pl.off_entries) + group * a.pl.stride;
    const int n = select_few<4 * X, X>(a, s_row, B, vis, sm, [&](int i, int w, int rem) { entries[i] = make_int2(w, rem); });
    if (threadIdx.x == 0) a.plan[a.pl.off_count + group] = n;
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

// A launch (and its scores' way through memory) costs more than scoring every group by itself while there is one product
// chain or two for each SIMD; fifteen of sixteen rows of each product are what it pays for.  Routing in us, two launches ->
// one, heads of 128 (heads of 64): 8 heads of 25 chunks 13.1 -> 8.4 (11.8 -> 8.1), of 60 chunks 14.8 -> 12.0 (13.1 -> 9.8), row
// blocks 15.4 -> 11.4; 2 heads of 128 chunks 14.6 -> 13.9 (12.8 -> 11.4); 4 heads of 100 chunks 14.8 -> 17.5 (13.1 -> 11.4), of
// 127 15.1 -> 22.8 (13.3 -> 14.3); 1 head of 140 chunks 14.5 -> 17.7 (12.8 -> 13.3).
bool score_select_ok(const Prob &p) {
    const int64_t rows = (int64_t)p.H_q * p.N_q;
    return p.N_c <= 64 ? rows < 512 : p.N_c <= 128 && rows <= 256;
}

hipError_t launch_score_select(const Prob &p, const PlanLayout &pl, const double *Qc, const double *Kc, double *Sc, int32_t *plan,
                               hipStream_t s) {
    const int n_rows = p.H_q * p.N_q;
    const SelectArgs a = {plan, pl, p.N_c, p.N_b, p.B_r, 0, p.N_q, 0, n_rows, 0, 0};
#define DHSA_SCORE_SELECT(DD, X) hipLaunchKernelGGL((k_score_select<DD, X>), dim3(n_rows), dim3(4 * X), 0, s, Qc, Kc, Sc, p.G, a)
    if (p.N_c <= 64) { if (p.D == 64) DHSA_SCORE_SELECT(64, 64); else DHSA_SCORE_SELECT(128, 64); }
    else { if (p.D == 64) DHSA_SCORE_SELECT(64, 128); else DHSA_SCORE_SELECT(128, 128); }
#undef DHSA_SCORE_SELECT
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
    // Eight waves where a CU has one row at most and that is long: a decoding step over 1634 chunks, 32 heads 46.6 -> 44.9 us, over
    // 4000, 16 heads 44.7 -> 34.8, over 1000, 8 heads 25.1 -> 24.2; over 400, 32 heads 25.4 -> 25.0, over 200 22.1 -> 22.3.  Sixteen
    // take 44.8, 33.8, 24.6, 25.6 and 23.0.
    const int nw = n_rows <= 256 && p.N_c > 512 ? 8 : n_rows < 512 ? 4 : p.N_c <= 512 ? 1 : p.N_c <= 1024 ? 2 : 4;
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
    else if (nw == 8) DHSA_SELECT(8);
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
