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

// Value of lane (lane ^ J) of the wave, J a power of two below 64: lane-crossing moves of the
// vector unit where there is one (quads, rows of 16), the LDS crossbar otherwise.
template <int J>
__device__ __forceinline__ int lane_xor(int v) {
    if constexpr (J == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);        // quad_perm [1,0,3,2]
    else if constexpr (J == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
    else if constexpr (J == 4) return __builtin_amdgcn_ds_swizzle(v, 0x101F);              // xor 4 inside 32 lanes
    else if constexpr (J == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);  // row_ror 8 == xor 8
    else if constexpr (J == 16) return __builtin_amdgcn_ds_swizzle(v, 0x401F);             // xor 16 inside 32 lanes
    else return __shfl_xor(v, 32);
}

// Bitonic sort of PS <= 256 (key, id) pairs, one per thread of the first PS threads, "first"
// = larger key, or equal key and smaller id.  In: skey[0..PS), sid[0..PS); out: the same
// arrays, sorted.  Exchanges at distances below 64 stay inside a wave, the few at 64 and 128
// go through the arrays.  Called by all 256 threads (barriers).
template <int PS, int SIZE, int J>
__device__ __forceinline__ void sort_step(unsigned long long &k, int &ci, unsigned long long *skey, int *sid,
                                          int tid, bool active) {
    unsigned long long pk = 0ull;
    int pi = 0;
    if constexpr (J < 64) {
        if (active) {
            const int lo = lane_xor<J>((int)(unsigned)k), hi = lane_xor<J>((int)(unsigned)(k >> 32));
            pk = ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
            pi = lane_xor<J>(ci);
        }
    } else {
        __syncthreads();           // the previous exchange has been read
        if (active) { skey[tid] = k; sid[tid] = ci; }
        __syncthreads();
        if (active) { pk = skey[tid ^ J]; pi = sid[tid ^ J]; }
    }
    if (active) {
        const bool first = (k > pk) || (k == pk && ci < pi);
        const bool want_first = ((tid & J) == 0) == ((tid & SIZE) == 0);
        if (first != want_first) { k = pk; ci = pi; }
    }
    if constexpr (J > 1) sort_step<PS, SIZE, J / 2>(k, ci, skey, sid, tid, active);
    else if constexpr (SIZE < PS) sort_step<PS, SIZE * 2, SIZE>(k, ci, skey, sid, tid, active);
}

template <int PS>
__device__ __forceinline__ void sort_in_registers(unsigned long long *skey, int *sid, int tid) {
    const bool active = tid < PS;      // PS is a multiple of 64: whole waves; the others only keep the barriers company
    unsigned long long k = active ? skey[tid] : 0ull;
    int ci = active ? sid[tid] : 0x7fffffff;
    sort_step<PS, 2, 1>(k, ci, skey, sid, tid, active);
    __syncthreads();
    if (active) { skey[tid] = k; sid[tid] = ci; }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Ranking + per-row budget for one (head, query chunk l): Alg. 1's Argsort and
// walk, done once for all rows of the chunk.
//   1. scores of key chunks 0..l -> LDS as order-preserving 64-bit integers;
//   2. only the best `stride` chunks can ever be listed (stride bounds the number
//      of chunks whose tokens fit the budget), so for rows of more than 256 chunks a
//      most-significant-digit radix select (8-bit digits, LDS histograms, prefix
//      scans) first cuts the row down to a candidate list: at first a short one,
//      sized for chunks of about the mean length (it is the answer whenever its
//      chunks hold the budget), else one of <= 512 that holds `stride` chunks;
//   3. bitonic sort of the candidates (of the whole row if there was no select),
//      larger score first, equal scores lower id first; up to 256 elements are
//      sorted in registers, one per thread, more in LDS;
//   4. exclusive prefix sum of chunk lengths along the ranking, chunk l left out
//      -> rem = N_b - (tokens of other chunks before this rank);
//   5. a chunk is kept if some row takes a token of it; kept chunks are
//      compacted in ascending chunk id (prefix sum of flags) into the plan.
// Row-block form (B_r > 0, Alg. 1 as printed): query group l is a row block,
// the candidates are the chunks that start before the block's end q_max, their
// lengths are clipped to q_max, there is no "own chunk", and an entry records
// how many tokens of the chunk the block's list holds (pos = 3).
// ---------------------------------------------------------------------------
constexpr int kMaxCand = 512;     // candidates kept by the radix select
constexpr int kSelectMin = 256;   // rows with more chunks than this use it; shorter rows are sorted whole, in registers

__global__ __launch_bounds__(256) void k_select(const double *__restrict__ Sc, int32_t *__restrict__ plan,
                                                PlanLayout pl, int N_c, int N_b, int B_r, int smem_bytes,
                                                int guess, int l_first) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_wave[4];
    __shared__ int s_p;
    __shared__ int s_hist[256];
    __shared__ int s_digit, s_above, s_equal;
    const int l = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const int32_t *B = plan + pl.off_B;
    const bool blocks = B_r > 0;
    const int q_max = blocks ? (plan + pl.off_RB)[l + 1] : 0x7fffffff;   // clip of the chunk lengths
    // l indexes Sc, RB and the plan; the group's number in the sequence is l_first + l (a launch
    // may cover a suffix of the groups, laid out from 0)
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
            unsigned long long u = 0ull;
            int k = 0x7fffffff;
            if (x < n) {
                double s = sc[e];
                if (s == 0.0) s = 0.0;  // -0.0 ties with +0.0
                u = (unsigned long long)__double_as_longlong(s);
                u = (u >> 63) ? ~u : (u | 0x8000000000000000ull);
                k = x;
            }
            key[x] = u;
            id[x] = k;
        }
    }
    __syncthreads();

    // What gets sorted: the whole row in place, or the candidates of a radix select.  The select
    // is tried first with `guess` chunks (the number that holds the budget if the best chunks
    // have about the mean length): the sorted candidates are exactly the head of the full
    // ranking, so if their lengths add up to the budget no later chunk can be listed and the
    // short sort is the answer.  Otherwise the select is redone with `stride` chunks, the bound
    // that always suffices.
    const bool can_select = n > kSelectMin && pl.stride <= kMaxCand - 64 && P * 8 + kMaxCand * 12 <= smem_bytes;
    int cap0 = 64;
    while (cap0 < guess) cap0 <<= 1;
    unsigned long long *skey = key;
    int *sid = id;
    int Ps = P, ns = n;
    int p = 0x7fffffff, run = 0;
    int lens[32];
    bool id_intact = true;
    for (int attempt = (can_select && guess < pl.stride && cap0 < kMaxCand) ? 0 : 1;; ++attempt) {
        skey = key;
        sid = id;
        Ps = P;
        ns = n;
        if (can_select) {
            // ---- radix select: smallest set {key >= threshold prefix} holding the best `need` ----
            const int cap = attempt == 0 ? cap0 : kMaxCand;
            const int goal = attempt == 0 ? guess : pl.stride;
            const int need = goal < n ? goal : n;
            unsigned long long prefix = 0ull;
            int above = 0, equal = n, shift = 64;
            for (int pass = 0; pass < 8 && above + equal > cap; ++pass) {
                shift = 56 - 8 * pass;
                s_hist[tid] = 0;
                __syncthreads();
                for (int x = tid; x < n; x += 256) {
                    const unsigned long long k = key[x];
                    if (pass == 0 || (k >> (shift + 8)) == prefix)
                        atomicAdd(&s_hist[(int)((k >> shift) & 255ull)], 1);
                }
                __syncthreads();
                // suffix counts over digits: thread t looks at digit 255 - t
                const int d = 255 - tid, cnt = s_hist[d];
                int total;
                const int gt = block_excl_scan(cnt, s_wave, &total);   // elements of the region with a larger digit
                const int want = need - above;                         // still to be found inside the region
                if (gt < want && gt + cnt >= want) { s_digit = d; s_above = gt; s_equal = cnt; }
                __syncthreads();
                above += s_above;
                equal = s_equal;
                prefix = (prefix << 8) | (unsigned long long)s_digit;
                __syncthreads();
            }
            if (above + equal <= cap) {
                // ---- compact the candidates, in chunk-id order, into their own arrays ----
                unsigned long long *ckey = reinterpret_cast<unsigned long long *>(smem + (size_t)P * 8);  // over id[]
                int *cid = reinterpret_cast<int *>(ckey + kMaxCand);
                const int per = (n + 255) / 256;
                const bool all = shift == 64;   // no radix pass ran (n <= cap): every element is a candidate
                int local = 0;
                for (int e = 0; e < per; ++e) {
                    const int x = tid * per + e;
                    if (x < n && (all || (key[x] >> shift) >= prefix)) ++local;
                }
                int total;
                int slot = block_excl_scan(local, s_wave, &total);
                __syncthreads();               // id[] is dead (ids are positions), its space is reused now
                id_intact = false;
                for (int e = 0; e < per; ++e) {
                    const int x = tid * per + e;
                    if (x < n && (all || (key[x] >> shift) >= prefix)) { ckey[slot] = key[x]; cid[slot] = x; ++slot; }
                }
                ns = total;
                Ps = 64;
                while (Ps < ns) Ps <<= 1;
                for (int x = ns + tid; x < Ps; x += 256) { ckey[x] = 0ull; cid[x] = 0x7fffffff; }
                skey = ckey;
                sid = cid;
                __syncthreads();
            } else if (attempt == 0) {
                continue;                      // too many equal scores for the short sort
            } else if (!id_intact) {           // whole-row sort after a first attempt: ids are positions
                for (int x = tid; x < P; x += 256) id[x] = x < n ? x : 0x7fffffff;
                __syncthreads();
            }
        }

        // ---- bitonic network; "a goes first" iff key larger, or equal and id smaller ----
        if (Ps <= 256) {
            if (Ps == 64) sort_in_registers<64>(skey, sid, tid);
            else if (Ps == 128) sort_in_registers<128>(skey, sid, tid);
            else sort_in_registers<256>(skey, sid, tid);
        } else
        for (int size = 2; size <= Ps; size <<= 1) {
            for (int j = size >> 1, lj = 31 - __clz(size >> 1); j > 0; j >>= 1, --lj) {   // j = 1 << lj
                for (int t = tid; t < (Ps >> 1); t += 256) {
                    int lo = ((t >> lj) << (lj + 1)) + (t & (j - 1));
                    int hi = lo + j;
                    bool up = (lo & size) == 0;
                    unsigned long long ka = skey[lo], kb = skey[hi];
                    int ia = sid[lo], ib = sid[hi];
                    bool a_first = (ka > kb) || (ka == kb && ia < ib);
                    if (a_first != up) {
                        skey[lo] = kb; skey[hi] = ka;
                        sid[lo] = ib; sid[hi] = ia;
                    }
                }
                __syncthreads();
            }
        }
        // rank of chunk l (beyond every candidate if it is not one of them)
        if (tid == 0) s_p = 0x7fffffff;
        __syncthreads();
        for (int x = tid; x < ns; x += 256)
            if (sid[x] == own) s_p = x;
        __syncthreads();
        p = s_p;
        // chunk lengths along the ranking (chunk l left out) and their exclusive prefix sum
        const int per = Ps / 256 > 0 ? Ps / 256 : 1;           // consecutive ranks per thread
        int local = 0;
        for (int e = 0; e < per; ++e) {
            int r = tid * per + e;
            int len = 0;
            if (r < ns) {
                int k = sid[r];
                const int end = B[k + 1] < q_max ? B[k + 1] : q_max;
                len = (k == own) ? 0 : end - B[k];
            }
            lens[e] = len;
            local += len;
        }
        int total;
        run = block_excl_scan(local, s_wave, &total);
        if (attempt == 0 && ns < n && total < N_b) {
            __syncthreads();                   // every thread is done with the candidates
            continue;
        }
        break;
    }
    // the row's key array is dead now: reuse it as rem_by_id / pos_by_id
    int *rem_by_id = reinterpret_cast<int *>(smem);        // [P]
    int *pos_by_id = rem_by_id + P;                        // [P]
    if (skey != key) {                                     // chunks that are no candidates are not listed
        for (int x = tid; x < n; x += 256) rem_by_id[x] = 0;
    }
    __syncthreads();  // the zero fill is complete
    {
        const int per = Ps / 256 > 0 ? Ps / 256 : 1;
        for (int e = 0; e < per; ++e) {
            int r = tid * per + e;
            if (r < ns) {
                int k = sid[r];
                int pos = blocks ? 3 : ((r < p) ? 0 : (r == p ? 1 : 2));
                int rem = N_b - run;                      // may be <= 0: not needed
                bool need = (pos == 2) ? (rem > 1) : (rem > 0);
                if (blocks && rem > lens[e]) rem = lens[e];   // tokens of the chunk in the block's list
                rem_by_id[k] = need ? rem : 0;
                pos_by_id[k] = pos;
            }
            run += lens[e];
        }
    }
    __syncthreads();
    // compact in ascending chunk id
    int32_t *entries = plan + pl.off_entries + ((int64_t)h * pl.N_q + l) * pl.stride * 2;
    {
        const int per_id = P / 256 > 0 ? P / 256 : 1;
        int local = 0;
        for (int e = 0; e < per_id; ++e) {
            int k = tid * per_id + e;
            if (k < n && rem_by_id[k] != 0) ++local;
        }
        int total;
        int slot = block_excl_scan(local, s_wave, &total);
        for (int e = 0; e < per_id; ++e) {
            int k = tid * per_id + e;
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
}

hipError_t launch_select(const Prob &p, const PlanLayout &pl, const double *Sc, int32_t *plan, hipStream_t s) {
    return launch_select_groups(p, pl, Sc, plan, 0, p.N_q, s);
}

hipError_t launch_select_groups(const Prob &p, const PlanLayout &pl, const double *Sc, int32_t *plan, int l_first,
                                int n_groups, hipStream_t s) {
    int P = 64;
    while (P < p.N_c) P <<= 1;
    size_t shmem = (size_t)P * 8 + std::max<size_t>((size_t)P * 4, (size_t)kMaxCand * 12);   // keys + (ids | candidates)
    if (shmem > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_select),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_select, dim3(n_groups, p.H_q), dim3(256), shmem, s, Sc, plan, pl, p.N_c, p.N_b, p.B_r,
                       (int)shmem, pl.guess > 0 ? pl.guess : 1, l_first);
    return hipGetLastError();
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
