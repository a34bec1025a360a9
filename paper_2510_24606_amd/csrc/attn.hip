// fp32 sparse attention kernel of libdhsa: exact softmax attention over the keys
// the routing plan selects (Alg. 2 / Alg. 3 of the paper, App. C "Backend
// implementations") for DHSA_F32 inputs, fp32 throughout.  The bf16 kernel is in
// attn_mfma.hip.
//
// Work unit: (query head, 16 RW consecutive rows of one row tile of the plan).  Four
// waves; each owns every fourth block of 16 selected keys and all rows, and the
// waves merge their softmax states at the end, so the loop over the keys has no
// barrier and K / V go from memory straight into registers.
//
// v_mfma_f32_16x16x4_f32 (full fp32 products and sums).  Lane l = 16 q + n.
// S^T (16 keys x 16 rows) += K (16 x 4) Q^T (4 x 16): the lane supplies K of key n and
// Q of row n at d = 16 s + 4 q + j (step j of the group s: the contraction index may
// be any order of d, this one makes both operands 16-byte loads) and receives the
// scores of row n against keys 4 q + {0..3}, which are the B operand of
// O^T (16 d x 16 rows) += V^T (16 x 4) P^T (4 x 16) when step i contracts the keys
// {4 q + i : q}.  V^T of step i: 16 bytes at d = 64 t + 4 n of key 4 q + i, one element
// for each of four output blocks (block (t, j) holds d = 64 t + 4 M + j in row M).
//
// Bound by the fp32 rate of the matrix unit once the chip is full; small problems by
// the chain of loads before the first product (plan, boundaries, keys).  L = 2048, four
// heads of D = 64, N_b = 256: 18 us; 135 us with one wave per row (no reuse of K and V, products on
// the vector unit, one key of V at a time).
#include <algorithm>
#include <type_traits>

#include "select.h"

namespace dhsa {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Keys = 1024;   // selected keys whose positions and masks are in LDS at a time
constexpr int kF32Seg = 256;     // plan entries per batch

// D = 64, RW = 2 is held to three waves per SIMD (168 registers, nothing spilled; left to itself it takes 178): L = 8192,
// N_b = 512, 16 heads 285 -> 250 us.  D = 128, RW = 2 spills four registers, once per window of
// keys; the loop over the keys has none.
// With F32RouteArgs the workgroup does its query group's routing itself (route_tile); what bounds problems of few tiles is the chain of
// launches, and of the loads that each begins with.
struct F32RouteArgs {
    SelectArgs sel;
    const double *Qc, *Kc;
    double *Sc;
};
struct NoRoute {};
template <int D, int RW, typename ROUTE>
__global__ __launch_bounds__(256, D == 64 && RW == 2 ? 3 : 2) void k_attn_f32(PlanView pv, ROUTE route, const float *__restrict__ Q,
                                                     const float *__restrict__ K, const float *__restrict__ V,
                                                     float *__restrict__ O, unsigned block0, int H_q, int G, float scale_log2e,
                                                     int64_t qs_h, int64_t qs_l, int64_t ks_h, int64_t ks_l,
                                                     int64_t vs_h, int64_t vs_l, int64_t os_h, int64_t os_l) {
    constexpr int NR = 16 * RW;      // rows of the workgroup
    constexpr int NS = D / 16;       // 16-byte pieces of a K / Q row per lane
    constexpr int NT = D / 64;
    constexpr int kPad = D + 4;
    struct Lists {
        int key[kF32Keys], lo[kF32Keys], hi[kF32Keys];           // a row takes the key iff lo < v < hi
        int start[kF32Seg + 1], b0[kF32Seg], pos[kF32Seg], rem[kF32Seg];
        int wave[8];
    };
    struct Merge {
        float o[4][NR][kPad];
        float m[4][NR], l[4][NR];
        int odd[4];
    };
    __shared__ __align__(16) union { Lists li; Merge me; } sm;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;

    // blockIdx -> (head, tile, piece of the tile): a tile of class c has at most 4 - c pieces of 32 rows; the
    // latest rows (most keys) of each class first
    const unsigned block = block0 + blockIdx.x;
    const int h = block % H_q, g = h / G;
    int b = block / H_q, tile = 0, piece = 0;
    {
        int first = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int pieces = (4 - c) * 32 / NR, T = pv.T_cls[c];
            if (b >= 0 && b < T * pieces) { tile = first + T - 1 - b / pieces; piece = b % pieces; }
            b -= T * pieces;
            first += T;
        }
    }
    const int l = pv.tiles[2 * tile], tile0 = pv.tiles[2 * tile + 1];
    if (!plan_matches(pv)) return;   // not this problem's plan: nothing else is used, O is not written
    const int row0 = tile0 + piece * NR;
    const int b_l = pv.RB[l], tile_end = tile0 + kRowTile;
    const int end = pv.RB[l + 1] < tile_end ? pv.RB[l + 1] : tile_end;
    const int nrows = end - row0 < NR ? end - row0 : NR;
    if (nrows <= 0) return;          // the tile has fewer pieces than its class allows
    const int v_lo = row0 + 1 - b_l, v_hi = v_lo + nrows - 1;
    constexpr bool kRoute = !std::is_same<ROUTE, NoRoute>::value;
    __shared__ std::conditional_t<kRoute, RouteScratch, NoRoute> rs;
    TileList list;
    if constexpr (kRoute) list = route_tile<D>(rs, pv, route.sel, route.Qc, route.Kc, route.Sc, G, h, l, row0 == b_l);
    else list = plan_list(pv, h, l);
    // the entries of the first batch do not wait for their number, and the query rows are requested behind what the key
    // list hangs on
    const int E = list.E;
    const int2 *ent = list.ent;
    int2 ent_e = ent[tid < pv.stride ? tid : 0];
    if (tid >= E) ent_e = int2{0, 0};   // past the list: nothing there has been written
    int b0_e = list.B[ent_e.x & kChunkMask], b1_e = list.B[(ent_e.x & kChunkMask) + 1];
    const float *Kg = K + (int64_t)g * ks_h + 4 * q4;
    const float *Vg = V + (int64_t)g * vs_h + 4 * n16;

    // rows past the end repeat the last one (never stored)
    f32x4 qf[RW][NS], oacc[RW][NT][4];
    int v_i[RW];
    float m[RW], lsum[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int row = 16 * r + n16 < nrows ? 16 * r + n16 : nrows - 1;
        const float *qp = Q + (int64_t)h * qs_h + (int64_t)(row0 + row) * qs_l + 4 * q4;
#pragma unroll
        for (int s = 0; s < NS; ++s) qf[r][s] = *reinterpret_cast<const f32x4 *>(qp + 16 * s);
        v_i[r] = v_lo + row;
        m[r] = -INFINITY;
        lsum[r] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) oacc[r][t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    bool odd = false;                // infinities or NaN of V were left out of the products
    for (int e0 = 0; e0 < E; e0 += kF32Seg) {
        // segments (entries some row takes a key from) of this batch, compacted
        if (e0 > 0) {
            ent_e = e0 + tid < E ? ent[e0 + tid] : int2{0, 0};
            b0_e = list.B[ent_e.x & kChunkMask];
            b1_e = list.B[(ent_e.x & kChunkMask) + 1];
        }
        int n_e = 0;
        const int pos_e = ent_e.x >> kPosShift, rem_e = ent_e.y;
        if (e0 + tid < E) {
            n_e = entry_take(pos_e, rem_e, b1_e - b0_e, pos_e == 1 ? v_hi : v_lo);
            if (pos_e == 3) {        // row-block form: keys past the last row are dropped
                const int vis = row0 + nrows - b0_e;
                n_e = vis < n_e ? (vis > 0 ? vis : 0) : n_e;
            }
        }
        int total, nseg, start, slot;
        block_excl_scan2(n_e, n_e > 0 ? 1 : 0, sm.li.wave, &start, &slot, &total, &nseg);
        if (n_e > 0) {
            sm.li.start[slot] = start;
            sm.li.b0[slot] = b0_e;
            sm.li.pos[slot] = pos_e;
            sm.li.rem[slot] = rem_e;
        }
        if (tid == 0) sm.li.start[nseg] = total;
        for (int x0 = 0; x0 < total; x0 += kF32Keys) {
            const int nk = total - x0 < kF32Keys ? total - x0 : kF32Keys;
            const int nb = (nk + 15) >> 4;
            __syncthreads();         // the segment table is complete; the last window's lists are done with
            for (int sg = wave; sg < nseg; sg += 4) {
                const int st = sm.li.start[sg], en = sm.li.start[sg + 1];
                const int lo = st > x0 ? st : x0, hi = en < x0 + nk ? en : x0 + nk;
                if (lo >= hi) continue;
                const int b0 = sm.li.b0[sg], pos = sm.li.pos[sg], rem = sm.li.rem[sg];
                for (int x = lo + lane; x < hi; x += 64) {
                    const int t = x - st, j = b0 + t;
                    sm.li.key[x - x0] = j;
                    // key j is at or below row i  <=>  j - b_l < v: the group's own chunk (pos 1) and every
                    // listed key of the row-block form (pos 3)
                    sm.li.lo[x - x0] = (pos & 1) ? (j > b_l ? j - b_l : 0) : 0;
                    sm.li.hi[x - x0] = (pos == 2) ? rem - t : 0x7fffffff;
                }
            }
            for (int x = nk + tid; x < nb * 16; x += 256) {   // padding: a row that exists, taken by nobody
                sm.li.key[x] = row0;
                sm.li.lo[x] = 0x7fffffff;
                sm.li.hi[x] = 0x7fffffff;
            }
            __syncthreads();

            f32x4 kf[NS], vf[4][NT];
#define DHSA_F32_K(kb)                                                                                       \
    {                                                                                                        \
        const float *kp_ = Kg + (int64_t)sm.li.key[(kb) * 16 + n16] * ks_l;                                  \
        _Pragma("unroll") for (int s = 0; s < NS; ++s) kf[s] = *reinterpret_cast<const f32x4 *>(kp_ + 16 * s); \
    }
#define DHSA_F32_V(kb)                                                                                       \
    {                                                                                                        \
        const int4 j_ = *reinterpret_cast<const int4 *>(&sm.li.key[(kb) * 16 + 4 * q4]);                     \
        const int jj_[4] = {j_.x, j_.y, j_.z, j_.w};                                                         \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                        \
            _Pragma("unroll") for (int t = 0; t < NT; ++t)                                                   \
                vf[i][t] = *reinterpret_cast<const f32x4 *>(Vg + (int64_t)jj_[i] * vs_l + 64 * t);           \
    }
            if (wave < nb) { DHSA_F32_K(wave); DHSA_F32_V(wave); }
            for (int kb = wave; kb < nb; kb += 4) {
                // Four partial sums of D / 4 products each, one after the other (all four at once spill 40 registers at
                // D = 128, RW = 2): rounded along one chain of D products a score, and with it O, is further from its
                // 64-bit value (relative 2.7e-7 against 1.5e-7 at L = 2048, D = 64; 3.3e-7 against 2.0e-7 at L = 5061,
                // D = 128).
                f32x4 s[RW];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4 part[RW];
#pragma unroll
                    for (int c = 0; c < NS; ++c)
#pragma unroll
                        for (int r = 0; r < RW; ++r)
                            part[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j], qf[r][c][j],
                                                                           c ? part[r] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < RW; ++r) s[r] = j ? s[r] + part[r] : part[r];
                }
                if (kb + 4 < nb) DHSA_F32_K(kb + 4);        // lands while this block is finished
                const int4 lo = *reinterpret_cast<const int4 *>(&sm.li.lo[kb * 16 + 4 * q4]);
                const int4 hi = *reinterpret_cast<const int4 *>(&sm.li.hi[kb * 16 + 4 * q4]);
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    s[r][0] = ((v_i[r] > lo.x) & (v_i[r] < hi.x)) ? s[r][0] : -INFINITY;
                    s[r][1] = ((v_i[r] > lo.y) & (v_i[r] < hi.y)) ? s[r][1] : -INFINITY;
                    s[r][2] = ((v_i[r] > lo.z) & (v_i[r] < hi.z)) ? s[r][2] : -INFINITY;
                    s[r][3] = ((v_i[r] > lo.w) & (v_i[r] < hi.w)) ? s[r][3] : -INFINITY;
                    float mx = fmaxf(fmaxf(s[r][0], s[r][1]), fmaxf(s[r][2], s[r][3]));
                    mx = fmaxf(mx, __shfl_xor(mx, 16));     // the four lanes of a row
                    mx = fmaxf(mx, __shfl_xor(mx, 32));
                    if (__any(mx > m[r])) {
                        const float m_new = fmaxf(m[r], mx);
                        const float alpha = m[r] == -INFINITY ? 0.f
                                            : __builtin_amdgcn_exp2f((m[r] - m_new) * scale_log2e);
                        lsum[r] *= alpha;
#pragma unroll
                        for (int t = 0; t < NT; ++t)
#pragma unroll
                            for (int j = 0; j < 4; ++j) oacc[r][t][j] *= alpha;
                        m[r] = m_new;
                    }
                    const float ref = m[r] == -INFINITY ? 0.f : m[r];   // no key seen yet: every p is 0
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s[r][i] = __builtin_amdgcn_exp2f((s[r][i] - ref) * scale_log2e);
                        lsum[r] += s[r][i];
                    }
                }
                // Infinities and NaN in V of a block with keys that not every row takes: 0 V does not keep them out of
                // the other rows, so the products get zeros and the rows that take them get them at the end.
                if (__any(max(max(lo.x, lo.y), max(lo.z, lo.w)) >= v_lo || min(min(hi.x, hi.y), min(hi.z, hi.w)) <= v_hi)) {
                    float z = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
#pragma unroll
                            for (int j = 0; j < 4; ++j) z = __builtin_fmaf(vf[i][t][j], 0.f, z);
                    if (__any(z != 0.f)) {
                        odd = true;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    vf[i][t][j] = fabsf(vf[i][t][j]) < INFINITY ? vf[i][t][j] : 0.f;
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int r = 0; r < RW; ++r)
                                oacc[r][t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][t][j], s[r][i], oacc[r][t][j],
                                                                                     0, 0, 0);
                if (kb + 4 < nb) DHSA_F32_V(kb + 4);
            }
#undef DHSA_F32_K
#undef DHSA_F32_V
        }
    }

    // ---- merge of the four waves, normalisation, store ----
    __syncthreads();                 // the lists are dead
    if (lane == 0) sm.me.odd[wave] = odd;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        lsum[r] += __shfl_xor(lsum[r], 16);
        lsum[r] += __shfl_xor(lsum[r], 32);
        if (q4 == 0) {
            sm.me.m[wave][16 * r + n16] = m[r];
            sm.me.l[wave][16 * r + n16] = lsum[r];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                *reinterpret_cast<f32x4 *>(&sm.me.o[wave][16 * r + n16][64 * t + 16 * q4 + 4 * x]) =
                    f32x4{oacc[r][t][0][x], oacc[r][t][1][x], oacc[r][t][2][x], oacc[r][t][3][x]};
    }
    __syncthreads();
    for (int x = tid; x < nrows * (D / 4); x += 256) {
        const int r = x / (D / 4), d = (x % (D / 4)) * 4;
        float M = sm.me.m[0][r];
#pragma unroll
        for (int w = 1; w < 4; ++w) M = fmaxf(M, sm.me.m[w][r]);
        float L = 0.f;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = sm.me.m[w][r];
            const float a = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mw - M) * scale_log2e);
            L += sm.me.l[w][r] * a;
            acc += *reinterpret_cast<const f32x4 *>(&sm.me.o[w][r][d]) * a;
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;   // a row that sees no key of its block's list: zeros
        acc *= inv;
        const bool none = L == 0.f;                  // no key at all, or only keys whose score is -inf: NaN
        if (none | sm.me.odd[0] | sm.me.odd[1] | sm.me.odd[2] | sm.me.odd[3]) {
            for (int e = 0; e < E; ++e) {
                const int2 w = ent[e];
                const int k = w.x & kChunkMask, pos = w.x >> kPosShift, b0 = list.B[k];
                int take = entry_take(pos, w.y, list.B[k + 1] - b0, v_lo + r);
                if (pos == 3 && row0 + r + 1 - b0 < take) take = row0 + r + 1 - b0;   // listed keys past the row
                if (none) {
                    if (take > 0) acc = f32x4{NAN, NAN, NAN, NAN};
                    continue;
                }
                for (int t = 0; t < take; ++t) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(V + (int64_t)g * vs_h + (int64_t)(b0 + t) * vs_l + d);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[j] += fabsf(v[j]) < INFINITY ? 0.f : v[j];
                }
            }
        }
        *reinterpret_cast<f32x4 *>(O + (int64_t)h * os_h + (int64_t)(row0 + r) * os_l + d) = acc;
    }
}

// ---------------------------------------------------------------------------
// Row blocks of so few rows that the 16-row products are mostly padding: a wave per row.  Lanes take the scores of up to
// 64 keys of a plan entry, then own output columns.  A score is four partial sums, as above.  Bound by latency (a key
// row per lane, one key of V at a time).  L = 6000, 8 heads, D = 128, B_r = 1: N_b = 16 694 -> 146 us, N_b = 700 4.8 -> 2.8 ms.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void k_attn_f32_rows(PlanView pv, const float *__restrict__ Q,
                                                       const float *__restrict__ K, const float *__restrict__ V,
                                                       float *__restrict__ O, int64_t L, int G, int B_r, float scale_log2e,
                                                       int64_t qs_h, int64_t qs_l, int64_t ks_h, int64_t ks_l,
                                                       int64_t vs_h, int64_t vs_l, int64_t os_h, int64_t os_l) {
    constexpr int NC = D / 64;       // output columns per lane
    __shared__ __align__(16) float s_q[4][D];
    if (!plan_matches(pv)) return;   // not this problem's plan: O is not written
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = blockIdx.y, g = h / G;
    const int64_t i = (int64_t)blockIdx.x * 4 + wave;
    const bool live = i < L;
    if (live)
        for (int d = lane; d < D; d += 64) s_q[wave][d] = Q[(int64_t)h * qs_h + i * qs_l + d];
    __syncthreads();
    if (!live) return;
    const float *Kg = K + (int64_t)g * ks_h, *Vg = V + (int64_t)g * vs_h;
    const int l = (int)(i / B_r);
    const int E = pv.count[(int64_t)h * pv.N_q + l];
    const int2 *ent = reinterpret_cast<const int2 *>(pv.entries) + ((int64_t)h * pv.N_q + l) * pv.stride;
    float m = -INFINITY, lsum = 0.f, o[NC];
    bool some = false;               // the row takes a key
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = 0.f;
    for (int e = 0; e < E; ++e) {
        const int2 w = ent[e];
        const int b0 = pv.B[w.x & kChunkMask];
        const int64_t vis = i + 1 - b0;                  // listed keys past the row are dropped
        const int take = vis < w.y ? (vis > 0 ? (int)vis : 0) : w.y;
        some |= take > 0;
        for (int t0 = 0; t0 < take; t0 += 64) {
            const int nv = take - t0 < 64 ? take - t0 : 64;
            float s = -INFINITY;
            if (lane < nv) {
                const float *kr = Kg + (int64_t)(b0 + t0 + lane) * ks_l;
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int d = 0; d < D; d += 4) {
                    const f32x4 k4 = *reinterpret_cast<const f32x4 *>(kr + d), q4 = *reinterpret_cast<const f32x4 *>(&s_q[wave][d]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[j] = __builtin_fmaf(k4[j], q4[j], acc[j]);
                }
                s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
            float mx = s;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
            const float m_new = fmaxf(m, mx), ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_new) * scale_log2e);
            const float p = lane < nv ? __builtin_amdgcn_exp2f((s - ref) * scale_log2e) : 0.f;
            lsum = lsum * alpha + p;
#pragma unroll
            for (int c = 0; c < NC; ++c) o[c] *= alpha;
            for (int jj = 0; jj < nv; ++jj) {
                const float pj = __shfl(p, jj);
                const float *vr = Vg + (int64_t)(b0 + t0 + jj) * vs_l + lane;
#pragma unroll
                for (int c = 0; c < NC; ++c) o[c] = __builtin_fmaf(pj, vr[64 * c], o[c]);
            }
            m = m_new;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
    // no key at all: zeros; only keys whose score is -inf: NaN
    const float inv = lsum > 0.f ? 1.f / lsum : some ? NAN : 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) O[(int64_t)h * os_h + i * os_l + lane + 64 * c] = o[c] * inv;
}

// A wave per row is the faster one for row blocks of one row whatever the budget, of 2 up to about 100 keys (95 us
// against 185 us with 16 keys, 408 against 344 us with 128; L = 6000, 8 heads, D = 64), of 3 up to 40, of 4 up to 25
// (D = 128: 136 against 189 us with 16 keys, 614 against 329 us with 128): B_r^2 N_b of about 400
static bool f32_by_rows(const Prob &p) { return p.B_r == 1 || (p.B_r > 0 && (int64_t)p.B_r * p.B_r * p.N_b <= 400); }
// workgroups of 32 rows
static int64_t f32_wg32(const Prob &p, const int32_t *T_cls) {
    return (int64_t)p.H_q * (4 * (int64_t)T_cls[0] + 3 * (int64_t)T_cls[1] + 2 * (int64_t)T_cls[2] + T_cls[3]);
}

// Every 16 rows repeat their group's routing, so few of them only; less so at D = 128, whose products for the scores are
// twice as many.  A call in us, three launches -> two: D = 64, 4 heads of 51 chunks of 40 tokens (408 workgroups of 32 rows) 26.5 ->
// 25.7, 8 heads of 26 chunks (416) 21.1 -> 19.6; D = 128, 4 heads of 26 chunks (208) 24.2 -> 22.5, 8 heads (416) 36.4 -> 37.0, 4
// heads in row blocks of 128 (256) 30.7 -> 29.1.
bool f32_route_attend_ok(const Prob &p, const int32_t *T_cls) {
    const int64_t wg32 = f32_wg32(p, T_cls);
    return !f32_by_rows(p) && wg32 < 512 && wg32 * p.D <= 256 * 128;
}

hipError_t launch_f32_route_attend(const Prob &p, const PlanLayout &pl, const PlanView &pv, const double *Qc, const double *Kc,
                                   double *Sc, int32_t *plan, const void *Q, const void *K, const void *V, void *O, hipStream_t s) {
    const F32RouteArgs route = {{plan, pl, p.N_c, p.N_b, p.B_r, 0, p.N_q, 0, p.H_q * p.N_q, 0, 0}, Qc, Kc, Sc};
#define DHSA_F32_ROUTE(DD)                                                                                                        \
    hipLaunchKernelGGL((k_attn_f32<DD, 1, F32RouteArgs>), dim3((unsigned)(2 * f32_wg32(p, pl.T_cls))), dim3(256), 0, s, pv, route, \
                       (const float *)Q, (const float *)K, (const float *)V, (float *)O, 0u, p.H_q, p.G,                          \
                       p.scale * 1.4426950408889634f, p.qs_h, p.qs_l, p.ks_h, p.ks_l, p.vs_h, p.vs_l, p.os_h, p.os_l)
    if (p.D == 64) DHSA_F32_ROUTE(64); else DHSA_F32_ROUTE(128);
#undef DHSA_F32_ROUTE
    return hipGetLastError();
}

hipError_t launch_attn_f32(const Prob &p, const PlanView &pv, const void *Q, const void *K, const void *V, void *O,
                           hipStream_t s) {
    if (f32_by_rows(p)) {
        const dim3 grid((unsigned)((p.L + 3) / 4), p.H_q);      // at most 2^20 row blocks: fewer than 2^32 threads
#define DHSA_F32_ROWS(DD)                                                                                      \
    hipLaunchKernelGGL(k_attn_f32_rows<DD>, grid, dim3(256), 0, s, pv, (const float *)Q, (const float *)K,     \
                       (const float *)V, (float *)O, p.L, p.G, p.B_r, p.scale * 1.4426950408889634f, p.qs_h,   \
                       p.qs_l, p.ks_h, p.ks_l, p.vs_h, p.vs_l, p.os_h, p.os_l)
        if (p.D == 64) DHSA_F32_ROWS(64); else DHSA_F32_ROWS(128);
#undef DHSA_F32_ROWS
        return hipGetLastError();
    }
    // 32 rows per workgroup read K and V half as often as 16; while that leaves CUs with fewer than two
    // workgroups, 16-row ones fill the chip better and waste less on the last rows of a tile
    const int64_t wg32 = f32_wg32(p, pv.T_cls);
    const bool small = wg32 < 512;
    const int64_t n_wg = small ? 2 * wg32 : wg32;
    const dim3 block(256);
#define DHSA_F32_ATTN(DD, RW)                                                                                 \
    hipLaunchKernelGGL((k_attn_f32<DD, RW, NoRoute>), grid, block, 0, s, pv, NoRoute{}, (const float *)Q, (const float *)K,       \
                       (const float *)V, (float *)O, block0, p.H_q, p.G, p.scale * 1.4426950408889634f, p.qs_h, p.qs_l, \
                       p.ks_h, p.ks_l, p.vs_h, p.vs_l, p.os_h, p.os_l)
    for (int64_t first = 0; first < n_wg; first += kGridMax) {
        const unsigned block0 = (unsigned)first;
        const dim3 grid((unsigned)std::min<int64_t>(kGridMax, n_wg - first));
        if (p.D == 64) {
            if (small) DHSA_F32_ATTN(64, 1); else DHSA_F32_ATTN(64, 2);
        } else {
            if (small) DHSA_F32_ATTN(128, 1); else DHSA_F32_ATTN(128, 2);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#undef DHSA_F32_ATTN
    return hipSuccess;
}

}  // namespace dhsa
