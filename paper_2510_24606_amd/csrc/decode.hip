// One decoding step of libdhsa (Sec. 3.4, the remark on decoding: the same sparse
// attention applied to each newly generated token by restricting the keys it
// attends).  The newest token is row i = L - 1 of a sequence whose K / V rows are
// cached; its key set is what the prefill path gives that row: its query group
// (the open chunk, or with B_r > 0 the open row block) is pooled, scored against
// every key chunk, ranked and walked with the budget N_b (Alg. 1), and the row
// attends to the selected keys (Alg. 2).
//
// Kernels of this file:
//   k_pool_decode     pooled keys (Eq. 4) of the chunks not pooled by an earlier
//                     step, pooled queries of the open group;
//   k_scores_decode   that group's scores against every key chunk (fp64 MFMA, heads of a kv-group as rows);
//   (the ranking and the walk are k_select of route.hip, launched for one group; with few chunks all of the routing
//   and often the step is k_decode_few)
//   k_attn_decode     the selected keys are split into slices; one workgroup
//                     per (slice, head) streams its K and V rows once, 16 bytes per
//                     lane, several rows in flight, and keeps an online-softmax
//                     state per row group; memory bound.  Where the slices are few, the workgroup
//                     that finishes a head's last one merges their states into the output row, else
//   k_decode_combine  does that.
// Around the stream of K and V a step is a chain of launches, each of which waits for the one before, so
// each is made short: fewer of them, everything requested at once.
#include <algorithm>

#include "select.h"

namespace dhsa {

// ---------------------------------------------------------------------------
// Pooling.  grid (max(N_c - kc_valid, 1), H_kv + H_q): y < H_kv pools key chunk
// kc_valid + x of kv-head y into Kc [H_kv][N_c_cap][D]; y >= H_kv (x = 0 only)
// pools the rows [rb0, L) of query head y - H_kv into Qc [H_q][D].  Same row
// traversal as the prefill pooling kernel.
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(256) void k_pool_decode(const T *__restrict__ Q, const T *__restrict__ K,
                                                     int32_t *__restrict__ B, BoundaryTail tail,
                                                     int32_t *__restrict__ RBw, int32_t *__restrict__ done,
                                                     double *__restrict__ Qc, double *__restrict__ Kc, int H_kv,
                                                     int N_c, int N_c_cap, int kc_valid, int rb0, int L, int B_r,
                                                     int pooling, int64_t qs_h, int64_t qs_l, int64_t ks_h,
                                                     int64_t ks_l) {
    constexpr int EPT = Elem<T>::kPer16;   // elements per thread per row
    constexpr int TPR = D / EPT;           // threads per row
    constexpr int RG = 256 / TPR;          // rows in flight
    __shared__ double s_sum[RG][D];
    const int tid = threadIdx.x;
    const bool is_q = (int)blockIdx.y >= H_kv;
    const T *X;
    double *Xc;
    int64_t s_l;
    int b0, b1;
    if (is_q) {
        if (blockIdx.x != 0) return;
        const int h = blockIdx.y - H_kv;
        X = Q + (int64_t)h * qs_h; s_l = qs_l; Xc = Qc + (int64_t)h * D;
        b0 = rb0; b1 = L;
        if (h == 0 && tid == 0) { RBw[0] = rb0; RBw[1] = L; }   // the one query group of the step's plan
        if (tid == 0) done[h] = 0;       // slices of the head finished so far (k_attn_decode)
        // boundaries that came as arguments go into the workspace for the kernels after this one
        if (h == 0 && tid <= tail.n && tail.n > 0) B[kc_valid + tid] = tail.b[tid];
    } else {
        const int k = kc_valid + blockIdx.x, g = blockIdx.y;
        if (k >= N_c) return;
        X = K + (int64_t)g * ks_h; s_l = ks_l; Xc = Kc + ((int64_t)g * N_c_cap + k) * D;
        if (tail.n > 0) { b0 = tail.b[blockIdx.x]; b1 = tail.b[blockIdx.x + 1]; }   // not yet in B (see below)
        else { b0 = B[k]; b1 = B[k + 1]; }
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
        Xc[tid] = pooling == DHSA_POOL_MEAN ? sum / len                                  // plain average (ablation)
                  : (is_q && B_r > 0)      ? sqrt((double)B_r) * (sum / len)            // Alg. 1 row blocks
                                           : (sqrt(len) / len) * sum;                   // Eq. 4
    }
}

// ---------------------------------------------------------------------------
// Scores of the open query group: Sc[h][k] = <Qc[h], Kc[h / G][k]>, k < N_c: the 16 x 16 block of a wave has
// up to 16 heads of a kv-group as rows and 16 chunks as columns, with the operand layout and the order of
// summation of the prefill's scores.  All of D is requested at once.  grid (ceil(N_c / 64), H_kv, ceil(G / 16)).
// 1634 chunks x 8 kv-heads of D = 128: 12 us with a wave per chunk and a sum over its lanes per head.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void k_scores_decode(const double *__restrict__ Qc, const double *__restrict__ Kc,
                                                       double *__restrict__ Sc, int N_c, int N_c_cap, int G) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k0 = blockIdx.x * 64 + wave * 16, g = blockIdx.y, h0 = blockIdx.z * 16;
    if (k0 >= N_c) return;
    const int n16 = lane & 15, q = lane >> 4;
    const double *A = Qc + (int64_t)(g * G + (h0 + n16 < G ? h0 + n16 : G - 1)) * D + 2 * q;
    const double *B = Kc + ((int64_t)g * N_c_cap + (k0 + n16 < N_c ? k0 + n16 : N_c - 1)) * D + 2 * q;
    f64x2 a[D / 8], b[D / 8];
#pragma unroll
    for (int s = 0; s < D / 8; ++s) {
        b[s] = *reinterpret_cast<const f64x2 *>(B + 8 * s);
        a[s] = *reinterpret_cast<const f64x2 *>(A + 8 * s);
    }
    __builtin_amdgcn_sched_barrier(0);   // left alone, the scheduler moves the loads next to their use
    f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < D / 8; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][j], b[s][j], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int hh = h0 + 4 * v + q, k = k0 + n16;
        if (hh < G && k < N_c) Sc[(int64_t)(g * G + hh) * N_c + k] = acc[v];
    }
}

// ---------------------------------------------------------------------------
// Attention of the newest row over slice blockIdx.x of its selected keys.
// The plan entries of (h, the open group) are walked like in the prefill
// kernels (ascending key position); packed positions [slice s, slice (s + 1)) are
// this workgroup's.  A key row is read by TPR = D sizeof(T) / 16 adjacent lanes
// (16 bytes each: coalesced), NG = 256 / TPR rows at a time, U batches in
// flight.
// FUSE: the state of a slice (m, l, o[D]) goes to memory with stores that bypass the XCD's own L2 (agent
// scope), waited for, before the workgroup counts itself as done with an atomic of that scope; the one that
// counts last reads all states of its head the same way and writes the output row.  Nothing
// else has to become visible, so no workgroup writes back its L2 (a release fence before the count did
// that: 150 us a step).  That saves a launch where the chip is nearly empty (a head of 512 keys: 10.9 + 3.8 us
// -> 8 us); where it is full, workgroups that wait for their stores hold up those behind them (64 slices x 32 heads:
// 41 us against 28 + 6 us), so the states are merged by k_decode_combine.
// ---------------------------------------------------------------------------
template <typename T> struct DecIO;
template <> struct DecIO<float> {
    __device__ static void unpack(const uint4 &u, float *x) {
        x[0] = __uint_as_float(u.x); x[1] = __uint_as_float(u.y);
        x[2] = __uint_as_float(u.z); x[3] = __uint_as_float(u.w);
    }
    __device__ static void store(float *p, float x) { *p = x; }
};
template <> struct DecIO<bf16_t> {
    __device__ static void unpack(const uint4 &u, float *x) {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = __uint_as_float(w[i] << 16);
            x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ static void store(bf16_t *p, float x) {   // round to nearest even
        uint32_t u = __float_as_uint(x);
        u += 0x7fffu + ((u >> 16) & 1u);
        p->bits = (uint16_t)(u >> 16);
    }
};

// Merge of the S slice states of one head into its output row by NTHR threads: thread = (two columns, every NSG-th
// slice), eight slices requested at a time.  AGENT: the states may have been written by workgroups of the same
// launch.  s_m, s_l, s_o: room for NSG partial states.
template <typename T, int D, int NTHR, bool AGENT>
__device__ __forceinline__ void merge_slices(const float *part, int S, float *s_m, float *s_l, float (*s_o)[D], T *O) {
    constexpr int NSG = NTHR / (D / 2);
    const int tid = threadIdx.x, c2 = tid % (D / 2), sg = tid / (D / 2);
    const unsigned long long *p64 = reinterpret_cast<const unsigned long long *>(part);
    const auto get = [](const unsigned long long *p) {
        if constexpr (AGENT) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else return *p;
    };
    float Mr = -INFINITY, lr = 0.f, o0 = 0.f, o1 = 0.f;
    for (int s0 = sg; s0 < S; s0 += 8 * NSG) {
        unsigned long long ml[8], ov[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const unsigned long long *ps = p64 + (int64_t)(s0 + u * NSG < S ? s0 + u * NSG : s0) * (D / 2 + 1);
            ml[u] = get(&ps[0]);
            ov[u] = get(&ps[1 + c2]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (s0 + u * NSG >= S) break;
            const float mu = __uint_as_float((unsigned)ml[u]);
            const float m_new = fmaxf(Mr, mu);
            const float a0 = (Mr == -INFINITY) ? 0.f : __expf(Mr - m_new), a1 = (mu == -INFINITY) ? 0.f : __expf(mu - m_new);
            lr = lr * a0 + __uint_as_float((unsigned)(ml[u] >> 32)) * a1;
            o0 = o0 * a0 + __uint_as_float((unsigned)ov[u]) * a1;
            o1 = o1 * a0 + __uint_as_float((unsigned)(ov[u] >> 32)) * a1;
            Mr = m_new;
        }
    }
    if (c2 == 0) { s_m[sg] = Mr; s_l[sg] = lr; }
    s_o[sg][2 * c2] = o0;
    s_o[sg][2 * c2 + 1] = o1;
    __syncthreads();
    if (tid < D) {
        float M = -INFINITY;
#pragma unroll
        for (int x = 0; x < NSG; ++x) M = fmaxf(M, s_m[x]);
        float ls = 0.f, acc = 0.f;
#pragma unroll
        for (int x = 0; x < NSG; ++x) {
            const float w = (s_m[x] == -INFINITY) ? 0.f : __expf(s_m[x] - M);
            ls += s_l[x] * w;
            acc += s_o[x][tid] * w;
        }
        DecIO<T>::store(O + tid, ls > 0.f ? acc / ls : 0.f);
    }
}

constexpr int kDecOwn = 8;   // keys of a chunk that a thread writes into the list of its slice by itself

template <typename T>
struct AttendArgs {
    const T *Q, *K, *V;
    T *O_row;
    float *part;
    int32_t *done, *idx, *cnt;
    int S, slice, stride, rb0, L, cap, G;
    float scale;
    int64_t qs_h, qs_l, ks_h, ks_l, vs_h, vs_l;
};

template <typename T, int D>
struct AttendSmem {
    static constexpr int EPT = 16 / (int)sizeof(T);   // elements per 16 bytes
    static constexpr int TPR = D / EPT;               // lanes per key row (8, 16 or 32)
    static constexpr int NG = 256 / TPR;              // key rows per batch
    int keys[kDecSliceMax];
    int4 seg[kDecSliceMax / (kDecOwn + 1) + 1];       // long pieces of chunks: first and last position in the slice, key - position
    int nseg;
    int wave[8];
    float m[NG], l[NG];
    float o[NG][D];
    int last;
};

// Slice s of head h by the first 256 threads of a workgroup of NTHR, over the plan entries ent[0 .. *count) and the
// boundaries B, in memory or LDS.
template <typename T, int D, bool FUSE, int NTHR>
__device__ __forceinline__ void attend_slice(AttendSmem<T, D> &sm, const AttendArgs<T> &a, int s, int h, const int2 *ent,
                                             const int32_t *count, const int32_t *B) {
    using Smem = AttendSmem<T, D>;
    constexpr int EPT = Smem::EPT, TPR = Smem::TPR, NG = Smem::NG;
    constexpr int U = 4;                       // batches in flight
    const int g = h / a.G, tid = threadIdx.x, slice = a.slice;
    const int i = a.L - 1;
    const int v = a.L - a.rb0;   // rows of the query group up to and including the newest
    const bool on = NTHR == 256 || tid < 256;
    const int gi = tid / TPR, r = tid % TPR;
    // the first batch of entries does not wait for their number
    int2 ent_e = ent[on && tid < a.stride ? tid : 0];
    const int E = *count;
    if (!on || tid >= E) ent_e = int2{0, 0};   // past the list: nothing there has been written
    int b0 = B[ent_e.x & kChunkMask], b1 = B[(ent_e.x & kChunkMask) + 1];
    const uint4 q16 = *reinterpret_cast<const uint4 *>(a.Q + (int64_t)h * a.qs_h + (int64_t)i * a.qs_l + r * EPT);
    const int x_lo = s * slice, x_hi = x_lo + slice;

    if (tid == 0) sm.nseg = 0;   // (the scan has barriers)
    int base = 0;   // selected keys of the entries walked so far (block-uniform)
    for (int e0 = 0; e0 < E; e0 += 256) {
        if (e0 > 0) {
            ent_e = on && e0 + tid < E ? ent[e0 + tid] : int2{0, 0};
            b0 = B[ent_e.x & kChunkMask];
            b1 = B[(ent_e.x & kChunkMask) + 1];
        }
        int take = 0;
        if (on && e0 + tid < E) {
            const int pos = ent_e.x >> kPosShift;
            take = entry_take(pos, ent_e.y, b1 - b0, v);
            if (pos == 3) {   // row-block form: of the block's list, the keys up to the row itself
                const int vis = i + 1 - b0;
                if (vis < take) take = vis > 0 ? vis : 0;
            }
        }
        int total;
        const int start = base + block_excl_scan(take, sm.wave, &total);   // (waves past the fourth add nothing)
        const int lo = start > x_lo ? start : x_lo;
        const int hi = start + take < x_hi ? start + take : x_hi;
        // a thread writes few keys by itself; a long piece (a slice holds a handful of them) is written by a wave
        if (hi - lo <= kDecOwn) {
            for (int x = lo; x < hi; ++x) sm.keys[x - x_lo] = b0 + (x - start);
        } else if (on) {
            sm.seg[atomicAdd(&sm.nseg, 1)] = make_int4(lo - x_lo, hi - x_lo, b0 - start + x_lo, 0);
        }
        __syncthreads();
        for (int sg = tid >> 6, n_seg = sm.nseg; sg < n_seg; sg += NTHR / 64) {
            const int4 w = sm.seg[sg];
            for (int x = w.x + (tid & 63); x < w.y; x += 64) sm.keys[x] = x + w.z;
        }
        base += total;
        if (base >= x_hi && s != 0) break;   // slice 0 walks on: it reports the row's key count
        __syncthreads();
        if (tid == 0) sm.nseg = 0;
    }
    __syncthreads();
    if (s == 0 && tid == 0 && a.cnt) a.cnt[h] = base;
    int n_mine = base - x_lo;
    n_mine = n_mine < 0 ? 0 : (n_mine > slice ? slice : n_mine);
    if (a.idx)
        for (int x = tid; x < slice && x_lo + x < a.cap; x += NTHR) a.idx[(int64_t)h * a.cap + x_lo + x] = x < n_mine ? sm.keys[x] : -1;

    if (on) {
        float q[EPT];
        DecIO<T>::unpack(q16, q);
        const T *Kg = a.K + (int64_t)g * a.ks_h + r * EPT;
        const T *Vg = a.V + (int64_t)g * a.vs_h + r * EPT;
        float m = -INFINITY, l = 0.f, o[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) o[e] = 0.f;
        for (int j0 = gi; j0 < n_mine; j0 += NG * U) {
            uint4 kf[U], vf[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int jj = j0 + u * NG;
                ok[u] = jj < n_mine;
                const int key = ok[u] ? sm.keys[jj] : sm.keys[j0];   // a valid row either way
                kf[u] = *reinterpret_cast<const uint4 *>(Kg + (int64_t)key * a.ks_l);
                vf[u] = *reinterpret_cast<const uint4 *>(Vg + (int64_t)key * a.vs_l);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float kx[EPT], vx[EPT];
                DecIO<T>::unpack(kf[u], kx);
                DecIO<T>::unpack(vf[u], vx);
                float d = 0.f;
#pragma unroll
                for (int e = 0; e < EPT; ++e) d += q[e] * kx[e];
#pragma unroll
                for (int off = TPR / 2; off > 0; off >>= 1) d += __shfl_xor(d, off);
                if (ok[u]) {
                    const float sc = d * a.scale;
                    const float m_new = fmaxf(m, sc);
                    const float alpha = __expf(m - m_new), p = __expf(sc - m_new);
                    l = l * alpha + p;
#pragma unroll
                    for (int e = 0; e < EPT; ++e) o[e] = o[e] * alpha + p * vx[e];
                    m = m_new;
                }
            }
        }
        if (r == 0) { sm.m[gi] = m; sm.l[gi] = l; }
#pragma unroll
        for (int e = 0; e < EPT; ++e) sm.o[gi][r * EPT + e] = o[e];
    }
    __syncthreads();
    if (tid < D) {
        float M = -INFINITY;
        for (int x = 0; x < NG; ++x) M = fmaxf(M, sm.m[x]);
        float ls = 0.f, acc = 0.f;
        for (int x = 0; x < NG; ++x) {
            const float w = (sm.m[x] == -INFINITY) ? 0.f : __expf(sm.m[x] - M);
            ls += sm.l[x] * w;
            acc += sm.o[x][tid] * w;
        }
        float *pp = a.part + ((int64_t)h * a.S + s) * (D + 2);
        const auto put = [](float *p, float x) {
            if constexpr (FUSE) __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *p = x;
        };
        put(&pp[2 + tid], acc);
        if (tid == 0) { put(&pp[0], M); put(&pp[1], ls); }
    }
    if constexpr (!FUSE) return;
    // The count below is relaxed, so by the memory model alone it orders nothing.  What it rests on is gfx950: a store of
    // agent scope is written through the XCD's L2, and vmcnt counts it until the memory side has acknowledged it.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // the compiler's order, and
    __builtin_amdgcn_s_waitcnt(0x0f70);                      // vmcnt(0): the stores have reached the memory side
    __syncthreads();
    if (tid == 0) {
        sm.last = __hip_atomic_fetch_add(&a.done[h], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.S - 1;
        if (sm.last) __hip_atomic_store(&a.done[h], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next step
    }
    __syncthreads();
    if (!sm.last || !on) return;
    merge_slices<T, D, 256, true>(a.part + (int64_t)h * a.S * (D + 2), a.S, sm.m, sm.l, sm.o, a.O_row + (int64_t)h * D);
}

template <typename T, int D, bool FUSE>
__global__ __launch_bounds__(256) void k_attn_decode(const int32_t *__restrict__ B, const int32_t *__restrict__ count,
                                                     const int2 *__restrict__ entries, AttendArgs<T> a) {
    __shared__ AttendSmem<T, D> sm;
    const int s = blockIdx.x, h = blockIdx.y;
    attend_slice<T, D, FUSE, 256>(sm, a, s, h, entries + (int64_t)h * a.stride, count + h, B);
}

// ---------------------------------------------------------------------------
// A step over few chunks by workgroups of eight waves.  Each does the whole routing of its head: the open group's queries and
// the new key chunks are pooled (the first four waves and the others side by side, in k_pool_decode's order), then scored and
// ranked.  The heads of a kv-group pool the same key chunks; the first workgroup of the first of them stores them for later
// steps.  Boundaries and pooled keys that come with the step are taken from LDS, the others from the workspace.
// ONE: a workgroup per slice goes on with the attention of it, over a list that never leaves LDS: the step is one launch.
// Else a workgroup per head leaves the plan to k_attn_decode.
// ---------------------------------------------------------------------------
constexpr int kDecodeFewChunks = 128;
constexpr int kDecodeFewNew = 3;     // key chunks to pool: with the group's queries two rounds of the workgroup's halves

template <typename T, int D, bool ONE>
__global__ __launch_bounds__(512, 2) void k_decode_few(AttendArgs<T> at, SelectArgs a, BoundaryTail tail, double *__restrict__ Kc,
                                                       int N_c_cap, int kc_valid, int pooling) {
    constexpr int EPT = Elem<T>::kPer16, TPR = D / EPT, RG = 256 / TPR;   // as in k_pool_decode
    __shared__ double s_sum[2][RG][D];
    __shared__ __align__(16) double s_pool[1 + kDecodeFewNew][D];       // the queries, then the new chunks
    __shared__ double s_row[kDecodeFewChunks];
    __shared__ int32_t s_B[kDecodeFewChunks + 1];
    __shared__ FewSmem<512, kDecodeFewChunks> s_few;
    __shared__ int2 s_ent[kDecodeFewChunks];
    __shared__ int s_count;
    __shared__ AttendSmem<T, D> sm;
    const int h = blockIdx.y, g = h / at.G, rb0 = at.rb0, L = at.L, tid = threadIdx.x;
    const bool first = !ONE || blockIdx.x == 0;             // of the head's workgroups
    const int half = __builtin_amdgcn_readfirstlane(tid >> 8), th = tid & 255;
    // 16 chunks for each wave: their pooled keys are requested before anything is pooled
    const int lane = tid & 63, k = (tid >> 6) * 16 + (lane & 15), k_c = k < a.N_c ? k : a.N_c - 1;
    f64x2 key[D / 8];
    load_pooled<D>(key, Kc + ((int64_t)g * N_c_cap + (k_c < kc_valid ? k_c : kc_valid - 1)) * D);
    int32_t *B = a.plan + a.pl.off_B;
    if (tid < kc_valid) s_B[tid] = B[tid];
#pragma unroll
    for (int j = 0; j <= kDecodeFewNew; ++j)                // (from scalar registers: kernel arguments are far from the vector unit)
        if (tid == 64 * j && j <= tail.n) {
            s_B[kc_valid + j] = tail.b[j];
            if (first && h == 0) B[kc_valid + j] = tail.b[j];   // for later steps and launches
        }
    const int rg = th / TPR, col = (th % TPR) * EPT;
    for (int x0 = 0; x0 <= tail.n; x0 += 2) {
        const int x = x0 + half;
        const bool is_q = x == 0;
        const T *X = is_q ? at.Q + (int64_t)h * at.qs_h : at.K + (int64_t)g * at.ks_h;
        const int64_t s_l = is_q ? at.qs_l : at.ks_l;
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
            if (!is_q && first && h == g * at.G) Kc[((int64_t)g * N_c_cap + kc_valid + x - 1) * D + th] = pooled;
        }
    }
    __syncthreads();
    if (k - (lane & 15) < a.N_c) {
        if (k_c >= kc_valid) load_pooled<D>(key, s_pool[1 + k_c - kc_valid]);
        f64x2 q[D / 8];
        load_pooled<D>(q, s_pool[0]);
        const double score = score_16<D>(q, key);
        if (lane < 16 && k < a.N_c) s_row[k] = score;
    }
    __syncthreads();
    const Visible vis = {a.B_r > 0 ? -1 : a.N_c - 1, L, a.N_c};   // the last group sees all chunks
    int2 *entries = ONE ? s_ent : reinterpret_cast<int2 *>(a.plan + a.pl.off_entries) + (int64_t)h * a.pl.stride;
    const int n = select_few<512, kDecodeFewChunks>(a, s_row, s_B, vis, s_few,
                                                    [&](int i, int w, int rem) { entries[i] = make_int2(w, rem); });
    if constexpr (ONE) {
        if (tid == 0) s_count = n;
        __syncthreads();
        attend_slice<T, D, true, 512>(sm, at, blockIdx.x, h, s_ent, &s_count, s_B);
    } else if (tid == 0) {
        a.plan[a.pl.off_count + h] = n;
    }
}

// grid H_q
template <typename T, int D>
__global__ __launch_bounds__(512) void k_decode_combine(const float *__restrict__ part, int S, T *__restrict__ O_row) {
    constexpr int NSG = 512 / (D / 2);
    __shared__ float s_m[NSG], s_l[NSG];
    __shared__ float s_o[NSG][D];
    const int h = blockIdx.x;
    merge_slices<T, D, 512, false>(part + (int64_t)h * S * (D + 2), S, s_m, s_l, s_o, O_row + (int64_t)h * D);
}

// Few chunks: one launch instead of three before the attention, or of four.  A step in us, launches apart -> this: 8 heads of 38
// chunks 18.9 -> 13.0, with two and three chunks to pool 19.2 -> 14.7 and 15.0, of 128 chunks 19.5 -> 17.4, 19.8 -> 18.9 and
// 19.2, of 16 chunks of 500 tokens 19.8 -> 13.9; 32 heads of 128 chunks, 512 keys 20.0 -> 17.7, 2048 keys (slices too many to be
// routed one by one) 23.8 -> 23.1, with two chunks to pool 24.3 -> 25.2; 64 heads of 16 chunks of 500 tokens 28.6 -> 25.8, with two
// and three to pool 33.5 -> 36.8 and 41.9: every head pools the chunks of its kv-head, one after the other.
static bool decode_few(const Prob &p, int rb0, const BoundaryTail &tail, bool fuse) {
    int64_t longest = p.L - rb0;
    for (int j = 0; j < tail.n; ++j) longest = std::max<int64_t>(longest, tail.b[j + 1] - tail.b[j]);
    if (p.N_c > kDecodeFewChunks || tail.n < 1 || tail.n > kDecodeFewNew) return false;
    return tail.n == 1 ? longest <= 512 : fuse && longest <= 128;
}

hipError_t launch_decode_step(const Prob &p, const DecodeLayout &dl, int N_c_cap, int kc_valid, int rb0, const BoundaryTail &tail,
                              const void *Q, const void *K, const void *V, void *ws, void *O_row, int32_t *idx, int32_t *cnt,
                              hipStream_t s) {
    char *w8 = static_cast<char *>(ws);
    double *Kc = reinterpret_cast<double *>(w8 + dl.off_Kc), *Qc = reinterpret_cast<double *>(w8 + dl.off_Qc);
    double *Sc = reinterpret_cast<double *>(w8 + dl.off_Sc);
    int32_t *plan = reinterpret_cast<int32_t *>(w8 + dl.off_plan), *done = reinterpret_cast<int32_t *>(w8 + dl.off_done);
    float *part = reinterpret_cast<float *>(w8 + dl.off_part);
    const int slice = decode_slice(p.H_q, p.N_b);
    const int S = (p.N_b + slice - 1) / slice;           // N_b is clamped to L: the row takes exactly N_b keys
    const bool fuse = slice < kDecSlice, few = decode_few(p, rb0, tail, fuse);
#define DHSA_TYPES(CALL)                                                                       \
    do {                                                                                       \
        if (p.dtype == DHSA_F32) {                                                             \
            if (p.D == 64) CALL(float, 64); else CALL(float, 128);                             \
        } else {                                                                               \
            if (p.D == 64) CALL(bf16_t, 64); else CALL(bf16_t, 128);                           \
        }                                                                                      \
        if ((e = hipGetLastError()) != hipSuccess) return e;                                   \
    } while (0)
#define DHSA_ARGS(T)                                                                                                              \
    AttendArgs<T>{(const T *)Q, (const T *)K, (const T *)V, (T *)O_row, part, done, idx, cnt, S, slice, dl.pl.stride, rb0,         \
                  (int)p.L, p.N_b, p.G, p.scale, p.qs_h, p.qs_l, p.ks_h, p.ks_l, p.vs_h, p.vs_l}
    hipError_t e;
    if (few) {
        const SelectArgs a = {plan, dl.pl, p.N_c, p.N_b, p.B_r, p.N_q - 1, 1, 0, p.H_q, 0, 0};
#define DHSA_FEW1(T, DD, ONE)                                                                                                 \
    hipLaunchKernelGGL((k_decode_few<T, DD, ONE>), dim3(ONE ? S : 1, p.H_q), dim3(512), 0, s, DHSA_ARGS(T), a, tail, Kc, \
                       N_c_cap, kc_valid, p.pooling)
#define DHSA_FEW(T, DD) do { if (fuse) DHSA_FEW1(T, DD, true); else DHSA_FEW1(T, DD, false); } while (0)
        DHSA_TYPES(DHSA_FEW);
#undef DHSA_FEW
#undef DHSA_FEW1
        if (fuse) return hipSuccess;
    } else {
        const int n_new = p.N_c - kc_valid;
        const dim3 grid(n_new > 1 ? n_new : 1, p.H_kv + p.H_q), block(256);
#define DHSA_POOLD(T, DD)                                                                                      \
    hipLaunchKernelGGL((k_pool_decode<T, DD>), grid, block, 0, s, (const T *)Q, (const T *)K,                  \
                       plan + dl.pl.off_B, tail, plan + dl.pl.off_RB, done, Qc, Kc, p.H_kv, p.N_c, N_c_cap, kc_valid, rb0, \
                       (int)p.L, p.B_r, p.pooling, p.qs_h, p.qs_l, p.ks_h, p.ks_l)
        DHSA_TYPES(DHSA_POOLD);
#undef DHSA_POOLD
        const dim3 sgrid((p.N_c + 63) / 64, p.H_kv, (p.G + 15) / 16);
        if (p.D == 64)
            hipLaunchKernelGGL(k_scores_decode<64>, sgrid, dim3(256), 0, s, Qc, Kc, Sc, p.N_c, N_c_cap, p.G);
        else
            hipLaunchKernelGGL(k_scores_decode<128>, sgrid, dim3(256), 0, s, Qc, Kc, Sc, p.N_c, N_c_cap, p.G);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        // ranking + walk of the one open group: group number N_q - 1 of the sequence, group 0 of this plan
        if ((e = launch_select_groups(p, dl.pl, Sc, plan, p.N_q - 1, 1, s)) != hipSuccess) return e;
    }
#define DHSA_ATTD1(T, DD, FUSE)                                                                                           \
    hipLaunchKernelGGL((k_attn_decode<T, DD, FUSE>), dim3(S, p.H_q), dim3(256), 0, s, plan + dl.pl.off_B, plan + dl.pl.off_count, \
                       (const int2 *)(plan + dl.pl.off_entries), DHSA_ARGS(T))
#define DHSA_ATTD(T, DD) do { if (fuse) DHSA_ATTD1(T, DD, true); else DHSA_ATTD1(T, DD, false); } while (0)
    DHSA_TYPES(DHSA_ATTD);
#undef DHSA_ATTD
#undef DHSA_ATTD1
#define DHSA_COMB(T, DD) hipLaunchKernelGGL((k_decode_combine<T, DD>), dim3(p.H_q), dim3(512), 0, s, part, S, (T *)O_row)
    if (!fuse) DHSA_TYPES(DHSA_COMB);
#undef DHSA_COMB
#undef DHSA_ARGS
#undef DHSA_TYPES
    return hipSuccess;
}

}  // namespace dhsa
