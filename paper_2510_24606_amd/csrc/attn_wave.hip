// bf16 MFMA sparse attention, one wave per SIMD (same algorithm as attn_mfma.hip, which describes the key lists, the masks
// and the exponent reference).  A tile gets the bits that attn_mfma.hip gives it, whichever of the two takes it: the
// products, sums and references of a row are made from the same numbers in the same order.
//
// A wave owns ALL rows of a tile of 33..64 or 65..96 rows (RB = 2, 3 blocks of 32), or one half of a tile of 97..128
// rows (RB = 2, two waves side by side), and walks the tile's whole key list.  It may use all 512 registers of a SIMD
// lane, so a K or V fragment that has been read from LDS serves all its row blocks (a third or half of the reads that
// four waves of one row block each need), and a tile of 65..96 rows leaves no wave without rows.  A wave that has a tile
// to itself has its own ring of K and V blocks in LDS, waits for its own loads only and meets no barrier; two waves of a
// tile fetch half of each block of a common ring and pass a barrier per block.
//
// What bounds a lone wave is its own instruction stream: a 32x32x16 product takes the matrix unit 32 cycles, of which
// issuing it takes 8; the rest holds six vector instructions (an exponential counts twice, an LDS read or a load three
// times).  So everything is laid out by hand beside the products: a phase is 8 products of scores of unit u + 1 and 8 of
// O += P V of unit u - 1 (a unit is one row block x 32 keys), with one exponential of unit u beside each, the reads of
// the next fragments, the loads and the key list of a later tile spread between them.  sched_barrier keeps the compiler
// from gathering them again.  Branches are decided a product before they are taken (a branch on a fresh comparison
// costs 44 cycles, one on an old one 8).
//
// Products are written as assembly so that O stays in fixed accumulation registers and scores in vector registers
// (the compiler moves whole accumulators between the two files otherwise).  The hardware does not wait for the result
// of a product: scores are used two products after their last one, O by the vector unit at least eight after.
//
// 131072 tokens, 32 heads, 8192 keys: tiles of more than 64 rows 17.4 -> 15.9 ms, of 33..64 rows 6.0 -> 5.8 ms, the call
// 24.7 -> 22.7 ms, with row blocks of 128 17.5 -> 16.3 ms.  The chip lowers its clock as the matrix units are busier (its
// power limit), so time falls by less than the cycles do.
#include "attn_mfma.h"

namespace dhsa {

constexpr int kWaveD = 128;   // head dimension

#if defined(__HIP_DEVICE_COMPILE__)
#define WAVE_ASM(...) asm volatile(__VA_ARGS__)
#else
#define WAVE_ASM(...)
#endif
#define WAVE_VMCNT(n) WAVE_ASM("s_waitcnt vmcnt(%0)" ::"i"(n) : "memory")

// O^T accumulators: group g = the 16 accumulation registers named below, in the text of every instruction that touches
// them, so that no value of the compiler ever stands for them.
#define WAVE_ACC_GROUPS(X) \
    X(0, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15) \
    X(1, 16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31) \
    X(2, 32, 33, 34, 35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47) \
    X(3, 48, 49, 50, 51, 52, 53, 54, 55, 56, 57, 58, 59, 60, 61, 62, 63) \
    X(4, 64, 65, 66, 67, 68, 69, 70, 71, 72, 73, 74, 75, 76, 77, 78, 79) \
    X(5, 80, 81, 82, 83, 84, 85, 86, 87, 88, 89, 90, 91, 92, 93, 94, 95) \
    X(6, 96, 97, 98, 99, 100, 101, 102, 103, 104, 105, 106, 107, 108, 109, 110, 111) \
    X(7, 112, 113, 114, 115, 116, 117, 118, 119, 120, 121, 122, 123, 124, 125, 126, 127) \
    X(8, 128, 129, 130, 131, 132, 133, 134, 135, 136, 137, 138, 139, 140, 141, 142, 143) \
    X(9, 144, 145, 146, 147, 148, 149, 150, 151, 152, 153, 154, 155, 156, 157, 158, 159) \
    X(10, 160, 161, 162, 163, 164, 165, 166, 167, 168, 169, 170, 171, 172, 173, 174, 175) \
    X(11, 176, 177, 178, 179, 180, 181, 182, 183, 184, 185, 186, 187, 188, 189, 190, 191) \
    X(12, 192, 193, 194, 195, 196, 197, 198, 199, 200, 201, 202, 203, 204, 205, 206, 207) \
    X(13, 208, 209, 210, 211, 212, 213, 214, 215, 216, 217, 218, 219, 220, 221, 222, 223) \
    X(14, 224, 225, 226, 227, 228, 229, 230, 231, 232, 233, 234, 235, 236, 237, 238, 239) \
    X(15, 240, 241, 242, 243, 244, 245, 246, 247, 248, 249, 250, 251, 252, 253, 254, 255)
#define WAVE_ACC_CLOBBER(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15) \
    "a" #r0, "a" #r1, "a" #r2, "a" #r3, "a" #r4, "a" #r5, "a" #r6, "a" #r7, "a" #r8, "a" #r9, "a" #r10, "a" #r11, "a" #r12, \
        "a" #r13, "a" #r14, "a" #r15

// O^T of group GR += V^T P^T
template <int GR, typename V, typename P>
__device__ __forceinline__ void acc_mfma(const V &v, const P &p) {
#define X(g, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                                                                                            \
    if constexpr (GR == g)                                                                                    \
        WAVE_ASM("v_mfma_f32_32x32x16_bf16 a[" #r0 ":" #r15 "], %0, %1, a[" #r0 ":" #r15 "]" ::"v"(v), "v"(p) \
                 : WAVE_ACC_CLOBBER(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15));
    WAVE_ACC_GROUPS(X)
#undef X
}
template <int GR>
__device__ __forceinline__ void acc_zero() {
#define WAVE_Z(r) "v_accvgpr_write_b32 a" #r ", 0\n\t"
#define X(g, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                                                                                             \
    if constexpr (GR == g)                                                                                     \
        WAVE_ASM(WAVE_Z(r0) WAVE_Z(r1) WAVE_Z(r2) WAVE_Z(r3) WAVE_Z(r4) WAVE_Z(r5) WAVE_Z(r6) WAVE_Z(r7)       \
                 WAVE_Z(r8) WAVE_Z(r9) WAVE_Z(r10) WAVE_Z(r11) WAVE_Z(r12) WAVE_Z(r13) WAVE_Z(r14) WAVE_Z(r15) \
                 ::: WAVE_ACC_CLOBBER(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15));
    WAVE_ACC_GROUPS(X)
#undef X
#undef WAVE_Z
}
template <int GR>
__device__ __forceinline__ void acc_scale(float f) {
    float t0, t1;
#define WAVE_S(a, b)                                                                                                    \
    "v_accvgpr_read_b32 %0, a" #a "\n\tv_accvgpr_read_b32 %1, a" #b "\n\tv_mul_f32 %0, %0, %2\n\tv_mul_f32 %1, %1, %2\n\t" \
    "v_accvgpr_write_b32 a" #a ", %0\n\tv_accvgpr_write_b32 a" #b ", %1\n\t"
#define X(g, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                                                                                            \
    if constexpr (GR == g)                                                                                    \
        WAVE_ASM(WAVE_S(r0, r1) WAVE_S(r2, r3) WAVE_S(r4, r5) WAVE_S(r6, r7) WAVE_S(r8, r9) WAVE_S(r10, r11)  \
                 WAVE_S(r12, r13) WAVE_S(r14, r15) : "=&v"(t0), "=&v"(t1) : "v"(f) : WAVE_ACC_CLOBBER(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15));
    WAVE_ACC_GROUPS(X)
#undef X
#undef WAVE_S
    (void)t0; (void)t1;
}
// registers 4 Q4 .. 4 Q4 + 3 of group GR
template <int GR, int Q4>
__device__ __forceinline__ void acc_read(float (&o)[4]) {
#define WAVE_R(a, b, c, d)                                                                                               \
    WAVE_ASM("v_accvgpr_read_b32 %0, a" #a "\n\tv_accvgpr_read_b32 %1, a" #b "\n\tv_accvgpr_read_b32 %2, a" #c            \
             "\n\tv_accvgpr_read_b32 %3, a" #d : "=v"(o[0]), "=v"(o[1]), "=v"(o[2]), "=v"(o[3]));
#define X(g, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                                               \
    if constexpr (GR == g && Q4 == 0) WAVE_R(r0, r1, r2, r3)     \
    if constexpr (GR == g && Q4 == 1) WAVE_R(r4, r5, r6, r7)     \
    if constexpr (GR == g && Q4 == 2) WAVE_R(r8, r9, r10, r11)   \
    if constexpr (GR == g && Q4 == 3) WAVE_R(r12, r13, r14, r15)
    WAVE_ACC_GROUPS(X)
#undef X
#undef WAVE_R
}

// S^T += K Q^T; the Q fragment lives in accumulation registers (QA) or vector registers
template <bool QA>
__device__ __forceinline__ void scores_mfma(f32x16 &s, const bf16x8 &k, const bf16x8 &q, bool first) {
    if (first) {
        if constexpr (QA) WAVE_ASM("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "a"(q));
        else WAVE_ASM("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "v"(q));
    } else {
        if constexpr (QA) WAVE_ASM("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "a"(q));
        else WAVE_ASM("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "v"(q));
    }
}

// 16 bytes per lane from global memory into LDS, load i of a group of up to four 1 KiB windows that lie behind one
// another; the first one sets M0 for all (nothing else uses it).  The instruction adds 1024 i to both addresses.
__device__ __forceinline__ void load_window(const char *base, unsigned off, unsigned lds_window, int i) {
    if (i == 0) WAVE_ASM("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_window) : "memory");
    if (i == 1) WAVE_ASM("global_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(off), "s"(base) : "memory");
    if (i == 2) WAVE_ASM("global_load_lds_dwordx4 %0, %1 offset:2048" ::"v"(off), "s"(base) : "memory");
    if (i == 3) WAVE_ASM("global_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(off), "s"(base) : "memory");
}
// one dword per lane
__device__ __forceinline__ void load_dwords(const void *base, unsigned off, unsigned lds_window) {
    WAVE_ASM("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds_window) : "memory");
}
__device__ __forceinline__ unsigned lds_address(const void *p) {
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)(const char *)p;
}

template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(Int<N - 1>());
    }
}

constexpr int kNoKey = 0x7fffffff;
constexpr int kListPart = 256;          // plan entries after which a list goes on with a new tile (attn_mfma.hip makes lists in such parts)
constexpr int kFirstTile = 256;         // flag of a list's first tile, beside the number of its keys that not every row takes
constexpr float kFar = 1048576.f;       // a sum of exponentials that moves the exponent reference (as in attn_mfma.hip)

// Key list of one wave.  Entry tables of four tiles of 64 packed keys; tile t of the list is at t mod 4.
struct WaveTables {
    alignas(16) unsigned off[4][64];   // byte offset of each key's row, in the order the loading lanes want them
    alignas(16) int lo[4][64];         // row takes key <=> lo < v < hi (written only for tiles that need it)
    alignas(16) int hi[4][64];
    int ent[2][128];                   // plan entries of the next two batches: first words, second words
    int cb[2][64];                     // first tokens of the chunks of the next batch, and of the chunks behind them
};

struct WaveKeys {
    WaveTables &tab;
    const int2 *ent;
    const int32_t *B;
    int E, lane, row_end, b_l, v_lo, v_hi;
    unsigned row_bytes;
    int off_slot_wr;
    unsigned win_fix;
    // lane = segment of the current batch of 64 plan entries: those that hold keys for this tile first, in list order
    int seg_start, seg_d, seg_pos, seg_rem;   // first packed key; token - packed key; pos and rem of the entry
    unsigned long long spec;                  // segments whose keys not every row need take
    int batch_end, e0, fetched, j_last;
    // the steps of one tile's list
    unsigned long long c0, c1, marks;
    int s_lo, n_new, a[4], dj, fast;

    __device__ __forceinline__ WaveKeys(WaveTables &t) : tab(t) {}

    // Entries of batch b, and chunk bounds of entries that are there, straight into LDS: nothing waits for them until the
    // batch is taken.
    __device__ __forceinline__ void fetch_entries(int b, int n) {
        const int e = b * 64 + lane;
        const unsigned off = 8u * (unsigned)(e < n ? e : 0), dst = lds_address(tab.ent[b & 1]);
        load_dwords(ent, off, dst);
        load_dwords(ent, off + 4u, dst + 256);
    }
    __device__ __forceinline__ void fetch_bounds(int b) {
        const unsigned off = b * 64 + lane < E ? 4u * (unsigned)(tab.ent[b & 1][lane] & kChunkMask) : 0u;
        const unsigned dst = lds_address(tab.cb);
        load_dwords(B, off, dst);
        load_dwords(B, off + 4u, dst + 256);
    }
    // t: the tile whose list is being made
    __device__ __forceinline__ void next_batch(int t) {
        const int b = e0 >> 6;
        if ((e0 & (kListPart - 1)) == 0) batch_end = (batch_end + 63) & ~63;   // the next tile's first key
        if (t < fetched + 2) { WAVE_VMCNT(0); }   // else a whole tile's loads went out behind these and have been waited for
        fetched = t;
        const int w0 = tab.ent[b & 1][lane], rem = tab.ent[b & 1][64 + lane];
        const int b0 = tab.cb[0][lane], b1 = tab.cb[1][lane];
        const int pos = w0 >> kPosShift;
        int n = 0;
        if (e0 + lane < E) {
            n = entry_take(pos, rem, b1 - b0, pos == 1 ? v_hi : v_lo);
            if (pos == 3) {   // keys past the tile's last row are nobody's
                const int vis = row_end - b0;
                n = vis < n ? (vis > 0 ? vis : 0) : n;
            }
        }
        const int inc = wave_incl_scan(n);
        const unsigned long long keep = __ballot(n > 0);
        const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(keep >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)keep, 0));
        const int to = 4 * (n > 0 ? below : __popcll(keep) + lane - below);   // segments without keys go behind the others
        const int st = batch_end + inc - n;
        batch_end += __builtin_amdgcn_readlane(inc, 63);
        seg_start = __builtin_amdgcn_ds_permute(to, n > 0 ? st : batch_end);
        seg_d = __builtin_amdgcn_ds_permute(to, b0 - st);
        seg_pos = __builtin_amdgcn_ds_permute(to, n > 0 ? pos : 0);
        const int seg_all = __builtin_amdgcn_ds_permute(to, pos == 3 && b0 + n <= v_lo + b_l);   // no key past the tile's first row
        seg_rem = __builtin_amdgcn_ds_permute(to, rem);
        spec = __ballot(seg_pos != 0 && !seg_all);
        e0 += 64;
        if (e0 < E) fetch_bounds(b + 1);
        if (e0 + 64 < E) fetch_entries(b + 2, E);
    }
    __device__ __forceinline__ void put_offset(int t, int j) { tab.off[t & 3][off_slot_wr] = __umul24(j, row_bytes) + win_fix; }

    // List of any tile (keys of several batches, keys that not every row takes, the end of the list or of a part).  Returns
    // the number of its keys; behind the last key the last one is repeated for no row.
    __device__ __forceinline__ int general(int t, int &flag) {
        int x = t * 64;
        const int xe = x + 64, xl = x + lane;
        int j = 0, lo = 0, hi = kNoKey;
        while (x < xe) {
            if (x >= batch_end) {
                if (e0 >= E || ((e0 & (kListPart - 1)) == 0 && x > t * 64)) break;
                next_batch(t);
                continue;
            }
            const int e = __popcll(__ballot(seg_start <= x)) - 1;
            const int d = __builtin_amdgcn_readlane(seg_d, e), ps = __builtin_amdgcn_readlane(seg_pos, e);
            const int en = e < 63 ? __builtin_amdgcn_readlane(seg_start, e + 1) : batch_end;
            if (xl >= x) { j = d + xl; lo = 0; hi = kNoKey; }
            if (ps != 0) {
                const int rem = __builtin_amdgcn_readlane(seg_rem, e), st = __builtin_amdgcn_readlane(seg_start, e);
                if (xl >= x) {
                    if (ps & 1) lo = j > b_l ? j - b_l : 0;   // key j is at or below row i <=> j - b_l < v
                    if (ps == 2) hi = rem - (xl - st);
                }
            }
            j_last = d + en - 1;
            x = en < xe ? en : xe;
        }
        if (xl >= x) { j = j_last; lo = kNoKey; hi = kNoKey; }
        put_offset(t, j);
        flag = __popcll(__ballot((lo >= v_lo) || (hi <= v_hi)));
        if (flag) {
            tab.lo[t & 3][lane] = lo;
            tab.hi[t & 3][lane] = hi;
        }
        return x - t * 64;
    }
    // The common tile in steps of a few instructions: 64 keys of the current batch that every row takes, with at most four
    // segments that start among them (else fast = 0 and `general`, which takes 900 cycles, makes the list anew).
    template <int S>
    __device__ __forceinline__ void step(int t) {
        const int x0 = t * 64;
        if constexpr (S == 0) { c0 = __ballot(seg_start <= x0); c1 = __ballot(seg_start < x0 + 64); }
        if constexpr (S == 1) {
            s_lo = __popcll(c0) - 1;
            n_new = __popcll(c1) - 1 - s_lo;
            a[0] = __builtin_amdgcn_readlane(seg_start, (s_lo + 1) & 63) - x0 - 1;
            a[1] = __builtin_amdgcn_readlane(seg_start, (s_lo + 2) & 63) - x0 - 1;
        }
        if constexpr (S == 2) {
            a[2] = __builtin_amdgcn_readlane(seg_start, (s_lo + 3) & 63) - x0 - 1;
            a[3] = __builtin_amdgcn_readlane(seg_start, (s_lo + 4) & 63) - x0 - 1;
        }
        // bit p - 1 for a segment that starts at key p of the tile; starts outside of it land on bit 63, which counts for no lane
        if constexpr (S == 3) { marks = 1ull << ((unsigned)a[0] < 63u ? a[0] : 63); marks |= 1ull << ((unsigned)a[1] < 63u ? a[1] : 63); }
        if constexpr (S == 4) { marks |= 1ull << ((unsigned)a[2] < 63u ? a[2] : 63); marks |= 1ull << ((unsigned)a[3] < 63u ? a[3] : 63); }
        if constexpr (S == 5) {
            const int sg = __builtin_amdgcn_mbcnt_hi((unsigned)(marks >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)marks, s_lo));
            dj = __builtin_amdgcn_ds_bpermute(4 * sg, seg_d);
        }
        if constexpr (S == 6)
            fast = (x0 + 64 <= batch_end) & (n_new <= 4) & (((spec >> (s_lo & 63)) & ((2ull << (n_new & 63)) - 1)) == 0);
        if constexpr (S == 7) put_offset(t, x0 + lane + dj);
    }
};

// LDS of one workgroup.  W = 1: two slots (blocks of 32 keys) of K and of V, block b of a tile in slot b.  W = 2: four,
// block j of the list in slot j mod 4.
template <int W>
struct WaveSmem {
    alignas(1024) uint16_t K[2 * W][32 * kWaveD];
    alignas(1024) uint16_t V[2 * W][32 * kWaveD];
    WaveTables tab[W];
};

template <int RB, int W>
__device__ __forceinline__ void attn_wave(WaveSmem<W> &sm, const PlanView &pv, const AttnArgs &a, const int h, const int l,
                                          const int row0) {
    constexpr int D = kWaveD, OPR = D / 8, RPW = 64 / OPR, NLD = 32 / RPW;   // 16-byte pieces per row, rows per window, windows per block
    constexpr int NS = D / 16, NDB = D / 32;                      // products per unit: NS scores, 2 NDB of P V
    constexpr int NM = NS + 2 * NDB;                              // products per phase
    constexpr int S0 = NS + 1;                  // the product beside which a unit's first exponential is taken
    constexpr int SLOT = 64 * D;                // bytes of a slot
    static_assert(NM == 16, "one exponential beside each product");
    constexpr int LPW = NLD / W;                // windows of a block that this wave fetches
    constexpr bool pair = W == 2;
    constexpr bool dense = RB == 2 && !pair;    // V fragments are read in the phase that uses the old ones last; else spread over two
    constexpr bool k_first = RB == 2;           // K fragments are read beside the products that use the old ones last; else behind them
    // Tiles of at most 64 rows, as attn_tile_16 has them: each half of a tile's keys has its own softmax state (reference,
    // sums, O), merged at the end; a row's sum is made in parts of 8 keys, 16 rows move their references together, and
    // P V takes the keys in the order of a 16x16x32 product (two 32x32x16 products, one after the other, give its bits).
    // The states cost a third of a percent of a prefill of 131072 tokens (22.31 -> 22.37 ms) and fill the accumulation
    // registers, so all Q fragments live in vector registers.
    constexpr bool split = RB == 2 && !pair;
    constexpr int NST = split ? 2 * RB : RB;    // softmax states: of row block r and key half hf: hf RB + r
    constexpr int NP = split ? 2 : 1;           // parts of a row's sum
    constexpr int QA = split ? 0 : 2;           // row blocks whose Q fragments live in accumulation registers

    const int lane = threadIdx.x & 63, wave = pair ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int lr = lane & 31, g2 = lane >> 5;
    const int g = h / a.G;
    const float scale_log2e = a.scale_log2e;
    const char *Kg8 = reinterpret_cast<const char *>(a.K + (int64_t)g * a.ks_h) - 3072;   // (see win_fix)
    const char *Vg8 = reinterpret_cast<const char *>(a.V + (int64_t)g * a.vs_h) - 3072;

    // What the list needs first: the entries do not wait for their number (a prologue is a chain of dependent loads).
    WaveKeys keys(sm.tab[wave]);
    keys.lane = lane;
    keys.ent = reinterpret_cast<const int2 *>(pv.entries) + ((int64_t)h * pv.N_q + l) * pv.stride;
    keys.B = pv.B;
    keys.fetch_entries(0, pv.stride);
    keys.fetch_entries(1, pv.stride);
    const int b_l = pv.RB[l];
    const int rows_left = pv.RB[l + 1] - row0;
    const int E = pv.count[(int64_t)h * pv.N_q + l];
    const int nrows = rows_left < 32 * RB * W ? rows_left : 32 * RB * W;
    const int v_lo = row0 + 1 - b_l, v_hi = v_lo + nrows - 1;

    // Q fragments (B operand of S^T = K Q^T): lane holds row lr of a row block, d = 16 s + 8 g2 .. + 7
    bf16x8 qf[RB][NS];
    float m_ref[NST], l_run[NST][NP];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const int rr = (wave * RB + r) * 32 + lr;
        const uint16_t *qp = a.Q + (int64_t)h * a.qs_h + (int64_t)(row0 + (rr >= nrows ? nrows - 1 : rr)) * a.qs_l + 8 * g2;
#pragma unroll
        for (int s = 0; s < NS; ++s) qf[r][s] = *reinterpret_cast<const bf16x8 *>(qp + 16 * s);
#pragma unroll
        for (int st = r; st < NST; st += RB) {
            m_ref[st] = rr >= nrows ? 1e30f : __builtin_nanf("");   // padding rows: q = 0, p = 0
#pragma unroll
            for (int k = 0; k < NP; ++k) l_run[st][k] = 0.f;
        }
    }
    static_for<NST * NDB>([](auto G) __attribute__((always_inline)) { acc_zero<decltype(G)::value>(); });

    keys.E = E;
    keys.row_end = row0 + nrows; keys.b_l = b_l; keys.v_lo = v_lo; keys.v_hi = v_hi;
    keys.row_bytes = (unsigned)a.ks_l * 2u;
    {
        // slot of key `lane` of a tile in the offset table: the rows one lane fetches for a block are adjacent.  The load of
        // window c adds 1024 (c mod 4) to its global address too, which the offset and the bases take back.
        const int x = lane & 31;
        keys.off_slot_wr = (lane & 32) + (x % RPW) * NLD + x / RPW;
        keys.win_fix = 3072u - 1024u * ((x / RPW) & 3);
    }
    keys.seg_start = keys.seg_d = keys.seg_pos = keys.seg_rem = 0;
    keys.spec = 0;
    keys.batch_end = keys.e0 = keys.fetched = keys.j_last = 0;

    // ---- staging: lane L of a window's load fills bytes [16 L, 16 L + 16) of it: a piece of row L / OPR of the window ----
    const int c_first = wave * LPW;
    const int off_slot_rd = (lane / OPR) * NLD + c_first;
    // byte offset of this lane's logical piece of its row in window c: the swizzle of a row 4 c further differs from that in
    // window 0.  The kernel of 33..64 rows has no registers to keep the four in.
    static_assert(RPW == 4 && LPW % 4 == 0, "rows of windows c and c + 4 have the same swizzle");
    unsigned piece[4];
    const auto flip = [](int c) __attribute__((always_inline)) { return 16u * ((c & 1) | (c & 2) << 2); };
#pragma unroll
    for (int c = 0; c < 4; ++c) piece[c] = 16u * ((lane % OPR) ^ piece_swizzle(lane / OPR, OPR)) ^ flip(c);
    const auto add_piece = [&](unsigned &off, int c) __attribute__((always_inline)) {
        if (!split || (c & 3) == 0) off += piece[c & 3];
        else WAVE_ASM("v_xad_u32 %0, %1, %2, %0" : "+v"(off) : "v"(piece[0]), "s"(flip(c)));
    };
    const unsigned lds_K = lds_address(sm.K) + c_first * 1024, lds_V = lds_address(sm.V) + c_first * 1024;
    unsigned offs[2][LPW];   // byte offsets of the pieces this lane fetches for an even and for an odd block, K and V alike
#define WAVE_OFFS(t, half) \
    { \
        _Pragma("unroll") for (int c = 0; c < LPW; ++c) offs[half][c] = keys.tab.off[(t) & 3][(half) * 32 + off_slot_rd + c]; \
        _Pragma("unroll") for (int c = 0; c < LPW; ++c) add_piece(offs[half][c], c); \
    }
#define WAVE_LOAD(base, dst, half, c) { load_window(base, offs[half][c], (dst) + ((c) & ~3) * 1024, (c) & 3); }

    // ---- fragment addresses (bytes inside K / V; the swizzles and the transpose reads of attn_mfma.hip) ----
    typedef __attribute__((address_space(3))) char lds_char;
    lds_char *const smK8 = (lds_char *)sm.K, *const smV8 = (lds_char *)sm.V;
    const int k_sw = piece_swizzle(lr, OPR);
    int k_off[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) k_off[s] = 2 * (lr * D + 8 * ((2 * s + g2) ^ k_sw));
    const int tr_c = (lane & 15) >> 2, tr_r = lane & 3, tr_dh = (lane >> 4) & 1;
    const int tr_low2 = ((tr_r >> 1) ^ g2) | ((tr_dh ^ (tr_c & 1)) << 1);
    const int tr_l0 = (4 * g2 + tr_c) * D + 8 * tr_low2 + 4 * (tr_r & 1);
    int v_base_e = 2 * (tr_l0 + 32 * (tr_c >> 1)), v_base_o = 2 * (tr_l0 - 32 * (tr_c >> 1));
    int toggle = 2 * SLOT;   // W = 2: +, -, ...: k_off and v_base follow the slots of even and odd tiles

    typedef long i64x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    bf16x8 kf[NS];        // K fragments of a block
    i64x2 vf[2 * NDB];    // V^T fragments of a block
    f32x16 sc[2];         // scores of a unit, by parity
    u32x4 pf[2][2];       // P of a unit as bf16 pairs: the two B operands
    float ex[16], psum[2][NP], mc = 0.f, mc_next = 0.f;
#define WAVE_READ_K(s, slot) kf[s] = *(bf16x8 __attribute__((address_space(3))) *)(smK8 + k_off[s] + (slot) * SLOT);
#define WAVE_READ_V(k, slot) /* half (k & 1) of fragment k / 2 */ \
    { \
        const int j_ = (k) / 2, half_ = (k) & 1; \
        const int up8_ = split ? j_ / NDB : half_, up16_ = split ? half_ : j_ / NDB; /* keys + 8, + 16 */ \
        const int x2_ = (j_ % NDB) ^ (2 * up8_); \
        union { s16x4 h; long u; } r_; \
        r_.h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)( \
            smV8 + ((x2_ & 1) ? v_base_o : v_base_e) + 2 * ((16 * up16_ + 8 * up8_) * D + 32 * x2_) + (slot) * SLOT)); \
        vf[j_][half_] = r_.u; \
    }
// exponentials of elements x0 .. x1-1 of the unit of parity p; their sums and rounding
#define WAVE_EXP(p, x0, x1) \
    _Pragma("unroll") for (int x = (x0); x < (x1); ++x) { \
        ex[x] = __builtin_amdgcn_exp2f(sc[p][x] * scale_log2e - mc); \
        WAVE_ASM("" : "+v"(ex[x])); \
    }
#define WAVE_PART(x) (split ? ((x) >> 2) & 1 : 0)
#define WAVE_P(p, x) pf[p][split ? ((x) >> 2) & 1 : (x) >> 3][split ? ((x) >> 3) * 2 + (((x) & 3) >> 1) : ((x) & 7) >> 1]
#define WAVE_SUM(p, x0, x1) \
    _Pragma("unroll") for (int x = (x0); x < (x1); ++x) { \
        const int part_ = WAVE_PART(x); \
        psum[p][part_] = x == 4 * part_ ? ex[x] : psum[p][part_] + ex[x]; \
        if (x & 1) { \
            unsigned w_; \
            WAVE_ASM("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(w_) : "v"(ex[x - 1]), "v"(ex[x])); \
            WAVE_P(p, x) = w_; \
        } \
        WAVE_ASM("" : "+v"(psum[p][part_])); \
    }
    // What only rare branches need is made there, from a copy of the lane number that nothing can be hoisted from: there are
    // no registers to keep it in.
    const auto fresh_lane = [&]() __attribute__((always_inline)) { int ln = lane; WAVE_ASM("" : "+v"(ln)); return ln; };
    // keys that not every row of the tile takes, row block r
    const auto mask = [&](int t, int half, f32x16 &s, int r) __attribute__((always_inline)) {
        const int ln = fresh_lane(), v = v_lo + (wave * RB + r) * 32 + (ln & 31), g2 = ln >> 5;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            __builtin_amdgcn_sched_barrier(0);   // one after another: there are few registers
            const int key = half * 32 + q4 * 8 + g2 * 4;
            const int4 lo = *reinterpret_cast<const int4 *>(&keys.tab.lo[t & 3][key]);
            const int4 hi = *reinterpret_cast<const int4 *>(&keys.tab.hi[t & 3][key]);
            s[q4 * 4 + 0] = ((v > lo.x) & (v < hi.x)) ? s[q4 * 4 + 0] : -INFINITY;
            s[q4 * 4 + 1] = ((v > lo.y) & (v < hi.y)) ? s[q4 * 4 + 1] : -INFINITY;
            s[q4 * 4 + 2] = ((v > lo.z) & (v < hi.z)) ? s[q4 * 4 + 2] : -INFINITY;
            s[q4 * 4 + 3] = ((v > lo.w) & (v < hi.w)) ? s[q4 * 4 + 3] : -INFINITY;
        }
    };

    // maximum of a unit of scores over the row (the two lanes of a row exchange their halves)
    const auto row_max = [&](const f32x16 &s) __attribute__((always_inline)) {
        float mx = s[0];
#pragma unroll
        for (int x = 1; x < 16; ++x) mx = fmaxf(mx, s[x]);
        return fmaxf(mx, __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (fresh_lane() ^ 32), __float_as_int(mx))));
    };
    // the first block of a softmax state: its reference is the row's maximum there
    const auto first_reference = [&](float &m, const f32x16 &s) __attribute__((always_inline)) {
        const float mx = row_max(s);
        if (mx != -INFINITY) m = fmaxf(m, mx);
    };

    // ---- lists of tiles 0..2 ----
    int fl0 = 0, fl1 = 0, fl2 = 0;      // keys of tiles t .. t + 2 that not every row takes
    int has0 = 0, has1 = 0, has2 = 0;   // keys of tiles t .. t + 2
    if (E > 0) {
        WAVE_VMCNT(0);
        keys.fetch_bounds(0);
#pragma nounroll
        for (int t = 0; t < 3; ++t) {
            keys.fetched = t;
            has0 = has1; has1 = has2;
            fl0 = fl1; fl1 = fl2;
            has2 = __builtin_amdgcn_readfirstlane(keys.general(t, fl2));
            fl2 = __builtin_amdgcn_readfirstlane(fl2);
        }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (m_ref[r] == 1e30f) qf[r][s] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            if constexpr (QA > 0) {
                if (r < QA) WAVE_ASM("" : "+a"(qf[r][s]));
                else WAVE_ASM("" : "+v"(qf[r][s]));
            } else WAVE_ASM("" : "+v"(qf[r][s]));
        }

    // ---- first loads, scores of unit 0 and the first of its exponentials ----
    if (has0 != 0) {
        WAVE_OFFS(0, 0)
#pragma unroll
        for (int c = 0; c < LPW; ++c) WAVE_LOAD(Kg8, lds_K, 0, c)
#pragma unroll
        for (int c = 0; c < LPW; ++c) WAVE_LOAD(Vg8, lds_V, 0, c)
        WAVE_OFFS(0, 1)
#pragma unroll
        for (int c = 0; c < LPW; ++c) WAVE_LOAD(Kg8, lds_K + SLOT, 1, c)
#pragma unroll
        for (int c = 0; c < LPW; ++c) WAVE_LOAD(Vg8, lds_V + SLOT, 1, c)
        if constexpr (pair) {
            WAVE_OFFS(1, 0)
#pragma unroll
            for (int c = 0; c < LPW; ++c) WAVE_LOAD(Kg8, lds_K + 2 * SLOT, 0, c)
#pragma unroll
            for (int c = 0; c < LPW; ++c) WAVE_LOAD(Vg8, lds_V + 2 * SLOT, 0, c)
            WAVE_OFFS(1, 1)
#pragma unroll
            for (int c = 0; c < LPW; ++c) WAVE_LOAD(Kg8, lds_K + 3 * SLOT, 1, c)
            WAVE_ASM("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(6 * LPW) : "memory");   // K(0) of both waves
        } else {
            WAVE_VMCNT(3 * NLD);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) WAVE_READ_K(s, 0)
#pragma unroll
        for (int s = 0; s < NS; ++s) scores_mfma<(QA > 0)>(sc[0], kf[s], qf[0][s], s == 0);
        WAVE_ASM("s_nop 15\n\ts_nop 7" : "+v"(sc[0]));
        if constexpr (!pair) {
            WAVE_OFFS(1, 0)
#pragma unroll
            for (int c = 0; c < NLD / 2; ++c) WAVE_LOAD(Kg8, lds_K, 0, c)   // (the other half in phase 0)
        }
        if (fl0 != 0) mask(0, 0, sc[0], 0);
        first_reference(m_ref[0], sc[0]);
        fl0 |= kFirstTile;
        mc = m_ref[0] * scale_log2e;
        WAVE_EXP(0, 0, NM - S0)
        WAVE_SUM(0, 0, NM - S0 - 1)
#pragma unroll
        for (int i = 0; i < 2 * NDB; ++i) vf[i] = i64x2{0, 0};
        pf[1][0] = pf[1][1] = u32x4{0, 0, 0, 0};
    }

    // ---- tile t: phases 0 .. 2 RB - 1, one per unit ----
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0), see the end of the loop
    for (int t = 0; has0 != 0; ++t) {
        // Phase P: scores of unit P + 1, then O += P V of unit P - 1; beside products up to S0 - 1 exponentials of unit P,
        // from S0 on of unit P + 1.
        const auto phase = [&](auto PC) __attribute__((always_inline)) {
            constexpr int P = decltype(PC)::value;
            constexpr int r = P % RB, rq = (P + 1) % RB, rp = (P + 2 * RB - 1) % RB;   // row blocks of the three units
            constexpr int p = P & 1, q = p ^ 1;
            constexpr int hf = P / RB;                                                  // block of unit P in the tile
            constexpr bool kref = rq == RB - 1, vref = rp == RB - 1;   // the K / V fragments of a block are used for the last time
            constexpr int st = split ? P : r, stq = split ? (P + 1) % NST : rq, stp = split ? (P + NST - 1) % NST : rp;   // and their states
            constexpr bool first = P + 1 < NST;                        // unit P + 1 may be the first block of its state
            unsigned long long far = 0;
            // Loads in flight when a block is needed: W = 1: those of three blocks behind V, of two behind K (of one and a half
            // where K is read first thing in the phase).  W = 2: those of the last two phases' pairs (V(j+3), K(j+4)); what a
            // wave has waited for the other may read behind the barrier, and then the slots of K(j) and V(j-1) are free.
            if constexpr (pair) {
                if (r == 0) WAVE_ASM("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(4 * LPW) : "memory");
            } else if (kref && dense) {
                WAVE_VMCNT(NLD + NLD / 2);
            }
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                __builtin_amdgcn_sched_barrier(0);
                const int j = i - NS;
                // the product, and the fragments it frees
                if (i < NS) {
                    scores_mfma<(rq < QA)>(sc[q], kf[i], qf[rq][i], i == 0);
                    if (kref && k_first) WAVE_READ_K(i, hf ^ 1)
                    if (!dense && r == 1) WAVE_READ_V(2 * NDB + i, hf)   // what the phase before left over
                } else {
                    if (j == 0 && !pair && vref && !dense) { WAVE_VMCNT(3 * NLD); }
                    if (j == 0 && kref && !k_first) { WAVE_VMCNT(2 * NLD); }
                    if (j == 0) WAVE_ASM("s_nop 1" ::: "memory");   // (a product reads P two issues after its conversion at the earliest)
                    static_for<NDB>([&](auto DB) __attribute__((always_inline)) {
                        constexpr int db = decltype(DB)::value;
                        if (j % NDB == db) acc_mfma<stp * NDB + db>(vf[j], pf[q][j / NDB]);
                    });
                    if (vref && dense) { WAVE_READ_V(2 * j, hf) WAVE_READ_V(2 * j + 1, hf) }
                    if (vref && !dense) WAVE_READ_V(j, hf)
                    if (kref && !k_first) WAVE_READ_K(j, hf ^ 1)
                }
                if constexpr (pair) {
                    // even phases: the offsets of block j + 4; odd ones: V(j+3) and K(j+4), beside a product each
                    const unsigned odd = (unsigned)(t & 1) * 2 * SLOT;
#pragma unroll
                    for (int c = 0; c < LPW; ++c) {
                        if (r == 1 && i == NS + c) WAVE_LOAD(Vg8, lds_V + (hf == 0 ? 3 * SLOT - odd : odd), hf ^ 1, c)
                        if (r == 0 && i == NS) offs[hf][c] = keys.tab.off[(t + 2) & 3][hf * 32 + off_slot_rd + c];
                        if (r == 1 && i == 2 * c) add_piece(offs[hf][c], c);
                        if (r == 1 && i == NS + LPW + c) WAVE_LOAD(Kg8, lds_K + odd + hf * SLOT, hf, c)
                    }
                    if (P == 1 && i < NS) k_off[i] += toggle;   // K(A) of the next tile is read in phase 2
                    if (P == 3 && i == NS) v_base_e += toggle;
                    if (P == 3 && i == NS + 1) v_base_o += toggle;
                } else {
                    // phase r = RB - 1: V of the next tile's block hf, then K of the block behind it, whose second half follows
                    // in the next phase; each beside a product of its own, as far as there are any
#pragma unroll
                    for (int c = 0; c < NLD; ++c) {
                        const int at_v = RB == 3 ? c + c / 2 : c + 2 + (c >= 6);
                        if (r == RB - 1) {
                            if (RB == 2 && c == 0 && i == 2) WAVE_ASM("s_waitcnt lgkmcnt(0)" ::: "memory");   // V fragments of this slot
                            if (at_v == i) WAVE_LOAD(Vg8, lds_V + hf * SLOT, hf, c)
                            if (c / 4 == i) offs[hf ^ 1][c] = keys.tab.off[(hf ? t + 2 : t + 1) & 3][(hf ^ 1) * 32 + off_slot_rd + c];
                            if (i == 4 + c) add_piece(offs[hf ^ 1][c], c);
                            if (c < NLD / 2 && i == 12 + c) WAVE_LOAD(Kg8, lds_K + (hf ^ 1) * SLOT, hf ^ 1, c)
                        }
                        if (r == 0 && c >= NLD / 2 && i == 2 * (c - 4) + dense) WAVE_LOAD(Kg8, lds_K + hf * SLOT, hf, c)
                    }
                }
                if (i == S0) {   // the scores of unit P + 1 are complete
                    int fl = (P + 1) / RB < 2 ? fl0 : fl1;
                    WAVE_ASM("" : "+s"(fl));
                    if (__builtin_expect(fl != 0, 0)) {
                        if (fl & ~kFirstTile) mask((P + 1) / RB < 2 ? t : t + 1, ((P + 1) / RB) & 1, sc[q], rq);
                        if (first && (fl & kFirstTile)) {
                            first_reference(m_ref[stq], sc[q]);
                            mc_next = m_ref[stq] * scale_log2e;
                        }
                    }
                    mc = mc_next;
                }
                if (i == S0 - 2) mc_next = m_ref[stq] * scale_log2e;
                {
                    const int k = (i + NM - S0) % NM, kl = (i + NM - 1 - S0) % NM;
                    WAVE_EXP((i >= S0 ? q : p), k, k + 1)
                    WAVE_SUM((i > S0 ? q : p), kl, kl + 1)
                }
                // list of tile t + 3
                static_for<8>([&](auto SC) __attribute__((always_inline)) {
                    constexpr int S = decltype(SC)::value;
                    constexpr int at_p = S < 4 ? 0 : S < 7 ? RB : 2 * RB - 1;
                    constexpr int at_i = S == 7 ? 10 : 2 * (S & 3) + (RB == 3);
                    if (P == at_p && i == at_i) keys.template step<S>(t + 3);
                });
                if (i == S0 + 1) {
                    if constexpr (split) far = __ballot(!(psum[p][0] < kFar) || !(psum[p][NP - 1] < kFar));
                    else far = __ballot(!(psum[p][0] < kFar));
                    WAVE_ASM("" : "+s"(far));
                }
                if (i == S0 + 3) {
                    // unit P: too large, inf or NaN, or no reference yet: move the reference, take the exponentials again
                    if (__builtin_expect(far != 0, 0)) {
                        const f32x16 &s = sc[p];
                        const bool mine = !split || (far & (0x0000ffff0000ffffull << (fresh_lane() & 16))) != 0;
                        const float m_old = m_ref[st], mx = row_max(s);
                        float scale = scale_log2e;   // one of its own: else the products below are made before the branch
                        WAVE_ASM("" : "+s"(scale));
                        const float m_new = mine ? fmaxf(m_old, mx) : m_old;   // the other one if one is NaN
                        const bool none = m_new == -INFINITY;
                        const float alpha = (m_old != m_old) ? 0.f : __builtin_amdgcn_exp2f((m_old - m_new) * scale);
                        static_for<NDB>([&](auto DB) __attribute__((always_inline)) { acc_scale<st * NDB + decltype(DB)::value>(alpha); });
                        const float ref = none ? 0.f : m_new * scale;
                        m_ref[st] = none ? __builtin_nanf("") : m_new;
#pragma unroll
                        for (int k = 0; k < NP; ++k) { l_run[st][k] *= alpha; psum[p][k] = 0.f; }
                        float e2[2];
#pragma unroll
                        for (int x = 0; x < 16; ++x) {
                            float d = s[x] * scale;   // rounded like ref: the row's maximum weighs 1 however large it is
                            WAVE_ASM("" : "+v"(d));
                            d -= ref;
                            if (split && !mine) d = __builtin_fmaf(s[x], scale, -ref);
                            e2[x & 1] = __builtin_amdgcn_exp2f(d);
                            psum[p][WAVE_PART(x)] += e2[x & 1];
                            if (x & 1) {
                                union { __bf16 b[2]; unsigned u; } w;
                                w.b[0] = (__bf16)e2[0]; w.b[1] = (__bf16)e2[1];
                                WAVE_P(p, x) = w.u;
                            }
                        }
                    }
#pragma unroll
                    for (int k = 0; k < NP; ++k) l_run[st][k] += psum[p][k];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        static_for<2 * RB>([&](auto PC) __attribute__((always_inline)) { phase(PC); });
        toggle = -toggle;
        int has3 = 64, fl3 = 0;
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(keys.fast) == 0, 0)) {
            has3 = keys.general(t + 3, fl3);
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): scalar loads in flight would make every later LDS wait a full one
        }
        has0 = has1; has1 = has2; has2 = __builtin_amdgcn_readfirstlane(has3);
        fl0 = fl1; fl1 = fl2; fl2 = __builtin_amdgcn_readfirstlane(fl3);
    }
    WAVE_VMCNT(0);   // no load may land in LDS that is another workgroup's by then
    if (keys.batch_end > 0)
        static_for<2 * NDB>([&](auto J) __attribute__((always_inline)) {   // O += P V of the last unit
            constexpr int j = decltype(J)::value;
            acc_mfma<(NST - 1) * NDB + j % NDB>(vf[j], pf[1][j / NDB]);
        });
    WAVE_ASM("s_nop 15\n\ts_nop 7" ::: "memory");

    // ---- normalise, round to bf16, store ----
    static_for<RB>([&](auto R) __attribute__((always_inline)) {
        constexpr int r = decltype(R)::value;
        float a0 = 1.f, a1 = 0.f;   // weights of the states of the two key halves
        if constexpr (split) {
            const float m0 = m_ref[r], m1 = m_ref[RB + r], mm = fmaxf(m0, m1);   // NaN: no key seen (and then the other one is taken)
            a0 = m0 != m0 ? 0.f : __builtin_amdgcn_exp2f((m0 - mm) * scale_log2e);
            a1 = m1 != m1 ? 0.f : __builtin_amdgcn_exp2f((m1 - mm) * scale_log2e);
        }
        float l_tot = 0.f;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            float l = l_run[r][k];
            if constexpr (split) l = __builtin_fmaf(l, a0, l_run[RB + r][k] * a1);
            l += __shfl_xor(l, 32);
            l_tot = k == 0 ? l : l_tot + l;
        }
        const int rr = (wave * RB + r) * 32 + lr;
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;   // no visible key (row-block form): zeros
        uint16_t *op = a.O + (int64_t)h * a.os_h + (int64_t)(row0 + rr) * a.os_l;
        static_for<4 * NDB>([&](auto X) __attribute__((always_inline)) {
            constexpr int db = decltype(X)::value / 4, q4 = decltype(X)::value % 4;
            float o[4];
            acc_read<r * NDB + db, q4>(o);
            if constexpr (split) {
                float o1[4];
                acc_read<(RB + r) * NDB + db, q4>(o1);
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = __builtin_fmaf(o[x], a0, o1[x] * a1);
            }
            union { __bf16 b[4]; uint2 u; } pk;
#pragma unroll
            for (int x = 0; x < 4; ++x) pk.b[x] = (__bf16)(o[x] * inv);
            if (rr < nrows) *reinterpret_cast<uint2 *>(op + db * 32 + q4 * 8 + g2 * 4) = pk.u;
        });
    });
#undef WAVE_OFFS
#undef WAVE_LOAD
#undef WAVE_READ_K
#undef WAVE_READ_V
#undef WAVE_EXP
#undef WAVE_SUM
#undef WAVE_PART
#undef WAVE_P
}

// Tiles tile0 .. tile0 + T - 1 of 97..128 rows (or 65..96 that ride along), two waves each, from the end of the sequence (most keys) to its start
__global__ __launch_bounds__(128, 1) void k_attn_wave2(PlanView pv, AttnArgs a, int order, int tile0, int T) {
    __shared__ WaveSmem<2> sm;
    int h, pos;
    if (!decode_block(order, blockIdx.x, a.G, T, &h, &pos)) return;
    const int tile = tile0 + T - 1 - pos;
    const int l = pv.tiles[2 * tile], row0 = pv.tiles[2 * tile + 1];   // query group, first row
    if (!plan_matches(pv)) return;   // not this problem's plan: nothing else is used, O is not written
    attn_wave<2, 2>(sm, pv, a, h, l, row0);
}

// Tiles tile0 .. tile0 + T - 1 of 65..96 (RB = 3) or 33..64 rows (RB = 2), a wave each
template <int RB>
__global__ __launch_bounds__(64, 1) void k_attn_wave1(PlanView pv, AttnArgs a, int order, int tile0, int T) {
    __shared__ WaveSmem<1> sm;
    int h, pos;
    if (!decode_block(order, blockIdx.x, a.G, T, &h, &pos)) return;
    const int tile = tile0 + T - 1 - pos;
    const int l = pv.tiles[2 * tile], row0 = pv.tiles[2 * tile + 1];
    if (!plan_matches(pv)) return;
    attn_wave<RB, 1>(sm, pv, a, h, l, row0);
}

// Which height classes of the tile table (bit c = class c) the kernels of this file take.  A wave has to itself what four
// waves share in attn_mfma.hip: it is faster per tile, but a tile takes longer, its prologue (6 us) is hidden by nothing,
// and a round is 1024 waves.  Hence heads of 128, lists of a thousand keys or more and so many tiles that the last ones
// leave few SIMDs without work.  Both sides below are four waves -> lone waves, us of attention, 32 heads of the LLaMA shape:
//   tiles of 33..64 rows: 4608 of them, 1024 keys 214 -> 208, 2048 344 -> 321, 8192 779 -> 701
//   ... of dynamic chunks: twice as many tiles are in flight, and their walks drift apart (a partly taken chunk makes a tile's
//     list a slow one), so the L2s serve less (131072 tokens, 16 heads, 8192 keys: 31 % against 53 %, row blocks of 64 64 % against
//     55 %).  That costs time where lists are dense or K and V of the heads in flight exceed the 256 MB memory-side cache:
//     16384 tokens, 2048 keys 863 -> 788; 32768, 4096 keys 3311 -> 3148; 51585, 3224 keys 4565 -> 4493, 6448 keys 8137 -> 8849;
//     four kv-heads of 131072 tokens, 8192 keys 8666 -> 8372, eight: 2800 keys 6107 -> 5955, 3328 7024 -> 7121, 8192 14918 -> 18036;
//     where taller tiles are more: eight kv-heads of 81920, 5120 keys 4681 -> 4513, of 65536, 8192 keys 5572 -> 5392, of
//     131072, 4096 keys 6377 -> 6243, 8192 keys 12411 -> 12947 with every other tile of them and, with every third,
//     11111 -> 11222, 32 heads 22233 -> 22615 on random keys, 22757 -> 22449 with needles among them, every fifth 14230 -> 14068
//   tiles of 65..96 rows alone: 3840, 1024 keys 251 -> 232, 4096 700 -> 615
//   tiles of 97..128 rows alone, row blocks of 128: 3584, 1024 keys 281 -> 286, 1536 379 -> 375, 4096 814 -> 781;
//     8192, 1024 keys 652 -> 657, 1536 899 -> 875
//   on dynamic chunks, whose tiles have lists of their own, they gain less, and the denser the lists, the more the four-wave
//     kernel gets out of the L2s: 112 rows, 9216 tiles of 32256 tokens: 2048 keys 1298 -> 1293, 8192 3999 -> 4263; 18720 of
//     65520: 2048 keys 2732 -> 2686, 8192 9559 -> 9573; 128 rows, 32768 of 131072: 4096 keys 9592 -> 9206
//   both tall classes: half and half, 3755 of each, 1024 keys 527 -> 550, 1536 767 -> 741; 5461, 1024 keys 779 -> 770;
//     10900, 2048 keys 2974 -> 2715.  attn_mfma.hip runs both in one launch; class 0 alone leaves it only for long lists
//     (5640 tiles beside 1640, 4096 keys 1757 -> 1696), class 1 alone too (6300 beside 190 of 97 rows, 2048 keys 714 ->
//     about 714, 4096 1247 -> 1164; 3100, 4096 keys 582 -> 588)
// A few tiles of 65..96 rows ride in the launch of the taller ones (row blocks of 128 and a last one of 80 rows: 3584
// tiles, 8192 keys 1328 -> 1264; 8192 tiles, 2048 keys 1140 -> 1096).  A few of at most 64 rows are `left` with a launch
// that takes as long as a list, where four-wave kernels would take them along: row blocks of 128 and a last one of 50 rows
// 3584, 2048 keys 489 -> 497, 4096 832 -> 820; tiles of 80 rows and one of 30, 3072, 1024 keys 203 -> 205, 1536 275 -> 266.
// Heads of 64 have half the products for the same exponentials and lists: 9000 tiles of each class gain 2 %, 4700 lose 3 %.
// Chunks so short that a tile of 64 keys spans more than four make its key list a `general` one; a pair of waves, which
// makes each list twice, loses by it from 32 tokens on average down (20 tokens: 1063 -> 1090 us), a single one does not
// (20 tokens, tiles of 96 rows: 465 -> 440 us).  Offsets are 32 bits with room for a window, made by a 24-bit product, the
// same for K and V.
int attn_wave_classes(const Prob &p, const int32_t *T_cls) {
    const int64_t row_bytes = 2 * p.ks_l;
    if (p.D != kWaveD || p.N_b < 1024 || p.L < 16 * (int64_t)p.N_c || p.ks_l != p.vs_l || p.L >= 1 << 24 || row_bytes >= 1 << 24 ||
        p.L * row_bytes > 0xffffffffll - 4096)
        return 0;
    int64_t n[4];                           // tiles of each class over all heads
    for (int c = 0; c < 4; ++c) n[c] = p.H_q * (int64_t)T_cls[c];
    const auto enough = [&](int c, int64_t least) { return n[c] >= least && n[c] <= kGridMax; };
    const int64_t keys = p.N_b;             // of a full list
    bool w0 = enough(0, 3584) && p.L >= 32 * (int64_t)p.N_c, w1 = enough(1, 3072);
    const bool left = n[2] > 0 ? n[2] <= 512 : n[3] > 0 && n[3] <= 512;
    if (w0 && w1) w0 = w1 = n[0] * keys >= 3584 * 1536;
    else if (w0 && n[1] > 512) w0 = keys >= 4096;
    else if (w0 && p.B_r > 0) w0 = keys >= 1536 && (!left || n[0] * keys >= 3584 * 4096);
    else if (w0) w0 = keys >= 2048 && p.L >= 16 * keys && n[0] >= (left ? 16384 : 8192);
    else if (w1 && n[0] > 0) w1 = keys >= 4096 && n[1] * keys >= 4608 * 4096;
    else if (w1) w1 = !left || n[1] * keys >= 3072 * 1536;
    bool w2 = enough(2, 4608);
    if (w2 && p.B_r == 0) {
        const bool alone = n[2] > n[0] + n[1];
        const double live = 4.0 * p.D * p.L * (p.H_kv < 8 ? p.H_kv : 8);   // bytes of K and V of the kv-heads in flight
        const bool few_of_all = 5 * n[2] <= 2 * (n[0] + n[1] + n[2]);
        if (live > (alone ? 288e6 : 384e6)) w2 = keys <= (alone ? 3072 : 4096) || few_of_all;
        else if (alone) w2 = keys <= 4096 || p.L >= 16 * keys;
    }
    return (w0 ? 1 : 0) | (w1 ? 2 : 0) | (w2 ? 4 : 0);
}

// T tiles from tile0 on for the kernel of class cls: 0: 65..128 rows, 1: 65..96, 2: at most 64 rows
hipError_t launch_attn_wave(const Prob &p, const PlanView &pv, const AttnArgs &a, int want, int cls, int tile0, int T, hipStream_t s) {
    const int order = attn_order(want, p, T);
    const dim3 grid(attn_grid(order, p, T));
    if (cls == 0) hipLaunchKernelGGL(k_attn_wave2, grid, dim3(128), 0, s, pv, a, order, tile0, T);
    else if (cls == 1) hipLaunchKernelGGL((k_attn_wave1<3>), grid, dim3(64), 0, s, pv, a, order, tile0, T);
    else hipLaunchKernelGGL((k_attn_wave1<2>), grid, dim3(64), 0, s, pv, a, order, tile0, T);
    return hipGetLastError();
}

}  // namespace dhsa
