// Pieces of the bf16 MFMA attention kernels that the translation units share.
#pragma once
#include "dhsa_internal.h"

namespace dhsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// XOR swizzle of the 16-byte pieces of LDS row r (only r mod 16 matters).  Eight
// (sixteen for 256-byte rows) consecutive rows get distinct values, so a column
// of 16-byte reads spreads over all banks; rows r..r+3 with r % 4 == 0 differ
// in bits 1-2, so the 32-byte row segments of a transpose read do too.
__device__ __forceinline__ int piece_swizzle(int r, int pieces_per_row) {
    int f = ((r & 3) << 1) | ((r >> 2) & 1);
    if (pieces_per_row == 16) f |= ((r >> 3) & 1) << 3;
    return f;
}

// 16 bytes per lane from global memory (uniform base + per-lane 32-bit byte
// offset) straight into LDS: lane L of the wave writes bytes [16 L, 16 L + 16)
// of the window at LDS byte address `lds_window` (wave-uniform, goes through
// M0, which nothing else in this kernel uses).  Completion is tracked by vmcnt;
// the caller waits and then passes a barrier before anyone reads the window.
__device__ __forceinline__ void load16_to_lds(const char *base, unsigned byte_off, unsigned lds_window) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(byte_off), "s"(base), "s"(lds_window) : "memory");
#else
    (void)base; (void)byte_off; (void)lds_window;
#endif
}

// blockIdx -> (head, tile).  Workgroups are dealt to the 8 XCDs round-robin and
// each XCD has its own L2.  `act` kv-heads (1, 2, 4 or 8) are worked on at a
// time, each by 8 / act XCDs: act = 8 gives every XCD its own kv-head (best L2
// reuse of the K/V slabs), smaller values keep fewer K/V slabs live at once
// (they then fit the memory-side cache).  Within a kv-head the query heads of
// the group are innermost; *tile is the tile's position in the order of issue
// (0 = first), which the kernel maps to a row tile.  False: a block that only
// makes the share of every XCD equal, without a tile.
__device__ __forceinline__ bool decode_block(int act, int b, int G, int T, int *h, int *tile) {
    const int per = 8 * ((act * G * T + 7) / 8);   // workgroups per set of `act` kv-heads
    const int p = b / per, r = b % per;
    const int x = r & 7;
    const int kv = p * act + (x & (act - 1));
    const int idx = (r >> 3) * (8 / act) + x / act;
    *tile = idx / G;
    *h = kv * G + idx % G;
    return *tile < T;
}

// kv-heads at a time (at most `want`), and the blocks of a launch of T tiles a head.  The share of an XCD is rounded up:
// an odd number of tiles of four kv-heads with seven query heads each is no multiple of 8 workgroups, and such a launch,
// dealt out in plain order, has every XCD walk all kv-heads: 65536 tokens, 8192 keys 10207 -> 8778 us a call.
inline int attn_order(int want, int H_kv) {
    int act = want;
    while (H_kv % act != 0) act >>= 1;
    return act;
}
inline int attn_grid(int act, int H_kv, int G, int T) { return H_kv / act * (8 * ((act * G * T + 7) / 8)); }

// Everything the tile bodies need beside the plan (kernel arguments, passed on by reference).
struct AttnArgs {
    const uint16_t *Q, *K, *V;
    uint16_t *O;
    int G;
    float scale_log2e;
    int64_t qs_h, qs_l, ks_h, ks_l, vs_h, vs_l, os_h, os_l;
};


template <int N> struct Int { static constexpr int value = N; };

// Which launch takes the tiles of each height class of the tile table (T_cls tiles per head).
struct AttnLaunches {
    bool wave[3];               // classes 0, 1, 2 with a launch of the kernels of attn_wave.hip
    bool middle_too, short_too; // class 1 runs in the wave launch of class 0, class 3 in that of class 2
    // Launches of k_attn_mfma<., c, .>: first tile, tiles of their own, and these with the shorter ones that joined; the
    // tiles of a launch lie behind one another in the table.
    int first[3], own[3], all[3];
    int slot[4];     // 0, 1, 2: the event of launch_attn_mfma behind which the tiles of a class are done
};
AttnLaunches attn_launches(const Prob &p, const int32_t *T_cls);

// attn_wave.hip: the height classes of the tile table that its kernels take, and T tiles of one from tile0 on
int attn_wave_classes(const Prob &p, const int32_t *T_cls);
hipError_t launch_attn_wave(const Prob &p, const PlanView &pv, const AttnArgs &a, int act, int cls, int tile0, int T, hipStream_t s);

}  // namespace dhsa
