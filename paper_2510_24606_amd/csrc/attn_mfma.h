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
// each XCD has its own L2.  act = 2^order kv-heads (1, 2, 4 or 8) are worked on at a
// time, each by 8 / act XCDs: act = 8 gives every XCD its own kv-head (best L2
// reuse of the K/V slabs), smaller values keep fewer K/V slabs live at once
// (they then fit the memory-side cache).  Within a kv-head the query heads of
// the group are innermost; *tile is the tile's position in the order of issue
// (0 = first), which the kernel maps to a row tile.  False: a block that only
// makes the share of every XCD equal, without a tile.  order < 0: all -order kv-heads
// at a time, whatever XCD their workgroups get.
__device__ __forceinline__ bool decode_block(int order, unsigned b, unsigned G, unsigned T, int *h, int *tile) {
    unsigned kv, idx;
    if (order < 0) {
        kv = b % (unsigned)-order;
        idx = b / (unsigned)-order;
    } else {
        const unsigned per = ((G << order) * T + 7u) & ~7u;   // workgroups per set of `act` kv-heads
        const unsigned p = b / per, r = b % per, x = r & 7u;
        kv = (p << order) + (x & ((1u << order) - 1u));
        idx = ((r >> 3) << (3 - order)) + (x >> order);
    }
    *tile = (int)(idx / G);
    *h = (int)(kv * G + idx % G);
    return idx < G * T;
}

// The order of a launch of T tiles a head (at most 2^want kv-heads at a time), and its blocks.  The share of an XCD is rounded up:
// an odd number of tiles of four kv-heads with seven query heads each is no multiple of 8 workgroups, and such a launch,
// dealt out head by head, has every XCD walk all kv-heads: 65536 tokens, 8192 keys 10207 -> 8778 us a call where the numbers
// of all its launches are odd, 9350 -> 8718 where those of some are.
// Where some kv-heads would have to wait for others (numbers that are no power of two, nor a multiple of 2^want), each
// begins with long lists again, and the chip is left to the last one's.  That costs more than the L2 gives while a head's K
// and V are a small part of it anyway, or there are few rounds of workgroups.  Attention in us, kv-heads x query heads of
// each, one kv-head or two at a time -> all: 20 x 1 of 3000 tokens, heads of 64, all keys 87.0 -> 71.5; 5 x 4 of 3500, heads
// of 128, all keys 161 -> 142; 3 x 1 of 8191, heads of 128 (411 workgroups), 511 keys 27.4 -> 24.0; 6 x 1 of 4500, heads of
// 64 (714), 1125 keys 27.1 -> 23.9; on the other side 7 x 4 of 4096, heads of 128 (3108), 256 keys 71.7 -> 74.8, of 8191
// (4032), 511 keys 159 -> 172; 10 x 4 of 12000 (8520) 392 -> 429.
inline int attn_order(int want, const Prob &p, int T) {
    int order = want;
    while (p.H_kv % (1 << order) != 0) --order;
    const bool wait = order < want && p.H_kv != 1 << order;
    return wait && (p.L < 4096 || (int64_t)p.H_q * T <= 1536) ? -p.H_kv : order;
}
inline int attn_grid(int order, const Prob &p, int T) {
    return order < 0 ? p.H_q * T : (p.H_kv >> order) * ((((p.G << order) * T) + 7) & ~7);
}

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
hipError_t launch_attn_wave(const Prob &p, const PlanView &pv, const AttnArgs &a, int want, int cls, int tile0, int T, hipStream_t s);

}  // namespace dhsa
