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
// (0 = first), which the kernel maps to a row tile.  act = 0: plain order.
__device__ __forceinline__ void decode_block(int act, int b, int H_q, int G, int T1, int *h, int *tile) {
    if (act > 0) {
        const int per = act * G * T1;          // workgroups per set of `act` kv-heads
        const int p = b / per, r = b % per;
        const int x = r & 7;
        const int kv = p * act + (x & (act - 1));
        const int idx = (r >> 3) * (8 / act) + x / act;
        *tile = idx / G;
        *h = kv * G + idx % G;
        return;
    }
    *tile = b / H_q;
    *h = b % H_q;
}

// act must divide H_kv and act * G * T1 must be a multiple of 8 for the mapping above
inline int attn_order(int want, int H_kv, int G, int T1) {
    for (int act = want; act >= 1; act >>= 1)
        if (H_kv % act == 0 && (act * G * T1) % 8 == 0) return act;
    return 0;
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
