// Internal structures shared by the host plan code, the C ABI and the kernels.
#ifndef KT_INTERNAL_H
#define KT_INTERNAL_H

#include <stdint.h>
#include <vector>

#include "kt.h"

// A tile is a fixed-size slice of one bucket; one workgroup processes one tile.
#ifndef KT_TILE_BYTES
#define KT_TILE_BYTES 16384
#endif
#define KT_VEC_BYTES 16
#define KT_TILE_VECS (KT_TILE_BYTES / KT_VEC_BYTES)
#define KT_BLOCK 256
// Mixed tiles holding at most this many tensors stage their slice of the
// tensor table in LDS; larger ones search the table in global memory.
#ifndef KT_LDS_TENSORS
#define KT_LDS_TENSORS 512
#endif

// Per-tile record (device table).  `nt == 0` marks a solid tile: tensor `t0`
// covers every element of the tile and the tile is a whole number of 16-byte
// vectors.  Otherwise tensors t0 .. t0+nt-1 are the ones that may own
// elements of the tile (the rest is padding).
struct KtTile {
    int32_t bucket;
    uint32_t tile_in_bucket;
    int32_t t0;
    int32_t nt;
};

struct KtHostPlan {
    kt_dtype dt;
    int elem_size;
    int64_t cap_bytes;
    int align_bytes;
    int64_t tile_elems;
    // per tensor
    std::vector<int64_t> t_numel, t_off;
    std::vector<int32_t> t_bucket;
    // per bucket
    std::vector<int64_t> b_elems;
    std::vector<int32_t> b_first, b_count;
    std::vector<int64_t> b_tile0;      // first tile of each bucket, nb+1 entries
    std::vector<KtTile> tiles;
};

// Builds the layout and the tile table.  Returns KT_OK or an error with `msg` set.
kt_status kt_build_host_plan(const int64_t *numel, int T, kt_dtype dt,
                             int64_t cap_bytes, int align_bytes,
                             KtHostPlan &hp, const char **msg);

// Device-side view of the plan tables plus the per-call pointer tables.
struct KtDeviceTables {
    const KtTile *tiles;
    const int64_t *t_off;
    const int64_t *t_numel;
    const int64_t *b_elems;
    bool packed = false;    // the launch before was this plan's pack (kt_launch_reduce)
};

// Launchers (defined next to their kernels in the .hip files).  `tile0`/`ntiles` select a contiguous tile range.
// All return a hipError_t cast to int.
int kt_launch_pack(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0,
                   int64_t ntiles, const void *const *d_tensor_ptrs,
                   void *const *d_bucket_ptrs, void *stream);
int kt_launch_unpack(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0,
                     int64_t ntiles, const void *const *d_bucket_ptrs,
                     float scale, void *const *d_tensor_ptrs, void *stream);
// Store window of the read-dominated kernels (reduce, fused pass, one-pass SGD of many copies) on large launches: every wave
// holds its finished results back until the device-wide constant-rate clock, masked to a period
// of 12 to 24 us, is inside the first `width` ticks, so that the whole chip alternates between
// reading and writing instead of sprinkling one written line among eight read ones.  Measured on
// 8 peers: 72-73 % -> 77-78 % of 8 TB/s, the same within a point for periods of 10-14 us, and a steep
// loss once the period exceeds the time the resident workgroups need for their loads (about 14-19 us
// at K = 8; the 14 us period leaves 0-5 us, the 12 us one 2-7), which is why it is used only where
// that time is known to be longer (7 and more copies, many tiles).  Launches below the limits here, all of up to 6
// copies, and those of 9 (bf16: and 10) do better with few workgroups per CU that share tiles (KtShape).
// width == 0: no window; the fused pass of up to 8 copies then finds the order of its pieces (kt_order) in `period`.
struct KtWindow {
    uint32_t period;  // clock ticks
    uint32_t width;   // ticks at the start of each period in which stores are issued
};
// The period in nanoseconds and the share of it, in per cent, in which stores are issued.  The best
// period grows with the time that the resident workgroups need for their loads, hence with the copies:
//   up to 8    12 us / 10 %; the fp32 reduce and the fp32 fused pass of 8 copies 14 us / 6 % (K = 8, 65 536 tiles 1.59 -> 1.57 ms and
//              1.60 -> 1.57 ms against 12 us; bf16 fused 1.3B set 3.86 ms, 4.01 with 14 us)
//   more, fp32 14 us up to 12 copies, 18 us up to 15, 24 us above (reduce and fused pass, 20 000 tiles: K = 12 692 us
//              against 703 with 12 us, 698 with 18; K = 15 800 against 817 with 14; K = 16 889 against 923;
//              K = 20 1 028 against 1 058); one-pass SGD, which reads p and v as well, as two copies more
//   more, bf16 12 us / 10 % up to 13 copies, 14 us up to 16, 18 us above (chunks of 6 copies; fused pass K = 12
//              664 us, 756 with 14; K = 15 793 against 818 with 12, 936 with 18; K = 20 1 037 against 1 054 with 14)
struct KtPeriod {
    int ns, pct;
};
constexpr KtPeriod KT_PERIOD_12{12000, 10}, KT_PERIOD_14{14000, 6}, KT_PERIOD_18{18000, 6}, KT_PERIOD_24{24000, 6};
inline KtPeriod kt_manyk_period(bool half, int K)
{
    if (half) return K < 14 ? KT_PERIOD_12 : K <= 16 ? KT_PERIOD_14 : KT_PERIOD_18;
    return K <= 12 ? KT_PERIOD_14 : K < 16 ? KT_PERIOD_18 : KT_PERIOD_24;
}
// The window for a launch of `ntiles` tiles on the current device (host); none below `min_tiles` tiles: a
// launch of a few generations of workgroups only pays for the waits of its first and last one.
// KT_STORE_WINDOW_NS sets one period for all (0: no windows).
KtWindow kt_store_window(KtPeriod period, int64_t ntiles, int64_t min_tiles);
// Smallest launches that use the window, in tiles read (tiles x copies) or, for the reduce of up to
// 8 copies, in tiles.  The fused pass of more copies gains from 65 536 tiles read on
// (K = 16: 8 192 tiles 399 -> 371 us, 4 096 tiles 212 -> 199 us), the fp32 one of 8 is even with quarter
// tiles from 10 331 to 20 623 tiles and better above (39 522 tiles 923 us, 935), the bf16 one from 131 072 on.  The reduce of 7 and 8 copies
// is 6-9 % slower with the window at 40 000 tiles and 2-5 % faster at 85 000 (K = 8, fp32 1 984 us against
// 2 066, bf16 2 016 against 2 075).  With more copies, from 262 144
// tiles read on, the reduce alone gains 2-8 % over held quarter tiles (fp32 K = 12, 29 439 tiles 1 046 -> 1 008 us; K = 16, 20 749
// tiles 956 -> 915; K = 24, 29 439 tiles 2 048 -> 1 894; bf16 K = 16, 20 449 tiles 946 -> 907), bf16 of 12 copies loses 1-2 % (30 030
// tiles 995 -> 1 012).  Inside the step, where the reduce displaces what pack wrote last, the window costs up to 6 % below 1 GiB
// per copy and 24 copies (fp32 K = 16, 16 574 tiles 929 -> 983 us, 39 661 tiles 2 204 -> 2 249; bf16 K = 12, 39 712 tiles
// 1 681 -> 1 791, K = 16, 20 449 tiles 1 143 -> 1 168, 30 030 even) and gains 1-2 % there (K = 24, 39 661 tiles 3 106 -> 3 072,
// bf16 3 170 -> 3 103); it is even with or faster than the whole tiles without a window that the limit was set against.
#ifndef KT_WINDOW_MIN_READS_FUSED
#define KT_WINDOW_MIN_READS_FUSED 65536
#endif
#ifndef KT_WINDOW_MIN_TILES_FUSED
#define KT_WINDOW_MIN_TILES_FUSED 16384
#endif
#ifndef KT_WINDOW_MIN_TILES_REDUCE
#define KT_WINDOW_MIN_TILES_REDUCE 65536
#endif
#ifndef KT_WINDOW_MIN_READS_REDUCE_MANYK
#define KT_WINDOW_MIN_READS_REDUCE_MANYK 262144
#endif

// The window of the reduce and the fused pass of 9 and more copies, from `min_reads` tiles read on.  9 copies (bf16: and
// 10) do better with held quarter tiles (20 000 tiles, K = 9: bf16 fused pass 527 us against 616, reduce 520 against 554; fp32
// 528 against 539, 508 against 550).
inline KtWindow kt_manyk_window(bool half, int K, int64_t ntiles, int64_t min_reads)
{
    if (K < (half ? 11 : 10)) return KtWindow{0, 0};
    return kt_store_window(kt_manyk_period(half, K), ntiles, (min_reads + K - 1) / K);
}

// LDS to ask for beyond a kernel's own `own` bytes, so that `wgs` workgroups share a CU: the smallest
// request of which one more does not fit.  A CU has 160 KiB and gives it out in granules of 1 280 bytes
// (workgroups counted while they run: 53 760 bytes hold 3, 54 272 hold 2; the runtime's occupancy
// query rounds to less and says 3 for both).
constexpr unsigned KT_CU_LDS = 163840, KT_LDS_GRANULE = 1280;
constexpr unsigned kt_hold_lds(unsigned wgs, unsigned own)
{
    return (KT_CU_LDS / (wgs + 1) / KT_LDS_GRANULE + 1) * KT_LDS_GRANULE - own;
}
constexpr bool kt_holds(unsigned wgs)
{
    const unsigned bytes = kt_hold_lds(wgs, 0);
    return bytes % KT_LDS_GRANULE == 0 && bytes <= 65536 && KT_CU_LDS / bytes == wgs;
}
static_assert(kt_holds(2) && kt_holds(3) && kt_holds(4) && kt_holds(5) && kt_holds(6), "the counts that launches ask for");

// false where the caller shares the GPU (KT_STORE_WINDOW_NS=0): held workgroups keep the LDS of every
// CU from kernels that run beside them.
bool kt_may_hold();

// How a launch of the reduce or the fused pass is laid out: workgroups that share a tile, and
// workgroups per CU that it is held to by asking for LDS (0: as many as fit).  `own`: the kernel's own LDS.
struct KtShape {
    int split;
    unsigned wgs;
};
inline unsigned kt_shape_lds(const KtShape &s, unsigned own) { return s.wgs && kt_may_hold() ? kt_hold_lds(s.wgs, own) : 0u; }

// Launches of two to four rounds over the 256 CUs, a tile each, whose last round is more than a sixth empty.
inline bool kt_uneven(int64_t ntiles) { return ntiles > 256 && ntiles < 1024 && 5 * ((ntiles + 255) / 256 * 256) > 6 * ntiles; }

// The K weights of a launch travel in the kernel-argument block (`w`), unless
// `dev` is set: then the kernels read them from that device array when they
// run (kt_plan_set_weights), so that a recorded graph follows later updates.
struct KtWeights {
    float w[KT_MAX_PEERS];
    const float *dev;
};
int kt_launch_reduce(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0,
                     int64_t ntiles, const void *const *d_peer_ptrs, int K,
                     const KtWeights &w, void *const *d_out_ptrs, void *stream);
int kt_launch_fused(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0,
                    int64_t ntiles, const void *const *d_local_ptrs,
                    const void *const *d_peer_ptrs, int K, const KtWeights &w,
                    float scale, void *const *d_out_ptrs, void *stream);

struct KtSgd {
    float scale, lr, mu, wd;
    int first;
    const float *dev;   // non-NULL: {scale, lr, mu, wd} are read from these 4 device floats when the kernel runs
};
int kt_launch_unpack_sgd(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0,
                         int64_t ntiles, const void *const *d_bucket_ptrs,
                         void *const *d_param_ptrs, void *const *d_mom_ptrs,
                         void *const *d_model_ptrs /* NULL: no bf16 model copy */,
                         const KtSgd &a, void *stream);

// The single pass from K gradient copies to updated parameters (kt_fused_sgd.hip).
int kt_launch_fused_sgd(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0,
                        int64_t ntiles, const void *const *d_local_ptrs,
                        const void *const *d_peer_ptrs, int K, const KtWeights &w,
                        void *const *d_param_ptrs, void *const *d_mom_ptrs,
                        void *const *d_model_ptrs /* NULL: no bf16 model copy */,
                        const KtSgd &a, void *stream);

// ---- shared between the C ABI (kt_api.cpp) and the entry point that
// allocates nothing (kt_static.hip) ------------------------------------------

void kt_set_error(const char *fmt, ...);

// The immutable host tables of a plan and a number that identifies the plan
// for the lifetime of the process (never reused).
const KtHostPlan &kt_plan_host(const kt_plan *p);
uint64_t kt_plan_serial(const kt_plan *p);

// Argument checks of the fused single pass and its pointer table
// [local tensors T | output tensors T | peers nb*(K-1)] written to `vals`
// (2T + nb*(K-1) entries).  *ntiles == 0 on return means nothing to do.
kt_status kt_fused_prepare(const kt_plan *p, int bucket, const void *const *local_tensor_ptrs,
                           const void *const *peer_bufs, int K, const float *weights,
                           void *const *out_tensor_ptrs, const char *who, std::vector<uint64_t> &vals,
                           KtWeights *w, int64_t *tile0, int64_t *ntiles);

#endif
