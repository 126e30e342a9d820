// HIP kernels for gfx950: the K-way weighted reduce.  HBM-bound (K reads, one write per
// element); nothing here is a contraction, so no MFMA.
#include "kt_device.h"

namespace {

// Vector `v` of a full tile at `out`.  SYS: system-scope stores (reduce_sys), where the tile starts on 64 bytes.
template <bool SYS, typename T> __device__ __forceinline__ void st_reduced(T *out, int v, u32x4 r)
{
    if (SYS && off64(out) == 0) st_tile_wt(tile_rsrc(out, KT_TILE_BYTES), v * KT_VEC_BYTES, r);
    else st_vec(reinterpret_cast<u32x4 *>(out) + v, r);
}

// SPLIT workgroups share a 16 KiB tile, each with KT_TILE_VECS / KT_BLOCK / SPLIT vectors of all K copies per
// lane in flight together.  The kernel is bound by how well the memory system takes K read streams and
// one write stream: few bytes in flight (40-96 KB per CU), in workgroups that the dispatcher starts
// in order, so that the chip sweeps every stream over a narrow front, in part of the launches each XCD on runs of
// neighbouring pieces (reduce_run), do best (reduce_shape); persistent workgroups with the same bytes in flight
// lose 5-10 %.  Copies and output may lie at any element address; the stores are not moved to 64-byte boundaries as pack and
// unpack do: it costs more than the 3 % of a misaligned non-temporal store stream.  INT: bf16 narrowing in integer
// instructions (f32_to_bf16_int).  Whole tiles test the window's width whether it is zero or not: without
// that test between loads and stores they are 1-3 % slower.
template <typename T, int K, bool DEVW, int SPLIT, bool INT, bool SYS>
__global__ __launch_bounds__(KT_BLOCK) void kt_reduce_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                             const void *const *peer_ptrs, void *const *out_ptrs,
                                                             uint32_t order, KtWindow win, FewWeights wts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK / SPLIT;   // vectors per lane, K loads each, all in flight at once

    const unsigned piece = SPLIT == 1 ? blockIdx.x : kt_piece(order);
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket);
    T *out = reinterpret_cast<T *>(ld_table(out_ptrs + tl.bucket));
    const T *x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = reinterpret_cast<const T *>(ld_table(peer_ptrs + (int64_t)tl.bucket * K + k));
    pin(b_n, (uint64_t)out, (uint64_t)x[0], (uint64_t)x[K - 1]);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] += g.start;
    out += g.start;
    float w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] = kt_weight<DEVW>(wts, k);

    const int64_t n = g.end - g.start;
    const int nvec = (int)(n / VE);

    if (nvec == KT_TILE_VECS) {
        const int v0 = part * VPT * KT_BLOCK + tid;        // the lane's first vector in the tile
        u32x4 r[VPT][K];
#pragma unroll
        for (int u = 0; u < VPT; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) r[u][k] = ld_vec(reinterpret_cast<const u32x4 *>(x[k]) + u * KT_BLOCK + v0);
        u32x4 res[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            Acc<T> acc;
            acc.first(r[u][0], w[0]);
#pragma unroll
            for (int k = 1; k < K; ++k) acc.add(r[u][k], w[k]);
            res[u] = acc.template finish<INT>();
        }
        if (SPLIT == 1) kt_wait_store_window(win);     // large launches: the chip writes in bursts (KtWindow)
#pragma unroll
        for (int u = 0; u < VPT; ++u) st_reduced<SYS>(out, u * KT_BLOCK + v0, res[u]);
    } else {
        for (int v = part * KT_BLOCK + tid; v < nvec; v += SPLIT * KT_BLOCK) {
            u32x4 r[K];
#pragma unroll
            for (int k = 0; k < K; ++k) r[k] = ld_vec(x[k] + (int64_t)v * VE);
            Acc<T> acc;
            acc.first(r[0], w[0]);
#pragma unroll
            for (int k = 1; k < K; ++k) acc.add(r[k], w[k]);
            st_vec(out + (int64_t)v * VE, acc.finish());
        }
        // tail of a densely packed bucket (fewer than VE elements)
        const int64_t e = (int64_t)nvec * VE + tid;
        if (part == 0 && e < n) {
            float a = __fmul_rn(w[0], widen(ld_elem(x[0] + e)));
#pragma unroll
            for (int k = 1; k < K; ++k) a = __fmaf_rn(w[k], widen(ld_elem(x[k] + e)), a);
            st_elem(out + e, narrow<T>(a));
        }
    }
}

// K > 8: peers in chunks, accumulators in registers across chunks (whole tiles: sum_in_chunks; quarter tiles, SPLIT 4:
// sum_rolling).
template <typename T, bool DEVW, int SPLIT, bool SYS>
__global__ __launch_bounds__(KT_BLOCK) void kt_reduce_manyk_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                                   const void *const *peer_ptrs, void *const *out_ptrs,
                                                                   int K, uint32_t order, KtWindow win, AllWeights wts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK / SPLIT;
    const unsigned piece = SPLIT == 1 ? blockIdx.x : kt_piece(order);
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const TileGeom g = tile_geom(tl, ld_table(b_elems + tl.bucket), TILE_ELEMS);
    const int tid = threadIdx.x;
    const void *const *pp = peer_ptrs + (int64_t)g.bucket * K;
    auto peer = [&](int k) { return reinterpret_cast<const T *>(ld_table(pp + k)) + g.start; };
    T *out = reinterpret_cast<T *>(ld_table(out_ptrs + g.bucket)) + g.start;
    const int64_t n = g.end - g.start;
    const int nvec = (int)(n / VE);
    if (nvec == KT_TILE_VECS) {
        const int v0 = part * VPT * KT_BLOCK + tid;
        Acc<T> acc[VPT];
        if constexpr (VPT == 1) sum_rolling<T, DEVW>(acc[0], peer, wts, K, v0);
        else sum_in_chunks<T, VPT, DEVW>(acc, peer, wts, K, v0);
        u32x4 res[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) res[u] = acc[u].finish();
        if (SPLIT == 1) kt_wait_store_window(win);
#pragma unroll
        for (int u = 0; u < VPT; ++u) st_reduced<SYS>(out, u * KT_BLOCK + v0, res[u]);
        return;
    }
    // the ragged last tile of a bucket: one vector at a time
    for (int v = part * KT_BLOCK + tid; v < nvec; v += SPLIT * KT_BLOCK) {
        Acc<T> acc;
        acc.first(ld_vec(peer(0) + (int64_t)v * VE), kt_weight<DEVW>(wts, 0));
#pragma unroll 4
        for (int k = 1; k < K; ++k) acc.add(ld_vec(peer(k) + (int64_t)v * VE), kt_weight<DEVW>(wts, k));
        st_vec(out + (int64_t)v * VE, acc.finish());
    }
    const int64_t e = (int64_t)nvec * VE + tid;
    if (part == 0 && e < n) {
        float a = __fmul_rn(kt_weight<DEVW>(wts, 0), widen(ld_elem(peer(0) + e)));
        for (int k = 1; k < K; ++k) a = __fmaf_rn(kt_weight<DEVW>(wts, k), widen(ld_elem(peer(k) + e)), a);
        st_elem(out + e, narrow<T>(a));
    }
}

// Bytes of a copy that an XCD takes in a run (kt_order; 0: launch order): 64 KiB on shared tiles of 3 and more copies.  `packed`: the
// plan's pack is the launch before, which has just brought the buckets through the chip.  Then runs gain 2-6 % up to 32 767 tiles, whatever ran
// before the pack (pack, reduce and unpack, in us, on the buffers of the step before / after 1 GiB of other reads: K = 8 fp32 19 993
// tiles 666 -> 644 / 657 -> 636, bf16 30 055 tiles 1 029 -> 975 / 1 018 -> 958; K = 5 fp32 10 331 tiles 261 -> 253 / 258 -> 251; K = 12 fp32
// 880 -> 851 / 872 -> 843; K = 16 fp32 10 331 tiles 1-2 % slower).  A reduce of buckets that other work has displaced loses with them
// where few bytes are in flight (fp32 K = 4 19 375 tiles 250 -> 244 / 246 -> 260, K = 9 506 -> 486 / 477 -> 498; bf16 K = 5 308 -> 297 / 298 -> 305)
// but for fp32 of 7 (19 992 tiles 435 -> 430 / 414 -> 407) and bf16 of 7 and 8 (19 772 tiles 466 -> 449 / 463 -> 447).  Smaller launches
// gain in both states (uneven launches: bf16 596 tiles, K = 5 10.9 -> 10.5).  2 copies are even.  Whole tiles stay in launch order: runs
// are 1 % faster for 4 and more copies at 1 600 to 5 400 tiles and 1-5 % slower below; so do launches of 32 768 tiles and more: between
// pack and unpack runs are even there (46 696 tiles, -0.3 to 0.9 %) or slower (K = 4 107 589 tiles, the whole step 3.2 % at three
// placements of its buffers, K = 6 fp32 4.7).
template <typename T> int reduce_run(int K, int64_t nt, bool packed, const KtShape &sh)
{
    constexpr bool half = sizeof(T) == 2;
    if (sh.split == 1 || K <= 2 || nt >= 32768 || (sh.wgs && !kt_may_hold())) return 0;
    if (!half && K > 12 && nt >= 8192) return 0;
    if (nt >= (half ? 8192 : 6144) && !packed && K != 7 && !(half && K == 8)) return 0;
    return 65536;
}

// Workgroups per tile and per CU (0: as many as fit) by type, copies and tiles, where no store window
// is open.  Quarter tiles held at 2 to 5 workgroups per CU (40-96 KB in flight) against whole tiles as
// the launches had them before (two per CU for 3 to 5 copies), flat out:
//   K   fp32                                             bf16
//   2   23 912 tiles 187.7 -> 180.0 us, 14 767 even (not held; held at 3 to 5: 2-10 % slower)   60 883 tiles 487 -> 463 us
//   3   8 459 tiles 88.5 -> 87.7 us, 23 912 250.5 -> 244.2   8 682 tiles 91.6 -> 89.7 us, 18 043 191.8 -> 185.7
//       (below, shared and held: 5 416 tiles even, 2 435 3 % slower than whole tiles not held, 7 907 2.5 % faster)
//   4   36 090 tiles 485 -> 467 us, 7 052 even           11 956 tiles 156.1 -> 153.3 us, 9 081 1 % slower
//   5   7 052 tiles 113.8 -> 109.7 us, 3 563 2 % slower  18 043 tiles 291.7 -> 280.2 us, 3 526 2 % slower
//   6   42 203 tiles 832 -> 761 us, 1 957 even           42 502 tiles 837 -> 741 us, 1 528 1 % slower
//   7   5 877 tiles 128.9 -> 125.5 us, 42 203 958 -> 889,    18 043 tiles 407 -> 375 us, 2 055 even
//       4 149 1 % slower, 2 047 to 3 472 1-2 % slower
//   8   39 522 tiles 1 006 -> 920 us, 1 957 1 % slower   39 961 tiles 1 020 -> 942 us, 2 055 55.7 -> 50.5 us
//       (two per CU; three: 931 us)
// Below, a launch is a few rounds of workgroups: quarter tiles only where whole ones would leave a sixth of
// the last round idle (551 tiles of bf16: K = 8 17.8 -> 15.4 us against 16.3, K = 4 10.5 -> 8.9 against
// 9.3; 491 tiles, 96 % of two rounds: whole tiles 4-8 % faster).
// fp32 of 7 copies holds 2 behind a pack (in runs: step of 19 993 tiles 611 -> 591 us, 601 with 3), else 3 (414 -> 407 after other reads, 437 with 2).
template <typename T> KtShape reduce_shape(int K, int64_t nt, bool packed)
{
    const bool half = sizeof(T) == 2;
    switch (K) {
    case 1: break;
    case 2: if (nt >= 12288) return {4, 0}; break;
    case 3: if (nt >= 8192) return {4, 5}; break;
    case 4: if (nt >= 4096) return nt >= (half ? 12288 : 8192) ? KtShape{4, 3} : KtShape{1, 2}; break;
    case 5: if (nt >= 4096) return {4, 3}; break;
    case 6: if (nt >= 2048) return {4, 3}; break;
    case 7: if (nt >= (half ? 2048 : 4096)) return {4, !half && packed && nt >= 6144 && nt < 32768 ? 2u : 3u}; break;
    default: if (nt >= (half ? 2048 : 3072)) return {4, half ? 3u : 2u}; break;
    }
    return {K >= 2 && kt_uneven(nt) ? 4 : 1, 0};
}

// 9 and more copies outside the store window.  Up to one tile per CU, and where whole tiles would leave a sixth of
// two or three rounds idle, quarter tiles (K = 16: 29 tiles fp32 8.6 -> 5.6 us, 111 tiles bf16 14.2 -> 8.0, 577 tiles
// bf16 28.9 -> 23.7; a workgroup's serial chunks and its own table reads are a quarter); even or 2-10 % slower
// than whole tiles on full rounds.  Shared tiles in runs as above (K = 9 fp32 3 243 tiles 87.5 -> 83.1 us; K = 16 bf16 2 706
// tiles 124 -> 117).  From 2 560 tiles on quarter tiles held at two per CU (64 KB in flight; K = 12 fp32
// 2 713 tiles even, 4 149 tiles 4 % faster, 20 749 tiles 769 -> 704 us; bf16 K = 16 7 896 tiles 378 -> 361).
inline KtShape reduce_manyk_shape(int64_t nt)
{
    if (nt >= 2560) return {4, 2};
    return {nt <= 256 || (nt <= 640 && kt_uneven(nt)) ? 4 : 1, 0};
}

// System-scope stores, not waited for, where the reduced buckets are 17 to 96 MiB: the L2s have nothing to write back when the
// kernel ends, and the next call reads the buckets out of the last-level cache.  Pack, reduce and unpack together: K = 8 fp32
// 1 191 tiles 46.4 -> 45.2 us, 3 243 tiles 110.8 -> 107.7 (116.0 -> 110.6 where nine sets of buffers take turns), 5 412 tiles 182 -> 175;
// K = 4 bf16 2 706 tiles 65.8 -> 63.6; K = 12 fp32 5 412 tiles 6 % faster; ViT-B/16 bucket by bucket (1 154 tiles each) 837 -> 799.  Below,
// steps are 2-5 % slower (434 tiles), above 16 384 tiles as well (19 993 tiles, K = 8 fp32 5 %).  A reduce without a pack before it
// (`packed`, as above) gains 2-12 % up to 6 copies (K = 5 fp32 5 322 tiles 84.9 -> 76.0 us, 2 % slower where 1 GiB of other data has just been
// written); of 7 and more it is up to 10 % slower then (K = 8 fp32 5 322 tiles 126.9 -> 137.5, bf16 K = 12 5 393 tiles 186 -> 204), 4-9 %
// faster on the buffers of the call before.  Between 7 600 and 11 300 tiles the reduce alone is 2-6 % slower where a step is 4 % faster.  More
// than 8 copies from 1 536 tiles on (K = 12 fp32 1 191 tiles alone 3 % slower).
inline bool reduce_sys(int K, int64_t nt, bool packed)
{
    return K > 1 && nt >= (K > 8 ? 1536 : 1100) && nt < 6144 && (packed || K <= 6);
}

template <typename T, int K, bool DEVW>
hipError_t launch_reduce_k(const KtTile *tiles, const KtDeviceTables &tb, int64_t nt, const void *const *peers,
                           const KtWeights &w, void *const *outs, hipStream_t s)
{
    const dim3 block(KT_BLOCK);
    const int64_t *b_elems = tb.b_elems;
    if constexpr (K >= 7) {
        const KtWindow win = kt_store_window(sizeof(T) == 4 ? KT_PERIOD_14 : KT_PERIOD_12, nt, KT_WINDOW_MIN_TILES_REDUCE);
        if (win.width) {
            kt_reduce_kernel<T, K, DEVW, 1, sizeof(T) == 2, false><<<dim3((unsigned)nt), block, 0, s>>>(tiles, b_elems, peers, outs, 0u, win, FewWeights(w));
            return hipGetLastError();
        }
    }
    const KtShape sh = reduce_shape<T>(K, nt, tb.packed);
    const bool sys = reduce_sys(K, nt, tb.packed);
    const unsigned lds = kt_shape_lds(sh, 0);
    return launch_in_chunks(tiles, nt, sh.split, [&](const KtTile *t, dim3 grid) {
        const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / sh.split, reduce_run<T>(K, nt, tb.packed, sh));
#define KT_LAUNCH(SPLIT, INT, SYS) \
    kt_reduce_kernel<T, K, DEVW, SPLIT, INT, SYS><<<grid, block, lds, s>>>(t, b_elems, peers, outs, order, KtWindow{0, 0}, FewWeights(w))
        constexpr bool INT = sizeof(T) == 2 && K >= 6;
        if constexpr (K == 1) KT_LAUNCH(1, false, false);
        else if (sh.split == 1) { if (sys) KT_LAUNCH(1, false, true); else KT_LAUNCH(1, false, false); }
        else if constexpr (K <= 4) KT_LAUNCH(4, INT, false);      // shared above and below the sizes of reduce_sys only
        else { if (sys) KT_LAUNCH(4, INT, true); else KT_LAUNCH(4, INT, false); }
#undef KT_LAUNCH
    });
}

template <typename T, bool DEVW>
hipError_t launch_reduce_t(const KtDeviceTables &tb, int64_t tile0, int64_t nt, const void *const *peers, int K,
                           const KtWeights &w, void *const *outs, hipStream_t s)
{
    const KtTile *tiles = tb.tiles + tile0;
    switch (K) {
#define KT_CASE(KK) case KK: return launch_reduce_k<T, KK, DEVW>(tiles, tb, nt, peers, w, outs, s);
        KT_CASE(1) KT_CASE(2) KT_CASE(3) KT_CASE(4) KT_CASE(5) KT_CASE(6) KT_CASE(7) KT_CASE(8)
#undef KT_CASE
    }
    const KtWindow win = kt_manyk_window(sizeof(T) == 2, K, nt, KT_WINDOW_MIN_READS_REDUCE_MANYK);
    const KtShape sh = win.width ? KtShape{1, 0} : reduce_manyk_shape(nt);
    const bool sys = reduce_sys(K, nt, tb.packed);
    const unsigned lds = kt_shape_lds(sh, 0);
    return launch_in_chunks(tiles, nt, sh.split, [&](const KtTile *t, dim3 grid) {
        const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / sh.split, reduce_run<T>(K, nt, tb.packed, sh));
#define KT_LAUNCH(SPLIT, SYS) \
    kt_reduce_manyk_kernel<T, DEVW, SPLIT, SYS><<<grid, dim3(KT_BLOCK), lds, s>>>(t, tb.b_elems, peers, outs, K, order, win, AllWeights(w))
        if (sys) { if (sh.split == 1) KT_LAUNCH(1, true); else KT_LAUNCH(4, true); }
        else { if (sh.split == 1) KT_LAUNCH(1, false); else KT_LAUNCH(4, false); }
#undef KT_LAUNCH
    });
}

}  // namespace

int kt_launch_reduce(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0, int64_t ntiles,
                     const void *const *d_peer_ptrs, int K, const KtWeights &w, void *const *d_out_ptrs,
                     void *stream)
{
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // weights by value (the usual case) and weights read from device memory are separate instantiations
    if (dt == KT_F32)
        return (int)(w.dev ? launch_reduce_t<float, true>(tb, tile0, ntiles, d_peer_ptrs, K, w, d_out_ptrs, s)
                           : launch_reduce_t<float, false>(tb, tile0, ntiles, d_peer_ptrs, K, w, d_out_ptrs, s));
    return (int)(w.dev ? launch_reduce_t<uint16_t, true>(tb, tile0, ntiles, d_peer_ptrs, K, w, d_out_ptrs, s)
                       : launch_reduce_t<uint16_t, false>(tb, tile0, ntiles, d_peer_ptrs, K, w, d_out_ptrs, s));
}
