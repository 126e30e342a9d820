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
// in order, so that the chip sweeps every stream over a narrow front, each XCD on runs of neighbouring
// pieces (kt_piece), do best (reduce_shape); persistent workgroups with the same bytes in flight lose 5-10 %.  Copies and output may lie at any element
// address; the stores are not moved to 64-byte boundaries as pack and unpack do: it costs more
// than the 3 % of a misaligned non-temporal store stream.  INT: bf16 narrowing in integer instructions
// (f32_to_bf16_int).  Whole tiles test the window's width whether it is zero or not: without
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

// Shared tiles go in runs of 64 KiB per XCD, of 128 KiB up to 3 copies (kt_order), which is 2-6 % faster than launch order
// (K = 4 fp32 19 993 tiles 259 -> 248 us; K = 5 fp32 315 -> 299; K = 6 bf16 31 528 tiles
// 585 -> 553; K = 7 bf16 698 -> 647; K = 8 fp32 19 993 tiles 480 -> 460, bf16 31 528 tiles 790 -> 742; uneven launches:
// bf16 596 tiles, K = 5 10.9 -> 10.5).  With runs 3 copies do best with 4 workgroups per CU (fp32 19 993 tiles 201 us with 5,
// 199 with 4; bf16 31 528 tiles 322, 318) and fp32 of 7 copies with 2 from 6 144 tiles on (19 993 tiles 424 us with 3, 410
// with 2; 5 412 tiles even; 6 copies alone 351 and 348 us, but a step of them 2 % slower than before with 2).  Whole tiles stay in launch order: runs are 1 % faster for 4 and more copies at
// 1 600 to 5 400 tiles and 1-5 % slower below; so do launches of 32 768 tiles and more: alone they would gain 3-5 %, but between pack and unpack
// runs are even there (46 696 tiles, -0.3 to 0.9 %; 38 449 tiles, K = 7 -1.4, K = 4 1.4) or slower (K = 4 107 589 tiles, the whole step 3.2 % at three
// placements of its buffers, K = 6 fp32 4.7).
inline bool reduce_runs(int64_t nt) { return nt < 32768; }

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
template <typename T> KtShape reduce_shape(int K, int64_t nt)
{
    const bool half = sizeof(T) == 2;
    switch (K) {
    case 1: break;
    case 2: if (nt >= 12288) return {4, 0}; break;
    case 3: if (nt >= 8192) return {4, reduce_runs(nt) ? 4u : 5u}; break;
    case 4: if (nt >= 4096) return nt >= (half ? 12288 : 8192) ? KtShape{4, 3} : KtShape{1, 2}; break;
    case 5: if (nt >= 4096) return {4, 3}; break;
    case 6: if (nt >= 2048) return {4, 3}; break;
    case 7: if (nt >= (half ? 2048 : 4096)) return {4, half || nt < 6144 || !reduce_runs(nt) ? 3u : 2u}; break;
    default: if (nt >= (half ? 2048 : 3072)) return {4, half ? 3u : 2u}; break;
    }
    return {K >= 2 && kt_uneven(nt) ? 4 : 1, 0};
}

// 9 and more copies outside the store window.  Up to one tile per CU, and where whole tiles would leave a sixth of
// two or three rounds idle, quarter tiles (K = 16: 29 tiles fp32 8.6 -> 5.6 us, 111 tiles bf16 14.2 -> 8.0, 577 tiles
// bf16 28.9 -> 23.7; a workgroup's serial chunks and its own table reads are a quarter); even or 2-10 % slower
// than whole tiles on full rounds.  Shared tiles in runs of 64 KiB per XCD (K = 9 fp32 3 243 tiles 87.5 -> 83.1 us, bf16 31 528
// tiles 882 -> 808; K = 16 bf16 2 706 tiles 124 -> 117).  From 2 560 tiles on quarter tiles held at two per CU (64 KB in flight; K = 12 fp32
// 2 713 tiles even, 4 149 tiles 4 % faster, 20 749 tiles 769 -> 704 us; bf16 K = 16 7 896 tiles 378 -> 361).
inline KtShape reduce_manyk_shape(int64_t nt)
{
    if (nt >= 2560) return {4, 2};
    return {nt <= 256 || (nt <= 640 && kt_uneven(nt)) ? 4 : 1, 0};
}

// System-scope stores, not waited for, where the reduced buckets are 17 to 96 MiB: the L2s have nothing to write back when the
// kernel ends, and the next call reads the buckets out of the last-level cache.  Pack, reduce and unpack together: K = 8 fp32
// 1 191 tiles 46.4 -> 45.2 us, 3 243 tiles 110.8 -> 107.7 (116.0 -> 110.6 where nine sets of buffers take turns), 5 412 tiles 182 -> 175;
// K = 4 bf16 2 706 tiles 65.8 -> 63.6; K = 12 fp32 5 412 tiles 6 % faster; ViT-B/16 bucket by bucket (1 154 tiles each) 837 -> 799.  Alone, in place
// over the first copy, 1 950 to 5 600 tiles 2-8 % faster, 1 200 even.  Below, steps are 2-5 % slower (434 tiles), above 16 384 tiles as well
// (19 993 tiles, K = 8 fp32 5 %); between 7 600 and 11 300 the reduce alone is 2-6 % slower where a step is 4 % faster, as is one of 5 and
// more copies at 1 038 tiles (2 %; a step 2 % faster).  More than 8 copies from 1 536 tiles on (K = 12 fp32 1 191 tiles alone 3 % slower).
inline bool reduce_sys(int K, int64_t nt) { return K > 1 && nt >= (K > 8 ? 1536 : 1100) && nt < 6144; }

template <typename T, int K, bool DEVW>
hipError_t launch_reduce_k(const KtTile *tiles, const int64_t *b_elems, int64_t nt, const void *const *peers,
                           const KtWeights &w, void *const *outs, hipStream_t s)
{
    const dim3 block(KT_BLOCK);
    if constexpr (K >= 7) {
        const KtWindow win = kt_store_window(sizeof(T) == 4 ? KT_PERIOD_14 : KT_PERIOD_12, nt, KT_WINDOW_MIN_TILES_REDUCE);
        if (win.width) {
            kt_reduce_kernel<T, K, DEVW, 1, sizeof(T) == 2, false><<<dim3((unsigned)nt), block, 0, s>>>(tiles, b_elems, peers, outs, 0u, win, FewWeights(w));
            return hipGetLastError();
        }
    }
    const KtShape sh = reduce_shape<T>(K, nt);
    const bool sys = reduce_sys(K, nt);
    const unsigned lds = kt_shape_lds(sh, 0);
    return launch_in_chunks(tiles, nt, sh.split, [&](const KtTile *t, dim3 grid) {
        const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / sh.split, sh.split == 1 || !reduce_runs(nt) ? 0 : K <= 3 ? 131072 : 65536);
#define KT_LAUNCH(SPLIT, INT, SYS) \
    kt_reduce_kernel<T, K, DEVW, SPLIT, INT, SYS><<<grid, block, lds, s>>>(t, b_elems, peers, outs, order, KtWindow{0, 0}, FewWeights(w))
        constexpr bool INT = sizeof(T) == 2 && K >= 6;
        if constexpr (K == 1) KT_LAUNCH(1, false, false);
        else if (sys) { if (sh.split == 1) KT_LAUNCH(1, false, true); else KT_LAUNCH(4, INT, true); }
        else { if (sh.split == 1) KT_LAUNCH(1, false, false); else KT_LAUNCH(4, INT, false); }
#undef KT_LAUNCH
    });
}

template <typename T, bool DEVW>
hipError_t launch_reduce_t(const KtDeviceTables &tb, int64_t tile0, int64_t nt, const void *const *peers, int K,
                           const KtWeights &w, void *const *outs, hipStream_t s)
{
    const KtTile *tiles = tb.tiles + tile0;
    switch (K) {
#define KT_CASE(KK) case KK: return launch_reduce_k<T, KK, DEVW>(tiles, tb.b_elems, nt, peers, w, outs, s);
        KT_CASE(1) KT_CASE(2) KT_CASE(3) KT_CASE(4) KT_CASE(5) KT_CASE(6) KT_CASE(7) KT_CASE(8)
#undef KT_CASE
    }
    const KtWindow win = kt_manyk_window(sizeof(T) == 2, K, nt, KT_WINDOW_MIN_READS_REDUCE_MANYK);
    const KtShape sh = win.width ? KtShape{1, 0} : reduce_manyk_shape(nt);
    const bool sys = reduce_sys(K, nt);
    const unsigned lds = kt_shape_lds(sh, 0);
    return launch_in_chunks(tiles, nt, sh.split, [&](const KtTile *t, dim3 grid) {
        const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / sh.split, sh.split == 1 || !reduce_runs(nt) ? 0 : 65536);
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
