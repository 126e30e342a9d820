// HIP kernels for gfx950: the fused single pass (pack + reduce + unpack-scale in one kernel).
#include "kt_device.h"

namespace {

// ---- fused single pass: tensors + peer buckets -> scaled tensors ------------
// out_t[i] = scale * round(sum_k w_k x_k), where x_0 is read straight from the
// local gradient tensor and x_1..x_{K-1} from the peer buckets.  The rounding
// sequence equals pack -> reduce -> unpack-scale (sum rounded to the storage
// type, then one multiplication), so the results are bit-identical to the
// chained path while moving (K+1) instead of (K+5) element sizes per element.
//
// SPLIT workgroups per 16 KiB tile (fused_shape); bound, like the reduce, by how well the memory
// system takes K reads and one write.  Tensors and buckets may lie at any
// element address (stores as in the reduce, at the tile's own offsets).  77.2 M fp32 elements, K = 4, odd
// tensor sizes in the dense layout: 652 us with one element per lane, which every
// dense plan and misaligned bucket took before, against 265 us.

// One element: tensor element `r` of source/destination p, ptr2; peers at element e of the tile.
template <typename T, int K>
__device__ __forceinline__ void fused_elem(const T *src, T *dst, const T *const *x, int64_t e, const float *w, float scale)
{
    float a = __fmul_rn(w[0], widen(ld_elem(src)));
#pragma unroll
    for (int k = 1; k < K; ++k) a = __fmaf_rn(w[k], widen(ld_elem(x[k - 1] + e)), a);
    st_elem(dst, scale_elem(narrow<T>(a), scale));
}

// Mixed tile of the fused pass: per vector, peer 0 comes from the owning tensor
// (tv.ptr = local gradients), the result goes to the same position of tv.ptr2.
// Vectors are taken MB at a time per lane, in two phases, so that the loads of
// all of them are in flight together: (1) find each vector's owner in the staged
// table and issue its K loads, (2) combine and store.  The elements of vectors that
// are not wholly inside one tensor go one per lane (each_cut_elem).
template <typename T, int K, typename V>
__device__ __forceinline__ void fused_mixed(const V &tv, int nt, const TileGeom &g,
                                            const T *const *x, const float *w, float scale, int part, int parts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int MB = K <= 4 ? 4 : 2;
    const int nvec = (int)((g.end - g.start + VE - 1) / VE);
#pragma unroll 1
    for (int v0 = part * KT_BLOCK + threadIdx.x; v0 < nvec; v0 += MB * parts * KT_BLOCK) {
        u32x4 r[MB][K];
        uintptr_t where[MB];      // destination of a whole vector, 0 = none
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int v = v0 + j * parts * KT_BLOCK;
            where[j] = 0;
            if (v < nvec) {
                const int64_t e0 = g.start + (int64_t)v * VE;
                const int i = find_owner_v(tv, nt, e0);
                const int64_t rr = i >= 0 ? e0 - tv.off[i] : -1;
                if (rr >= 0 && rr + VE <= tv.numel[i]) {
                    r[j][0] = ld_vec(reinterpret_cast<const T *>(tv.ptr[i]) + rr);
#pragma unroll
                    for (int k = 1; k < K; ++k) r[j][k] = ld_vec(reinterpret_cast<const u32x4 *>(x[k - 1]) + v);
                    where[j] = tv.ptr2[i] + (uintptr_t)rr * sizeof(T);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            if (where[j]) {
                Acc<T> acc;
                acc.first(r[j][0], w[0]);
#pragma unroll
                for (int k = 1; k < K; ++k) acc.add(r[j][k], w[k]);
                st_vec(reinterpret_cast<void *>(where[j]), scale_vec<T>(acc.finish(), scale));
            }
        }
    }
    each_cut_elem<VE>(tv, nt, g.start, (int)(g.end - g.start), part * KT_BLOCK + threadIdx.x, parts * KT_BLOCK, [&](int i, int64_t r, int e) {
        fused_elem<T, K>(reinterpret_cast<const T *>(tv.ptr[i]) + r, reinterpret_cast<T *>(tv.ptr2[i]) + r, x, e, w, scale);
    });
}

template <typename T, int K, bool DEVW, int SPLIT, bool INT>
__global__ __launch_bounds__(KT_BLOCK) void kt_fused_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                            const int64_t *t_offs, const void *const *local_ptrs,
                                                            const void *const *peer_ptrs, void *const *out_ptrs,
                                                            float scale, KtWindow win,
                                                            const int64_t *t_numel, FewWeights wts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK / SPLIT;
    constexpr int KP = K > 1 ? K - 1 : 1;
    __shared__ LdsTable lds;

    // launches without a window have their order in the place of its period (one argument more would no longer arrive in registers)
    const unsigned piece = SPLIT > 1 || K == 4 || K == 5 ? kt_piece(win.period) : blockIdx.x;      // fused_run
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    const T *src = reinterpret_cast<const T *>(ld_table(local_ptrs + tl.t0));
    T *dst = reinterpret_cast<T *>(ld_table(out_ptrs + tl.t0));
    const T *x[KP];   // peers 1..K-1
#pragma unroll
    for (int k = 1; k < K; ++k)
        x[k - 1] = reinterpret_cast<const T *>(ld_table(peer_ptrs + (int64_t)tl.bucket * (K - 1) + (k - 1)));
    pin(b_n, t_off, (uint64_t)src, (uint64_t)dst);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 1; k < K; ++k) x[k - 1] += g.start;      // at the tile start
    float w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] = kt_weight<DEVW>(wts, k);

    if (tl.nt == 0) {
        src += g.start - t_off;
        dst += g.start - t_off;
        const int nvec = (int)((g.end - g.start) / VE);
        if (nvec == KT_TILE_VECS) {
            const int v0 = part * VPT * KT_BLOCK + tid;        // the lane's first vector in the tile
            u32x4 r[VPT][K];
#pragma unroll
            for (int u = 0; u < VPT; ++u) {
                r[u][0] = ld_vec(reinterpret_cast<const u32x4 *>(src) + u * KT_BLOCK + v0);
#pragma unroll
                for (int k = 1; k < K; ++k)
                    r[u][k] = ld_vec(reinterpret_cast<const u32x4 *>(x[k - 1]) + u * KT_BLOCK + v0);
            }
            u32x4 res[VPT];
#pragma unroll
            for (int u = 0; u < VPT; ++u) {
                Acc<T> acc;
                acc.first(r[u][0], w[0]);
#pragma unroll
                for (int k = 1; k < K; ++k) acc.add(r[u][k], w[k]);
                res[u] = scale_vec<T, INT>(acc.template finish<INT>(), scale);
            }
            if (SPLIT == 1) kt_wait_store_window(win);     // large launches: the chip writes in bursts (KtWindow)
#pragma unroll
            for (int u = 0; u < VPT; ++u) st_vec(reinterpret_cast<u32x4 *>(dst) + u * KT_BLOCK + v0, res[u]);
        } else {
#pragma unroll 1
            for (int v = part * KT_BLOCK + tid; v < nvec; v += SPLIT * KT_BLOCK) {
                Acc<T> acc;
                acc.first(ld_vec(reinterpret_cast<const u32x4 *>(src) + v), w[0]);
#pragma unroll
                for (int k = 1; k < K; ++k) acc.add(ld_vec(reinterpret_cast<const u32x4 *>(x[k - 1]) + v), w[k]);
                st_vec(reinterpret_cast<u32x4 *>(dst) + v, scale_vec<T>(acc.finish(), scale));
            }
        }
        return;
    }

    // mixed tile: stage (offset, size, source, destination) of its tensors in LDS
    const void *const *op = reinterpret_cast<const void *const *>(out_ptrs);
    if (tl.nt <= KT_LDS_TENSORS) {
        const LdsView tv = stage_lds(lds, t_offs, t_numel, local_ptrs, op, tl.t0, tl.nt);
        fused_mixed<T, K>(tv, tl.nt, g, x, w, scale, part, SPLIT);
    } else {
        const GlobalView tv = global_view(t_offs, t_numel, local_ptrs, op, tl.t0);
        fused_mixed<T, K>(tv, tl.nt, g, x, w, scale, part, SPLIT);
    }
}

// K > 8: full solid tiles take the peers in chunks with the accumulators in
// registers (sum_in_chunks, quarter tiles sum_rolling; peer 0 is the local tensor); every other tile goes
// vector by vector with a loop over the peers.
template <typename T, bool DEVW, typename V>
__device__ __forceinline__ void fused_mixed_manyk(const V &tv, int nt, const TileGeom &g,
                                                  const void *const *pp, int K, const AllWeights &wts, float scale,
                                                  int part, int parts)
{
    constexpr int VE = Elem<T>::VE;
    const int nvec = (int)((g.end - g.start + VE - 1) / VE);
#pragma unroll 1
    for (int v = part * KT_BLOCK + threadIdx.x; v < nvec; v += parts * KT_BLOCK) {
        const int64_t e0 = g.start + (int64_t)v * VE;
        const int i = find_owner_v(tv, nt, e0);
        const int64_t r = i >= 0 ? e0 - tv.off[i] : -1;
        if (r >= 0 && r + VE <= tv.numel[i]) {
            Acc<T> acc;
            acc.first(ld_vec(reinterpret_cast<const T *>(tv.ptr[i]) + r), kt_weight<DEVW>(wts, 0));
#pragma unroll 4
            for (int k = 1; k < K; ++k)
                acc.add(ld_vec(reinterpret_cast<const T *>(ld_table(pp + k - 1)) + e0), kt_weight<DEVW>(wts, k));
            st_vec(reinterpret_cast<T *>(tv.ptr2[i]) + r, scale_vec<T>(acc.finish(), scale));
        }
    }
    each_cut_elem<VE>(tv, nt, g.start, (int)(g.end - g.start), part * KT_BLOCK + threadIdx.x, parts * KT_BLOCK, [&](int i, int64_t r, int e) {
        float a = __fmul_rn(kt_weight<DEVW>(wts, 0), widen(ld_elem(reinterpret_cast<const T *>(tv.ptr[i]) + r)));
#pragma unroll 4
        for (int k = 1; k < K; ++k)
            a = __fmaf_rn(kt_weight<DEVW>(wts, k), widen(ld_elem(reinterpret_cast<const T *>(ld_table(pp + k - 1)) + g.start + e)), a);
        st_elem(reinterpret_cast<T *>(tv.ptr2[i]) + r, scale_elem(narrow<T>(a), scale));
    });
}

template <typename T, bool DEVW, int SPLIT>
__global__ __launch_bounds__(KT_BLOCK) void kt_fused_manyk_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                                  const int64_t *t_offs, const void *const *local_ptrs,
                                                                  const void *const *peer_ptrs, void *const *out_ptrs,
                                                                  uint32_t order, int K, float scale, KtWindow win,
                                                                  const int64_t *t_numel, AllWeights wts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK / SPLIT;
    __shared__ LdsTable lds;

    const unsigned piece = SPLIT == 1 ? blockIdx.x : kt_piece(order);
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    const T *src = reinterpret_cast<const T *>(ld_table(local_ptrs + tl.t0));
    T *dst = reinterpret_cast<T *>(ld_table(out_ptrs + tl.t0));
    pin(b_n, t_off, (uint64_t)src, (uint64_t)dst);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;
    const void *const *pp = peer_ptrs + (int64_t)g.bucket * (K - 1);   // peers 1..K-1 of this bucket

    if (tl.nt == 0 && g.end - g.start == TILE_ELEMS) {
        src += g.start - t_off;
        dst += g.start - t_off;
        const int v0 = part * VPT * KT_BLOCK + tid;
        Acc<T> acc[VPT];
        auto copy = [&](int k) { return k == 0 ? src : reinterpret_cast<const T *>(ld_table(pp + k - 1)) + g.start; };
        if constexpr (VPT == 1) sum_rolling<T, DEVW>(acc[0], copy, wts, K, v0);
        else sum_in_chunks<T, VPT, DEVW>(acc, copy, wts, K, v0);
        u32x4 res[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) res[u] = scale_vec<T, SPLIT == 1>(acc[u].template finish<SPLIT == 1>(), scale);
        if (SPLIT == 1) kt_wait_store_window(win);
#pragma unroll
        for (int u = 0; u < VPT; ++u) st_vec(reinterpret_cast<u32x4 *>(dst) + u * KT_BLOCK + v0, res[u]);
        return;
    }
    const int nt = tl.nt == 0 ? 1 : tl.nt;
    const void *const *op = reinterpret_cast<const void *const *>(out_ptrs);
    if (nt <= KT_LDS_TENSORS) {
        const LdsView tv = stage_lds(lds, t_offs, t_numel, local_ptrs, op, tl.t0, nt);
        fused_mixed_manyk<T, DEVW>(tv, nt, g, pp, K, wts, scale, part, SPLIT);
    } else {
        const GlobalView tv = global_view(t_offs, t_numel, local_ptrs, op, tl.t0);
        fused_mixed_manyk<T, DEVW>(tv, nt, g, pp, K, wts, scale, part, SPLIT);
    }
}

// Workgroups per tile and per CU, as for the reduce (before: whole tiles, two per CU for 3 to 5
// copies, the store window from 65 536 tiles read on):
//   K   fp32 (quarter tiles)                              bf16 (half tiles, two per CU)
//   4   91 562 tiles 1 246 -> 1 186 us, 7 052 even        42 502 tiles 562 -> 553 us, 18 043 even
//   5   7 052 tiles 114.2 -> 111.9 us, 3 563 2 % slower   5 393 tiles 89.9 -> 87.6 us, 3 526 2 % slower
//   6   12 206 tiles 236.4 -> 222.2 us, 2 367 2 % slower  4 727 tiles 93.2 -> 86.3 us, 85 285 1 612 -> 1 582
//   7   42 203 tiles 917 -> 894 us, 84 997 even           18 043 tiles 390 -> 368 us
//   8   7 052 tiles 174.3 -> 165.2 us (two per CU),       7 117 tiles 181.8 -> 163.3 us, 85 285 2 089 -> 2 046,
//       20 623 even with the window, 84 997 4 % slower    158 564 tiles 1 % slower than with the window
// Quarter tiles of bf16 and half tiles of fp32 are 1-3 % behind on most sizes.  bf16 launches of a few rounds
// (below 1 024 tiles) take half tiles as well, not held (551 tiles: K = 8 18.4 -> 15.4 us against 17.1
// for whole tiles, K = 4 11.6 -> 9.4 against 10.5); fp32 ones quarter tiles where whole ones are uneven
// (828 tiles, K = 4: 14.5 -> 12.9 against 13.4).
template <typename T> struct FusedSplit { static constexpr int N = 4; };
template <> struct FusedSplit<uint16_t> { static constexpr int N = 2; };

template <typename T> KtShape fused_shape(int K, int64_t nt)
{
    constexpr int S = FusedSplit<T>::N;
    if (sizeof(T) == 2) {
        if (K >= 6) return {S, nt >= 1024 ? 2u : 0u};
        if (K >= 4 && nt < 1024) return {S, 0};
        if (nt >= (K == 4 ? 32768 : 5120) && K >= 4) return {S, 2};
    } else {
        if (K == 4 && nt >= 8192) return {S, nt < 32768 ? 4u : 3u};       // 4 in runs, fused_run
        if (K == 5 && nt >= 6144) return {S, 3};
        if (K >= 6 && nt >= 4096) return {S, K == 8 ? 2u : 3u};
        if (K >= 4 && kt_uneven(nt)) return {S, 0};
    }
    // whole tiles, two per CU for 3 to 5 copies (2 729 tiles, K = 4: 38.0 -> 37.7 us against none held; 3 copies,
    // fp32, aligned: 2 500 tiles 4-7 % slower, 7 000 even, 10 000 1 % faster)
    return {1, K >= 3 && K <= 5 && nt >= (K == 3 ? 8192 : 2048) ? 2u : 0u};
}

// Bytes of a copy that an XCD takes in a run (kt_order; 0: launch order), where launches with runs are no slower after 512 MiB and more
// of ordinary reads or writes of other data, as a backward pass makes.  In us, launch order -> runs on the buffers of the call before / after
// 1 GiB of other reads:
//   bf16   4, 6 and 7 copies 128 KiB, 5 on whole tiles only: K = 4 94 645 tiles 1 285 -> 1 228 / 1 298 -> 1 254, K = 6 32 824 tiles
//          644 -> 623 / 640 -> 623, K = 7 93 682 tiles 2 155 -> 2 073 / 2 144 -> 2 075 (64 KiB: even); K = 5 on half tiles 19 772 tiles
//          314 -> 308 / 295 -> 306
//   fp32   4 copies 32 KiB on quarter tiles, 4 workgroups per CU, up to 32 767 tiles: 8 618 tiles 116.8 -> 112.8 / 117.9 -> 116.4, 19 993
//          tiles 267 -> 257 / 264 -> 262, 44 031 tiles 570 -> 575 / 559 -> 569, 92 895 tiles 2 and 4 % slower; 4 and 5 copies 128 KiB where whole tiles
//          are held (K = 5 2 587 tiles 44.0 -> 43.1 / 46.4 -> 45.6)
// The others gain 1-4 % from runs on the buffers of the call before and lose 2-10 % after other reads (fp32 K = 6 44 031 tiles 817 -> 799 /
// 769 -> 816, K = 8 9 892 tiles 236 -> 233 / 234 -> 244; bf16 K = 8 94 645 tiles 2 341 -> 2 306 / 2 133 -> 2 216).  Launches that hold nothing
// stay in launch order (whole tiles, K = 4 fp32 1 950 tiles 2 % slower in runs), and the whole tiles of other numbers of copies do not look for
// an order at all (K = 3 bf16, 596 tiles 9.7 us, 9.9 when they do).
template <typename T> int fused_run(int K, int64_t nt, const KtShape &sh)
{
    if (!sh.wgs || !kt_may_hold() || nt < 1024) return 0;
    if (sizeof(T) == 2) return K >= 4 && K <= 7 && (K != 5 || sh.split == 1) ? 131072 : 0;
    if (sh.split == 1) return K == 4 || K == 5 ? 131072 : 0;
    return K == 4 && nt < 32768 ? 32768 : 0;
}

// 9 and more copies outside the store window: quarter tiles, whose mixed tiles are shared too (a vector with a
// serial loop over the copies decides small launches: K = 16 fp32 29 tiles 18.3 -> 6.3 us, 222 tiles 22.1 -> 13.0, 763 tiles
// 41 -> 37.5, bf16 508 tiles 32.6 -> 27.2) in runs of 64 KiB per XCD from 640 tiles on (K = 9 fp32 3 243 tiles 87.5 -> 84.8 us;
// K = 16 bf16 975 tiles 48.3 -> 45.7; K = 12 5 322 tiles 1-3 % in every state; copies that have no window up to 4 095 tiles only: K = 9 fp32 19 375
// tiles 509 -> 495 us on the buffers of the call before, 479 -> 511 after other reads), held at two per CU above 1 152 (against whole ones, two types, K = 9 to 16, 1 141 to
// 3 006 tiles: 0-8 % faster, K = 9 to 14 up to 2 % slower where whole tiles make full rounds: fp32 K = 9 1 228 tiles
// 36.7 -> 35.9 us, 1 692 tiles 46.5 -> 46.9, K = 14 1 228 tiles 52.6 -> 53.6, K = 12 2 172 tiles 84.4 -> 79.6).
inline KtShape fused_manyk_shape(int64_t nt) { return {4, nt > 1152 ? 2u : 0u}; }
template <typename T> int fused_manyk_run(int K, int64_t nt, const KtShape &sh)
{
    if (sh.split == 1 || nt < 640 || (nt > 1152 && !kt_may_hold())) return 0;
    return nt < 4096 || K >= (sizeof(T) == 2 ? 11 : 10) ? 65536 : 0;
}

template <typename T, int K, bool DEVW>
hipError_t launch_fused_k(const KtDeviceTables &tb, const KtTile *tiles, int64_t nt, const void *const *locals,
                          const void *const *peers, const KtWeights &w, float scale, void *const *outs, hipStream_t s)
{
    const dim3 block(KT_BLOCK);
#define KT_ARGS(TILES, WIN) TILES, tb.b_elems, tb.t_off, locals, peers, outs, scale, WIN, tb.t_numel, FewWeights(w)
    if constexpr (K >= 7) {
        const int64_t least = sizeof(T) == 2 ? 131072 : K == 8 ? KT_WINDOW_MIN_TILES_FUSED : KT_WINDOW_MIN_TILES_REDUCE;
        const KtWindow win = kt_store_window(sizeof(T) == 4 && K == 8 ? KT_PERIOD_14 : KT_PERIOD_12, nt, least);
        if (win.width) {
            kt_fused_kernel<T, K, DEVW, 1, sizeof(T) == 2><<<dim3((unsigned)nt), block, 0, s>>>(KT_ARGS(tiles, win));
            return hipGetLastError();
        }
    }
    const KtShape sh = fused_shape<T>(K, nt);
    const unsigned lds = kt_shape_lds(sh, (unsigned)sizeof(LdsTable));
    return launch_in_chunks(tiles, nt, sh.split, [&](const KtTile *t, dim3 grid) {
        const KtWindow off{kt_order(grid.x, KT_TILE_BYTES / sh.split, fused_run<T>(K, nt, sh)), 0};
        if constexpr (K >= 4) {
            if (sh.split > 1) { kt_fused_kernel<T, K, DEVW, FusedSplit<T>::N, (sizeof(T) == 2 && K >= 6)><<<grid, block, lds, s>>>(KT_ARGS(t, off)); return; }
        }
        if constexpr (K < 6 || sizeof(T) == 4) kt_fused_kernel<T, K, DEVW, 1, (sizeof(T) == 2 && K == 1)><<<grid, block, lds, s>>>(KT_ARGS(t, off));
    });
#undef KT_ARGS
}

template <typename T, bool DEVW>
hipError_t launch_fused_t(const KtDeviceTables &tb, int64_t tile0, int64_t nt, const void *const *locals,
                          const void *const *peers, int K, const KtWeights &w, float scale, void *const *outs,
                          hipStream_t s)
{
    const KtTile *tiles = tb.tiles + tile0;
    switch (K) {
#define KT_CASE(KK) case KK: return launch_fused_k<T, KK, DEVW>(tb, tiles, nt, locals, peers, w, scale, outs, s);
        KT_CASE(1) KT_CASE(2) KT_CASE(3) KT_CASE(4) KT_CASE(5) KT_CASE(6) KT_CASE(7) KT_CASE(8)
#undef KT_CASE
    }
    const KtWindow win = kt_manyk_window(sizeof(T) == 2, K, nt, KT_WINDOW_MIN_READS_FUSED);
    const KtShape sh = win.width ? KtShape{1, 0} : fused_manyk_shape(nt);
    const unsigned lds = kt_shape_lds(sh, (unsigned)sizeof(LdsTable));
    return launch_in_chunks(tiles, nt, sh.split, [&](const KtTile *t, dim3 grid) {
        const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / sh.split, fused_manyk_run<T>(K, nt, sh));
#define KT_ARGS t, tb.b_elems, tb.t_off, locals, peers, outs, order, K, scale, win, tb.t_numel, AllWeights(w)
        if (sh.split == 1) kt_fused_manyk_kernel<T, DEVW, 1><<<grid, dim3(KT_BLOCK), lds, s>>>(KT_ARGS);
        else kt_fused_manyk_kernel<T, DEVW, 4><<<grid, dim3(KT_BLOCK), lds, s>>>(KT_ARGS);
#undef KT_ARGS
    });
}

}  // namespace

int kt_launch_fused(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0, int64_t ntiles,
                    const void *const *d_local_ptrs, const void *const *d_peer_ptrs, int K, const KtWeights &w,
                    float scale, void *const *d_out_ptrs, void *stream)
{
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
#define KT_FUSED(TT, DD) \
    (int)launch_fused_t<TT, DD>(tb, tile0, ntiles, d_local_ptrs, d_peer_ptrs, K, w, scale, d_out_ptrs, s)
    if (dt == KT_F32) return w.dev ? KT_FUSED(float, true) : KT_FUSED(float, false);
    return w.dev ? KT_FUSED(uint16_t, true) : KT_FUSED(uint16_t, false);
#undef KT_FUSED
}
