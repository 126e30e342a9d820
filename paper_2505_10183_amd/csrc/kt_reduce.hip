// HIP kernels for gfx950: the K-way weighted reduce.  HBM-bound (K reads, one write per
// element); nothing here is a contraction, so no MFMA.
#include "kt_device.h"

namespace {

// One workgroup per 16 KiB tile.  A full tile keeps all K copies of the lane's 4 vectors in flight
// together (32 loads at K = 8): the kernel is bound by what the memory system sustains for reads
// with one written line in K + 1.  Copies and output may lie at any element address.  The stores
// are not moved to 64-byte boundaries as pack and unpack do: with the offsets in registers the
// loads issue back to back, which inside the store windows lost 3-10 % (1.3B set 3.77 -> 3.89 ms),
// more than the 3 % of a misaligned non-temporal store stream.
template <typename T, int K, bool DEVW>
__global__ __launch_bounds__(KT_BLOCK) void kt_reduce_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                             const void *const *peer_ptrs, void *const *out_ptrs,
                                                             KtWindow win, FewWeights wts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK;   // vectors per lane, K loads each, all in flight at once

    const KtTile tl = ld_tile(tiles + blockIdx.x);
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
        u32x4 r[VPT][K];
#pragma unroll
        for (int u = 0; u < VPT; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) r[u][k] = ld_vec(reinterpret_cast<const u32x4 *>(x[k]) + u * KT_BLOCK + tid);
        u32x4 res[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            Acc<T> acc;
            acc.first(r[u][0], w[0]);
#pragma unroll
            for (int k = 1; k < K; ++k) acc.add(r[u][k], w[k]);
            res[u] = acc.template finish<(K >= 6)>();
        }
        kt_wait_store_window(win);     // large launches: the chip writes in bursts (KtWindow)
#pragma unroll
        for (int u = 0; u < VPT; ++u) st_vec(reinterpret_cast<u32x4 *>(out) + u * KT_BLOCK + tid, res[u]);
    } else {
        for (int v = tid; v < nvec; v += KT_BLOCK) {
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
        if (e < n) {
            float a = __fmul_rn(w[0], widen(ld_elem(x[0] + e)));
#pragma unroll
            for (int k = 1; k < K; ++k) a = __fmaf_rn(w[k], widen(ld_elem(x[k] + e)), a);
            st_elem(out + e, narrow<T>(a));
        }
    }
}

// K > 8: peers in chunks, accumulators in registers across chunks (sum_in_chunks).
template <typename T, bool DEVW>
__global__ __launch_bounds__(KT_BLOCK) void kt_reduce_manyk_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                                   const void *const *peer_ptrs, void *const *out_ptrs,
                                                                   int K, KtWindow win, AllWeights wts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK;
    const KtTile tl = ld_tile(tiles + blockIdx.x);
    const TileGeom g = tile_geom(tl, ld_table(b_elems + tl.bucket), TILE_ELEMS);
    const int tid = threadIdx.x;
    const void *const *pp = peer_ptrs + (int64_t)g.bucket * K;
    auto peer = [&](int k) { return reinterpret_cast<const T *>(ld_table(pp + k)) + g.start; };
    T *out = reinterpret_cast<T *>(ld_table(out_ptrs + g.bucket)) + g.start;
    const int64_t n = g.end - g.start;
    const int nvec = (int)(n / VE);
    if (nvec == KT_TILE_VECS) {
        Acc<T> acc[VPT];
        sum_in_chunks<T, DEVW>(acc, peer, wts, K, tid);
        u32x4 res[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) res[u] = acc[u].finish();
        kt_wait_store_window(win);
#pragma unroll
        for (int u = 0; u < VPT; ++u) st_vec(reinterpret_cast<u32x4 *>(out) + u * KT_BLOCK + tid, res[u]);
        return;
    }
    // the ragged last tile of a bucket: one vector at a time
    for (int v = tid; v < nvec; v += KT_BLOCK) {
        Acc<T> acc;
        acc.first(ld_vec(peer(0) + (int64_t)v * VE), kt_weight<DEVW>(wts, 0));
#pragma unroll 4
        for (int k = 1; k < K; ++k) acc.add(ld_vec(peer(k) + (int64_t)v * VE), kt_weight<DEVW>(wts, k));
        st_vec(out + (int64_t)v * VE, acc.finish());
    }
    const int64_t e = (int64_t)nvec * VE + tid;
    if (e < n) {
        float a = __fmul_rn(kt_weight<DEVW>(wts, 0), widen(ld_elem(peer(0) + e)));
        for (int k = 1; k < K; ++k) a = __fmaf_rn(kt_weight<DEVW>(wts, k), widen(ld_elem(peer(k) + e)), a);
        st_elem(out + e, narrow<T>(a));
    }
}

template <typename T, bool DEVW>
hipError_t launch_reduce_t(const KtDeviceTables &tb, int64_t tile0, int64_t ntiles, const void *const *peers,
                           int K, const KtWeights &w, void *const *outs, hipStream_t s)
{
    dim3 grid((unsigned)ntiles), block(KT_BLOCK);
    const KtTile *tiles = tb.tiles + tile0;
    const KtWindow win = kt_store_window(K, ntiles, K <= 8 ? KT_WINDOW_MIN_TILES_REDUCE : (KT_WINDOW_MIN_READS_REDUCE_MANYK + K - 1) / K,
                                         sizeof(T) == 4);
    const unsigned lds = kt_mix_lds(win, K, ntiles, 4096, 0);
    switch (K) {
#define KT_CASE(KK) \
    case KK: kt_reduce_kernel<T, KK, DEVW><<<grid, block, lds, s>>>(tiles, tb.b_elems, peers, outs, win, FewWeights(w)); break;
        KT_CASE(1) KT_CASE(2) KT_CASE(3) KT_CASE(4) KT_CASE(5) KT_CASE(6) KT_CASE(7) KT_CASE(8)
#undef KT_CASE
    default: kt_reduce_manyk_kernel<T, DEVW><<<grid, block, 0, s>>>(tiles, tb.b_elems, peers, outs, K, win, AllWeights(w)); break;
    }
    return hipGetLastError();
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
