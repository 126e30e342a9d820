// HIP kernels for gfx950: multi-tensor pack and unpack-scale driven by the device-side
// tile + tensor-offset table.  Streaming, zero-reuse, HBM-bound: workgroups of 256 lanes
// (4 wavefronts), four to a 16 KiB tile, 16-byte vectors at any element address (non-temporal
// loads, system-scope stores), all loads of a lane in flight before its first store.
#include "kt_device.h"

// The copy kernels do best with little work per workgroup (unlike the
// read-dominated reduce, which wants many loads in flight per lane): the
// 16 KiB tile of the table is shared by KT_COPY_SPLIT workgroups, each moving
// KT_TILE_VECS / KT_BLOCK / KT_COPY_SPLIT vectors per lane.  With one vector
// per lane and workgroup (the default: 4 workgroups per 16 KiB tile) pack runs
// at 84 % of 8 TB/s on 1.3 G bf16 elements against 76 % with one workgroup per tile.
// That is the rate of a plain copy; a wavefront lives for little more than one memory latency,
// so the scalar loads ahead of its data load count: with one more dependent load on the way
// pack took 841 us instead of 785 and unpack 945 instead of 795.
// Tensors and buckets may lie at any element address.  24.4 M bf16 elements in 400 tensors of odd
// sizes, dense layout, gradients as views: pack 47 -> 20.5 us and unpack 48 -> 20 us against one
// element per lane, which misaligned addresses took before.
#ifndef KT_COPY_SPLIT
#define KT_COPY_SPLIT (KT_TILE_VECS / KT_BLOCK)
#endif

namespace {

constexpr int COPY_SPLIT = KT_COPY_SPLIT;
constexpr int COPY_VPT = KT_TILE_VECS / KT_BLOCK / COPY_SPLIT;     // vectors per lane and workgroup
static_assert(COPY_VPT >= 1 && COPY_VPT * COPY_SPLIT * KT_BLOCK == KT_TILE_VECS, "workgroups per tile");

// ---- pack ----------------------------------------------------------------

// Mixed tile: (1) find each vector's owner in the staged table and issue its load, (2) store.
// A vector that is not wholly inside one tensor (tensor ends, padding) gathers its elements, all
// loads in flight together, so that a tile's few such vectors cost one memory latency more and
// not one per element.
template <typename T, typename V>
__device__ __forceinline__ void pack_mixed(const V &tv, int nt, const TileGeom &g, int64_t b_n, T *dst, int part)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int VPT = COPY_VPT;
    const int nvec = (int)((g.end - g.start + VE - 1) / VE);
    u32x4 val[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int v = (part * VPT + j) * KT_BLOCK + threadIdx.x;
        if (v < nvec) {
            const int64_t e0 = g.start + (int64_t)v * VE;
            const int i = find_owner_v(tv, nt, e0);
            const int64_t r = i >= 0 ? e0 - tv.off[i] : -1;
            if (r >= 0 && r + VE <= tv.numel[i] && e0 + VE <= b_n)
                val[j] = ld_vec(reinterpret_cast<const T *>(tv.ptr[i]) + r);
            else
                val[j] = gather_vec<T>(tv, nt, i, e0, b_n);
        }
    }
    const bool wt = off64(dst) == 0;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int v = (part * VPT + j) * KT_BLOCK + threadIdx.x;
        if (v < nvec) {
            const int64_t e0 = g.start + (int64_t)v * VE;
            if (e0 + VE <= b_n) st_vec_pick(dst + e0, val[j], wt);
            else {                    // the last, partial vector of a densely packed bucket
#pragma unroll
                for (int q = 0; q < VE; ++q)
                    if (e0 + q < b_n) st_elem(dst + e0 + q, elem_of<T>(val[j], q));
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(KT_BLOCK) void kt_pack_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                           const int64_t *t_offs, const void *const *tensor_ptrs,
                                                           void *const *bucket_ptrs, const int64_t *t_numel)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = COPY_VPT;
    __shared__ LdsTable lds;

    const int part = COPY_SPLIT == 1 ? 0 : (int)(blockIdx.x % COPY_SPLIT);
    const KtTile tl = ld_tile(tiles + blockIdx.x / COPY_SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    T *dst = reinterpret_cast<T *>(ld_table(bucket_ptrs + tl.bucket));
    const T *src = reinterpret_cast<const T *>(ld_table(tensor_ptrs + tl.t0));
    pin(b_n, t_off, (uint64_t)dst, (uint64_t)src);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;

    if (tl.nt == 0) {
        // Solid tile: one tensor owns everything; straight 16-byte copy at any address.
        src += g.start - t_off;
        T *d = dst + g.start;
        const int o = off64(d);
        const int nvec = (int)((g.end - g.start) / VE);
        if (nvec == KT_TILE_VECS) {
            u32x4 r[VPT];
            RotVec rv[VPT];
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                rv[j] = rot_vec<KT_TILE_BYTES>(((part * VPT + j) * KT_BLOCK + tid) * KT_VEC_BYTES, o);
                r[j] = ld_vec(reinterpret_cast<const char *>(src) + rv[j].at);
            }
            const __amdgpu_buffer_rsrc_t rs = tile_rsrc(d, KT_TILE_BYTES);
#pragma unroll
            for (int j = 0; j < VPT; ++j)
                if (rv[j].whole) st_tile_wt(rs, rv[j].at, r[j]);
            if ((o & (KT_VEC_BYTES - 1)) && part == 0 && tid < VE) {
                const int e = edge_elem<KT_TILE_BYTES>(tid, sizeof(T), o) / (int)sizeof(T);
                st_elem(d + e, ld_elem(src + e));
            }
        } else {
#pragma unroll 1
            for (int v = part * KT_BLOCK + tid; v < nvec; v += COPY_SPLIT * KT_BLOCK)
                st_vec_pick(d + (int64_t)v * VE, ld_vec(src + (int64_t)v * VE), o == 0);
        }
        return;
    }

    // a short last tile leaves the later workgroups of the tile without vectors
    if ((int64_t)part * VPT * KT_BLOCK * VE >= g.end - g.start) return;
    if (tl.nt <= KT_LDS_TENSORS) {
        const LdsView tv = stage_lds(lds, t_offs, t_numel, tensor_ptrs, nullptr, tl.t0, tl.nt);
        pack_mixed<T>(tv, tl.nt, g, b_n, dst, part);
    } else {
        const GlobalView tv = global_view(t_offs, t_numel, tensor_ptrs, nullptr, tl.t0);
        pack_mixed<T>(tv, tl.nt, g, b_n, dst, part);
    }
}

// ---- unpack with scale ----------------------------------------------------

// Mixed tile.  The bucket's vectors (`val`) were loaded before the table was staged: their
// addresses do not depend on it.  The elements of vectors that are not wholly inside one tensor go
// one per lane (each_cut_elem).
template <typename T, typename V>
__device__ __forceinline__ void unpack_mixed(const V &tv, int nt, const TileGeom &g, const u32x4 *val, const T *src,
                                             float scale, int part)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int VPT = COPY_VPT;
    const int nvec = (int)((g.end - g.start) / VE);
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int v = (part * VPT + j) * KT_BLOCK + threadIdx.x;
        if (v < nvec) {
            const int64_t e0 = g.start + (int64_t)v * VE;
            const int i = find_owner_v(tv, nt, e0);
            const int64_t r = i >= 0 ? e0 - tv.off[i] : -1;
            if (r >= 0 && r + VE <= tv.numel[i]) {
                T *p = reinterpret_cast<T *>(tv.ptr[i]) + r;
                // whole 64-byte pieces per wavefront: the address of the lane that starts the piece
                st_vec_pick(p, scale_vec<T>(val[j], scale), off64(reinterpret_cast<char *>(p) - (size_t)(threadIdx.x & 3) * KT_VEC_BYTES) == 0);
            }
        }
    }
    each_cut_elem<VE>(tv, nt, g.start, (int)(g.end - g.start), part * KT_BLOCK + threadIdx.x, COPY_SPLIT * KT_BLOCK,
                      [&](int i, int64_t r, int e) {
                          st_elem(reinterpret_cast<T *>(tv.ptr[i]) + r, scale_elem(ld_elem(src + g.start + e), scale));
                      });
}

template <typename T>
__global__ __launch_bounds__(KT_BLOCK) void kt_unpack_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                             const int64_t *t_offs, const void *const *bucket_ptrs,
                                                             void *const *tensor_ptrs, float scale,
                                                             const int64_t *t_numel)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = COPY_VPT;
    __shared__ LdsTable lds;

    const int part = COPY_SPLIT == 1 ? 0 : (int)(blockIdx.x % COPY_SPLIT);
    const KtTile tl = ld_tile(tiles + blockIdx.x / COPY_SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    const T *src = reinterpret_cast<const T *>(ld_table(bucket_ptrs + tl.bucket));
    T *dst = reinterpret_cast<T *>(ld_table(tensor_ptrs + tl.t0));
    pin(b_n, t_off, (uint64_t)dst, (uint64_t)src);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;

    if (tl.nt == 0) {
        dst += g.start - t_off;
        const T *s = src + g.start;
        const int o = off64(dst);
        const int nvec = (int)((g.end - g.start) / VE);
        if (nvec == KT_TILE_VECS) {
            u32x4 r[VPT];
            RotVec rv[VPT];
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                rv[j] = rot_vec<KT_TILE_BYTES>(((part * VPT + j) * KT_BLOCK + tid) * KT_VEC_BYTES, o);
                r[j] = ld_vec(reinterpret_cast<const char *>(s) + rv[j].at);
            }
            const __amdgpu_buffer_rsrc_t rs = tile_rsrc(dst, KT_TILE_BYTES);
#pragma unroll
            for (int j = 0; j < VPT; ++j)
                if (rv[j].whole) st_tile_wt(rs, rv[j].at, scale_vec<T>(r[j], scale));
            if ((o & (KT_VEC_BYTES - 1)) && part == 0 && tid < VE) {
                const int e = edge_elem<KT_TILE_BYTES>(tid, sizeof(T), o) / (int)sizeof(T);
                st_elem(dst + e, scale_elem(ld_elem(s + e), scale));
            }
        } else {
#pragma unroll 1
            for (int v = part * KT_BLOCK + tid; v < nvec; v += COPY_SPLIT * KT_BLOCK)
                st_vec_pick(dst + (int64_t)v * VE, scale_vec<T>(ld_vec(s + (int64_t)v * VE), scale), o == 0);
        }
        return;
    }

    if ((int64_t)part * VPT * KT_BLOCK * VE >= g.end - g.start && part * KT_BLOCK >= tl.nt * 2 * VE) return;
    u32x4 val[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int64_t e0 = g.start + (int64_t)((part * VPT + j) * KT_BLOCK + tid) * VE;
        if (e0 + VE <= g.end) val[j] = ld_vec(src + e0);
    }
    const void *const *tp = reinterpret_cast<const void *const *>(tensor_ptrs);
    if (tl.nt <= KT_LDS_TENSORS) {
        const LdsView tv = stage_lds(lds, t_offs, t_numel, tp, nullptr, tl.t0, tl.nt);
        unpack_mixed<T>(tv, tl.nt, g, val, src, scale, part);
    } else {
        const GlobalView tv = global_view(t_offs, t_numel, tp, nullptr, tl.t0);
        unpack_mixed<T>(tv, tl.nt, g, val, src, scale, part);
    }
}

}  // namespace

int kt_launch_pack(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0, int64_t ntiles,
                   const void *const *d_tensor_ptrs, void *const *d_bucket_ptrs, void *stream)
{
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const dim3 block(KT_BLOCK);
    return (int)launch_in_chunks(tb.tiles + tile0, ntiles, COPY_SPLIT, [&](const KtTile *tiles, dim3 grid) {
        if (dt == KT_F32) kt_pack_kernel<float><<<grid, block, 0, s>>>(tiles, tb.b_elems, tb.t_off, d_tensor_ptrs, d_bucket_ptrs, tb.t_numel);
        else kt_pack_kernel<uint16_t><<<grid, block, 0, s>>>(tiles, tb.b_elems, tb.t_off, d_tensor_ptrs, d_bucket_ptrs, tb.t_numel);
    });
}

int kt_launch_unpack(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0, int64_t ntiles,
                     const void *const *d_bucket_ptrs, float scale, void *const *d_tensor_ptrs, void *stream)
{
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const dim3 block(KT_BLOCK);
    return (int)launch_in_chunks(tb.tiles + tile0, ntiles, COPY_SPLIT, [&](const KtTile *tiles, dim3 grid) {
        if (dt == KT_F32) kt_unpack_kernel<float><<<grid, block, 0, s>>>(tiles, tb.b_elems, tb.t_off, d_bucket_ptrs, d_tensor_ptrs, scale, tb.t_numel);
        else kt_unpack_kernel<uint16_t><<<grid, block, 0, s>>>(tiles, tb.b_elems, tb.t_off, d_bucket_ptrs, d_tensor_ptrs, scale, tb.t_numel);
    });
}
