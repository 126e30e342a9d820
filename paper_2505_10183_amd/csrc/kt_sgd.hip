// HIP kernels for gfx950: unpack fused with SGD momentum / weight decay.
#include "kt_sgd_device.h"

namespace {

// A tile of the bucket (16 KiB of gradient) goes with 16 KiB (fp32) or 32 KiB
// (bf16) each of parameters and momentum, read and written in place.  SPLIT
// workgroups share one tile; every workgroup has one quad of 4 elements per lane
// (it reads 4 KiB of p and of v and writes the same 4 KiB back at once), which
// keeps few bytes in flight: 79 % of 8 TB/s for either gradient type, 75 % (bf16)
// and 78 % (fp32) with two quads.  Every tensor may lie at any element address: the
// quads of a full tile are laid out from a 64-byte boundary of the parameters
// (rot_vec), which the system-scope stores of the bf16 form need.  45.1 M bf16
// elements in 600 tensors of odd sizes, with the model copy: unpack 200 -> 178 us.
// bf16: a full tile whose parameters start elsewhere in their 64 bytes takes non-temporal stores although all of its
// stores but two fill whole pieces (the same set, dense layout: 180 -> 149 us without the model copy), mixed tiles system-scope ones
// wherever they lie (600 tensors of 75 208 elements 146 -> 139 us).
template <typename T> struct SgdShape {
    static constexpr int SPLIT = (int)(KT_TILE_VECS * Elem<T>::VE / 4 / KT_BLOCK);   // workgroups per tile
    static constexpr int PBYTES = KT_TILE_VECS * Elem<T>::VE * 4;                     // bytes of p in a tile
};

// The quads of a lane's turn: parameters p, momentum v, model copy m (bf16, or NULL).
// MASTER: 0 no model copy, 1 non-temporal stores of it, 2 system-scope ones.
template <typename T, int MASTER>
__device__ __forceinline__ void sgd_store(float *p, float *v, uint16_t *m, u32x4 pr, u32x4 vr, bool p64, bool v64)
{
    // with bf16 gradients 44 % of the bytes are written: system-scope stores where the tile starts on 64 bytes and in
    // mixed tiles
    if (sizeof(T) == 2 && p64) st_vec_copy<true>(p, pr); else st_vec(p, pr);
    if (sizeof(T) == 2 && v64) st_vec_copy<true>(v, vr); else st_vec(v, vr);
    if (MASTER) st_model_quad<MASTER == 2>(m, pr);
}

template <typename T, int MASTER>
__device__ __forceinline__ void sgd_one(const T *g, float *p, float *v, uint16_t *m, const KtSgd &a)
{
    float pv = ld_elem(p), vv = ld_elem(a.first ? p : v);
    sgd_elem(widen(ld_elem(g)), pv, vv, a);
    st_elem(p, pv);
    st_elem(v, vv);
    if (MASTER) st_elem(m, (uint16_t)f32_to_bf16(pv));
}

// Mixed tile: tv.ptr = parameters, tv.ptr2 = momentum of the owning tensor; model (MASTER only) =
// the model-parameter pointers of the tile's tensors, in registers or in the global pointer table.  Quads wholly
// inside one tensor one per lane, the elements of the others one per lane (each_cut_elem): with bf16
// gradients between the quads' loads and their stores, which are system-scope at any address here and waited for.
template <typename T, int MASTER, typename V, typename M>
__device__ __forceinline__ void sgd_mixed(const V &tv, int nt, const TileGeom &g, const T *src, const KtSgd &a, int part,
                                          const M &model)
{
    const int len = (int)(g.end - g.start);
    const int q = part * KT_BLOCK + threadIdx.x;
    auto cut = [&] {
        each_cut_elem<4>(tv, nt, g.start, len, q, SgdShape<T>::SPLIT * KT_BLOCK, [&](int i, int64_t r, int e) {
            sgd_one<T, MASTER>(src + g.start + e, reinterpret_cast<float *>(tv.ptr[i]) + r, reinterpret_cast<float *>(tv.ptr2[i]) + r,
                               MASTER ? reinterpret_cast<uint16_t *>(model[i]) + r : nullptr, a);
        });
    };
    float *p = nullptr, *v = nullptr;
    uint16_t *m = nullptr;
    Quad<T> gq;
    u32x4 pr, vr;
    auto update = [&] {
        sgd_quad(gq, pr, vr, a);
        sgd_store<T, MASTER>(p, v, m, pr, vr, true, true);
    };
    if (q < len / 4) {
        const int64_t e0 = g.start + 4 * (int64_t)q;
        const int i = find_owner_v(tv, nt, e0);
        const int64_t r = i >= 0 ? e0 - tv.off[i] : -1;
        if (r >= 0 && r + 4 <= tv.numel[i]) {
            p = reinterpret_cast<float *>(tv.ptr[i]) + r;
            v = reinterpret_cast<float *>(tv.ptr2[i]) + r;
            if (MASTER) m = reinterpret_cast<uint16_t *>(model[i]) + r;
            gq = ld_quad(reinterpret_cast<const Quad<T> *>(src + e0));
            pr = ld_vec(p);
            vr = ld_vec(a.first ? p : v);
            if (sizeof(T) == 4) update();
        }
    }
    cut();
    if (sizeof(T) == 2 && p) update();
}

// DEVS: the four optimizer scalars come from device memory (uniform scalar loads, issued with
// the tile-table load) instead of the kernel-argument block, so that a recorded launch follows
// a learning-rate schedule.  A separate instantiation: launches with scalars by value run the
// code they always ran.
template <typename T, int MASTER, bool DEVS>
__global__ __launch_bounds__(KT_BLOCK) void kt_unpack_sgd_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                                 const int64_t *t_offs, const void *const *bucket_ptrs,
                                                                 void *const *param_ptrs, void *const *mom_ptrs,
                                                                 uint32_t order, void *const *model_ptrs, KtSgd a,
                                                                 const int64_t *t_numel)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int SPLIT = SgdShape<T>::SPLIT, PBYTES = SgdShape<T>::PBYTES;
    __shared__ LdsTable lds;

    const unsigned piece = kt_piece(order);
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    const T *src = reinterpret_cast<const T *>(ld_table(bucket_ptrs + tl.bucket));
    float *p = reinterpret_cast<float *>(ld_table(param_ptrs + tl.t0));
    float *v = reinterpret_cast<float *>(ld_table(mom_ptrs + tl.t0));
    uint16_t *m = MASTER ? reinterpret_cast<uint16_t *>(ld_table(model_ptrs + tl.t0)) : nullptr;
    if (DEVS) {
        const float *d = a.dev;
        a.scale = ld_table(d);
        a.lr = ld_table(d + 1);
        a.mu = ld_table(d + 2);
        a.wd = ld_table(d + 3);
    }
    pin(b_n, t_off, (uint64_t)src, (uint64_t)p);
    pin((uint64_t)v, (uint64_t)m, 0, 0);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;

    if (tl.nt == 0) {
        // Solid tile, processed in quads of 4 elements so that every access is
        // coalesced: 16 bytes of p and of v per lane, 16 (fp32) or 8 (bf16)
        // bytes of gradient.
        const int64_t rel = g.start - t_off;
        src += g.start;
        p += rel;
        v += rel;
        if (MASTER) m += rel;
        const int len = (int)(g.end - g.start);
        if (len == TILE_ELEMS) {
            const int o = off64(p);
            const RotVec rv = rot_vec<PBYTES>((part * KT_BLOCK + tid) * 16, o);
            if (rv.whole) {
                const int e = rv.at / 4;
                const Quad<T> gq = ld_quad(reinterpret_cast<const Quad<T> *>(src + e));
                u32x4 pr = ld_vec(p + e), vr = ld_vec((a.first ? p : v) + e);
                sgd_quad(gq, pr, vr, a);
                sgd_store<T, MASTER>(p + e, v + e, MASTER ? m + e : nullptr, pr, vr, o == 0, o == 0 && off64(v) == 0);
            }
            if ((o & 15) && part == 0 && tid < 4) {
                const int e = edge_elem<PBYTES>(tid, 4, o) / 4;
                sgd_one<T, MASTER>(src + e, p + e, v + e, MASTER ? m + e : nullptr, a);
            }
        } else {
            // a short solid tile is a whole number of quads
            const int e = (part * KT_BLOCK + tid) * 4;
            if (e < len) {
                const Quad<T> gq = ld_quad(reinterpret_cast<const Quad<T> *>(src + e));
                u32x4 pr = ld_vec(p + e), vr = ld_vec((a.first ? p : v) + e);
                sgd_quad(gq, pr, vr, a);
                sgd_store<T, MASTER>(p + e, v + e, MASTER ? m + e : nullptr, pr, vr, off64(p) == 0, off64(v) == 0);
            }
        }
        return;
    }

    if (part * KT_BLOCK * 4 >= g.end - g.start && part * KT_BLOCK >= tl.nt * 8) return;
    const void *const *pp = reinterpret_cast<const void *const *>(param_ptrs);
    const void *const *mp = reinterpret_cast<const void *const *>(mom_ptrs);
    void *const *model = MASTER ? model_ptrs + tl.t0 : nullptr;
    if (sizeof(T) == 2 && tl.nt <= KT_REG_TENSORS) {
        const Regs<uintptr_t> mr = ld_regs<uintptr_t>(MASTER ? model_ptrs : mom_ptrs, tl.t0, tl.nt);
        sgd_mixed<T, MASTER>(reg_view(t_offs, t_numel, pp, mp, tl.t0, tl.nt), tl.nt, g, src, a, part, mr);
    } else if (tl.nt <= KT_LDS_TENSORS) {
        const LdsView tv = stage_lds(lds, t_offs, t_numel, pp, mp, tl.t0, tl.nt);
        sgd_mixed<T, MASTER>(tv, tl.nt, g, src, a, part, model);
    } else {
        const GlobalView tv = global_view(t_offs, t_numel, pp, mp, tl.t0);
        sgd_mixed<T, MASTER>(tv, tl.nt, g, src, a, part, model);
    }
}

// LDS asked for beyond the kernel's own, to hold the number of workgroups per CU (8 without) and
// with it the reads in flight: fewer mix better with the writes.  bf16: 5 (1.3B
// set 3.78 -> 3.47 ms, with the model copy 4.30 -> 3.92); fp32: 4 (ViT-B/16 0.281 -> 0.269 ms,
// 65 536 tiles 0.914 -> 0.835 ms).  Launches of less than 64 MiB of gradient do not fill the chip
// long enough to gain (2 729 tiles fp32 36 us either way) and go without.
static unsigned sgd_lds(kt_dtype dt, int64_t ntiles)
{
    if (ntiles < 4096 || !kt_may_hold()) return 0;
    return kt_hold_lds(dt == KT_F32 ? 4 : 5, (unsigned)sizeof(LdsTable));
}

// Bytes of gradient that an XCD takes in a run (kt_order; 0: launch order).  Behind pack and reduce: fp32 from 1 024 tiles on (whole step of
// 6 332 tiles 197 -> 192 us, 16 337 tiles of odd tensors 502 -> 494, others 0-2 %, also after 1 GiB of other reads or writes; 63 057
// tiles 1 % either way); bf16, whose stores are system-scope ones, from 1 792 to 4 095 (1 916 tiles with the model copy 84.8 -> 83.2, 3 177 tiles of
// odd tensors 150.7 -> 147.7; 883 to 1 320 tiles 2-5 % slower in runs, 9 996 tiles 257 us, 265 in runs).
static int sgd_run(kt_dtype dt, int64_t ntiles)
{
    return (dt == KT_F32 ? ntiles >= 1024 && ntiles < 32768 : ntiles >= 1792 && ntiles < 4096) ? 131072 : 0;
}

}  // namespace

int kt_launch_unpack_sgd(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0, int64_t ntiles,
                         const void *const *d_bucket_ptrs, void *const *d_param_ptrs, void *const *d_mom_ptrs,
                         void *const *d_model_ptrs, const KtSgd &a, void *stream)
{
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    dim3 block(KT_BLOCK);
    const int split = dt == KT_F32 ? SgdShape<float>::SPLIT : SgdShape<uint16_t>::SPLIT;
    const unsigned lds = sgd_lds(dt, ntiles);
    return (int)launch_in_chunks(tb.tiles + tile0, ntiles, split, [&](const KtTile *tiles, dim3 grid) {
        const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / split, sgd_run(dt, ntiles));
#define KT_SGD_LAUNCH(TT, MM, DD)                                                                                    \
    kt_unpack_sgd_kernel<TT, MM, DD><<<grid, block, lds, s>>>(tiles, tb.b_elems, tb.t_off, d_bucket_ptrs, d_param_ptrs, \
                                                              d_mom_ptrs, order, d_model_ptrs, a, tb.t_numel)
        if (dt == KT_F32) {
            if (d_model_ptrs) { if (a.dev) KT_SGD_LAUNCH(float, 2, true); else KT_SGD_LAUNCH(float, 2, false); }
            else { if (a.dev) KT_SGD_LAUNCH(float, 0, true); else KT_SGD_LAUNCH(float, 0, false); }
        } else {
            // model copy of 2 bytes per element: half pieces wherever p starts on an odd 64 bytes.  Non-temporal (19 837 tiles
            // 517 -> 506 us, 59 899 tiles 1 526 -> 1 505, odd tensors 15 770 tiles 475 -> 438; 69 818 to 97 261 tiles within 1 % either way)
            // below 98 304 tiles (104 124 to 138 759 tiles 0.3-0.8 % slower, 158 785 2.5 %); fp32 keeps system scope (20 000 tiles 300 -> 295 us without, odd tensors 11 007 tiles 160 -> 168)
            if (d_model_ptrs && ntiles >= 98304) { if (a.dev) KT_SGD_LAUNCH(uint16_t, 2, true); else KT_SGD_LAUNCH(uint16_t, 2, false); }
            else if (d_model_ptrs) { if (a.dev) KT_SGD_LAUNCH(uint16_t, 1, true); else KT_SGD_LAUNCH(uint16_t, 1, false); }
            else { if (a.dev) KT_SGD_LAUNCH(uint16_t, 0, true); else KT_SGD_LAUNCH(uint16_t, 0, false); }
        }
#undef KT_SGD_LAUNCH
    });
}
