// HIP kernels for gfx950: the single pass from K gradient copies to updated parameters
// (fused single pass + SGD momentum / weight decay in one kernel).
#include "kt_sgd_device.h"

namespace {

// ---- tensors + peer buckets -> parameters and momentum ----------------------
// Per element: r = round_T(sum_k w_k x_k) with x_0 read from the local gradient
// tensor and x_1..x_{K-1} from the peer buckets (product for k = 0, then one
// fused multiply-add per peer in ascending k, rounded to the storage type T as
// the reduce does), then the update of unpack-with-SGD on x = widen(r):
// g = scale*x; g' = fma(wd,p,g); v' = g' or fma(mu,v,g'); p' = fma(-lr,v',p).
// The results are bit-identical to pack -> reduce -> unpack-with-SGD; the
// reduced gradient is never written: (K-1)*s + s + 16 bytes per element move
// instead of (K+1)*s + s + 16.

struct FsgdArgs {
    const void *const *local_ptrs;   // T gradient tensors (peer 0)
    const void *const *peer_ptrs;    // nb * (K-1) peer buckets
    void *const *param_ptrs;         // T
    void *const *mom_ptrs;           // T
    void *const *model_ptrs;         // T, or NULL: no bf16 model copy
};

__device__ __forceinline__ KtSgd resolve_sgd(KtSgd a)
{
    if (a.dev) {        // uniform: the optimizer scalars set with kt_plan_set_sgd
        a.scale = ld_table(a.dev);
        a.lr = ld_table(a.dev + 1);
        a.mu = ld_table(a.dev + 2);
        a.wd = ld_table(a.dev + 3);
    }
    return a;
}

// The tensor side of a tile: pointers of its first tensor, advanced to the tile by `at`.
template <typename T> struct TensorSide {
    const T *src;
    float *p, *v;
    uint16_t *m;      // NULL: no model copy
    __device__ __forceinline__ TensorSide(const FsgdArgs &f, int t0)
    {
        src = reinterpret_cast<const T *>(ld_table(f.local_ptrs + t0));
        p = reinterpret_cast<float *>(ld_table(f.param_ptrs + t0));
        v = reinterpret_cast<float *>(ld_table(f.mom_ptrs + t0));
        // read in any case, so that no branch stands between the table loads
        m = reinterpret_cast<uint16_t *>(ld_table((f.model_ptrs ? f.model_ptrs : f.mom_ptrs) + t0));
        pin((uint64_t)src, (uint64_t)p, (uint64_t)v, (uint64_t)m);
        if (!f.model_ptrs) m = nullptr;
    }
    __device__ __forceinline__ void advance(int64_t rel)
    {
        src += rel;
        p += rel;
        v += rel;
        if (m) m += rel;
    }
};

// Stores of a lane's N updated quads (quad j at q4 + j * LANES): parameters, momentum and, for
// mixed precision, the model copy.
template <int N, int LANES> __device__ __forceinline__ void st_quads(u32x4 *p4, u32x4 *v4, u32x2 *m2, const u32x4 *pr, const u32x4 *vr)
{
#pragma unroll
    for (int j = 0; j < N; ++j) {
        st_vec(p4 + j * LANES, pr[j]);
        st_vec(v4 + j * LANES, vr[j]);
    }
    if (m2) {
#pragma unroll
        for (int j = 0; j < N; ++j) st_model_quad(m2 + j * LANES, pr[j]);
    }
}

// The quads of a lane against their gradients.  bf16: a lane's 16-byte vector holds 8 elements =
// 32 bytes of p; the reduced values go through LDS once and come back in quads of 4 elements, so
// that every access to p and v is one coalesced 16 bytes per lane.  binary32: a vector is a quad.
template <int VPT, int LANES> __device__ __forceinline__ void update_quads(const u32x4 *red, u32x4 *, u32x4 *pr, u32x4 *vr, const KtSgd &a, float)
{
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        Quad<float> q;
        q.d = red[u];
        sgd_quad(q, pr[u], vr[u], a);
    }
}
template <int VPT, int LANES> __device__ __forceinline__ void update_quads(const u32x4 *red, u32x4 *lds, u32x4 *pr, u32x4 *vr, const KtSgd &a, uint16_t)
{
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < VPT; ++u) lds[u * LANES + tid] = red[u];
    __syncthreads();
    const u32x2 *l2 = reinterpret_cast<const u32x2 *>(lds);
#pragma unroll
    for (int j = 0; j < 2 * VPT; ++j) {
        const u32x2 t = l2[j * LANES + tid];
        Quad<uint16_t> q;
        q.d[0] = t[0];
        q.d[1] = t[1];
        sgd_quad(q, pr[j], vr[j], a);
    }
}

// How a 16 KiB tile is shared out (K <= 8): one 16-byte vector of every copy per lane, i.e. 4 workgroups of 256 lanes
// per tile or 16 of 64.
template <typename T> struct FsgdShape {
    static constexpr int QPV = Elem<T>::VE / 4;                  // quads per vector
};

// Everything that is not a full solid tile: vectors wholly inside one tensor one per lane with the
// loads of all copies, p and v in flight together (K > 8: four copies at a time); the elements of
// the others one per lane (each_cut_elem).  tv.ptr = local gradients, tv.ptr2 = parameters;
// momentum and model pointers come from the global pointer table (mom, model: already advanced to
// the tile's first tensor).  KC: K at compile time, or 0.
template <typename T, int KC, bool DEVW, int LANES, typename V, typename W>
__device__ __forceinline__ void fsgd_mixed(const V &tv, int nt, const TileGeom &g, const void *const *pp, int K_,
                                           const W &wts, const KtSgd &a, void *const *mom, void *const *model,
                                           int part, int parts)
{
    constexpr int VE = Elem<T>::VE;
    constexpr int PV = SgdVec<T>::PV;
    const int K = KC ? KC : K_;
    const int nvec = (int)((g.end - g.start) / VE);
    auto peer = [&](int k) { return reinterpret_cast<const T *>(ld_table(pp + k - 1)) + g.start; };
#pragma unroll 1
    for (int v = part * LANES + threadIdx.x; v < nvec; v += parts * LANES) {
        const int64_t e0 = g.start + (int64_t)v * VE;
        const int i = find_owner_v(tv, nt, e0);
        const int64_t r = i >= 0 ? e0 - tv.off[i] : -1;
        if (r < 0 || r + VE > tv.numel[i]) continue;
        u32x4 *pa = reinterpret_cast<u32x4 *>(tv.ptr2[i] + (uintptr_t)r * 4);
        u32x4 *va = reinterpret_cast<u32x4 *>(reinterpret_cast<float *>(mom[i]) + r);
        const u32x4 x0 = ld_vec(reinterpret_cast<const T *>(tv.ptr[i]) + r);
        u32x4 pr[PV], vr[PV];
#pragma unroll
        for (int h = 0; h < PV; ++h) {
            pr[h] = ld_vec(pa + h);
            vr[h] = ld_vec((a.first ? pa : va) + h);
        }
        Acc<T> acc;
        if (KC) {
            u32x4 x[KC ? KC : 1];
#pragma unroll
            for (int k = 1; k < KC; ++k) x[k] = ld_vec(reinterpret_cast<const u32x4 *>(peer(k)) + v);
            acc.first(x0, kt_weight<DEVW>(wts, 0));
#pragma unroll
            for (int k = 1; k < KC; ++k) acc.add(x[k], kt_weight<DEVW>(wts, k));
        } else {
            acc.first(x0, kt_weight<DEVW>(wts, 0));
#pragma unroll 4
            for (int k = 1; k < K; ++k) acc.add(ld_vec(reinterpret_cast<const u32x4 *>(peer(k)) + v), kt_weight<DEVW>(wts, k));
        }
        SgdVec<T>::apply(acc.finish(), pr, vr, a);
#pragma unroll
        for (int h = 0; h < PV; ++h) {
            st_vec(pa + h, pr[h]);
            st_vec(va + h, vr[h]);
            if (model) st_model_quad(reinterpret_cast<uint16_t *>(model[i]) + r + 4 * h, pr[h]);
        }
    }
    each_cut_elem<VE>(tv, nt, g.start, (int)(g.end - g.start), part * LANES + threadIdx.x, parts * LANES,
                      [&](int i, int64_t r, int e) {
                          float *pe = reinterpret_cast<float *>(tv.ptr2[i]) + r;
                          float *ve = reinterpret_cast<float *>(mom[i]) + r;
                          float pv = ld_elem(pe), vv = ld_elem(a.first ? pe : ve);
                          float s = __fmul_rn(kt_weight<DEVW>(wts, 0), widen(ld_elem(reinterpret_cast<const T *>(tv.ptr[i]) + r)));
#pragma unroll
                          for (int k = 1; k < (KC ? KC : 1); ++k) s = __fmaf_rn(kt_weight<DEVW>(wts, k), widen(ld_elem(peer(k) + e)), s);
                          if (!KC) {
#pragma unroll 4
                              for (int k = 1; k < K; ++k) s = __fmaf_rn(kt_weight<DEVW>(wts, k), widen(ld_elem(peer(k) + e)), s);
                          }
                          sgd_elem(widen(narrow<T>(s)), pv, vv, a);
                          st_elem(pe, pv);
                          st_elem(ve, vv);
                          if (model) st_elem(reinterpret_cast<uint16_t *>(model[i]) + r, (uint16_t)f32_to_bf16(pv));
                      });
}

// LDS of a workgroup: the tensor-table slice of a mixed tile, or the reduced
// values of a full solid bf16 tile on their way from vector to quad order.
union FsgdLds {
    LdsTable table;
    u32x4 red[KT_TILE_VECS];
};

template <typename T, int KC, bool DEVW, int LANES, typename W>
__device__ __forceinline__ void fsgd_other_tile(LdsTable &lds, const int64_t *t_offs, const int64_t *t_numel, const KtTile &tl,
                                                const TileGeom &g, const FsgdArgs &f, const void *const *pp, int K,
                                                const W &wts, const KtSgd &a, int part, int parts)
{
    const int nt = tl.nt == 0 ? 1 : tl.nt;
    const void *const *prm = reinterpret_cast<const void *const *>(f.param_ptrs);
    void *const *mom = f.mom_ptrs + tl.t0;
    void *const *model = f.model_ptrs ? f.model_ptrs + tl.t0 : nullptr;
    if (nt <= KT_LDS_TENSORS) {
        const LdsView tv = stage_lds<LANES>(lds, t_offs, t_numel, f.local_ptrs, prm, tl.t0, nt);
        fsgd_mixed<T, KC, DEVW, LANES>(tv, nt, g, pp, K, wts, a, mom, model, part, parts);
    } else {
        const GlobalView tv = global_view(t_offs, t_numel, f.local_ptrs, prm, tl.t0);
        fsgd_mixed<T, KC, DEVW, LANES>(tv, nt, g, pp, K, wts, a, mom, model, part, parts);
    }
}

// K = 1..8.  SPLIT workgroups share a tile; on a full solid tile the loads of all copies, of p and
// of v are in flight together.  The kernel reads K * s + 8 bytes (24 and 40 at K = 8) and writes
// 8 or 10 per element, and what bounds it is how well the memory system mixes the two: the fewer
// bytes the chip has in flight beyond what hides the latency the better, in small workgroups (FsgdLaunch).
template <typename T, int K, bool DEVW, int LANES>
__global__ __launch_bounds__(LANES) void kt_fused_sgd_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                                const int64_t *t_offs, const void *const *local_ptrs,
                                                                const void *const *peer_ptrs, void *const *param_ptrs,
                                                                uint32_t order, void *const *mom_ptrs,
                                                                void *const *model_ptrs, const int64_t *t_numel, KtSgd a_in,
                                                                FewWeights wts)
{
    const FsgdArgs f{local_ptrs, peer_ptrs, param_ptrs, mom_ptrs, model_ptrs};
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = 1, SPLIT = KT_TILE_VECS / LANES, QPL = VPT * FsgdShape<T>::QPV;
    constexpr int KP = K > 1 ? K - 1 : 1;
    __shared__ FsgdLds lds;

    const unsigned piece = kt_piece(order);
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    const void *const *pp = f.peer_ptrs + (int64_t)tl.bucket * (K - 1);   // peers 1..K-1 of this bucket
    const T *x[KP];
#pragma unroll
    for (int k = 1; k < K; ++k) x[k - 1] = reinterpret_cast<const T *>(ld_table(pp + k - 1));
    TensorSide<T> t(f, tl.t0);
    const KtSgd a = resolve_sgd(a_in);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;

    if (tl.nt == 0 && g.end - g.start == TILE_ELEMS) {
        t.advance(g.start - t_off);
        const int v0 = part * VPT * LANES + tid;       // the lane's first vector in the tile
        const int q0 = part * QPL * LANES + tid;       // and its first quad of p, v and the model copy
        u32x4 r[VPT][K], pr[QPL], vr[QPL];
        u32x4 *p4 = reinterpret_cast<u32x4 *>(t.p) + q0, *v4 = reinterpret_cast<u32x4 *>(t.v) + q0;
        u32x4 *vs = a.first ? p4 : v4;                     // a first step does not read the momentum
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            r[u][0] = ld_vec(reinterpret_cast<const u32x4 *>(t.src) + v0 + u * LANES);
#pragma unroll
            for (int k = 1; k < K; ++k)
                r[u][k] = ld_vec(reinterpret_cast<const u32x4 *>(x[k - 1] + g.start) + v0 + u * LANES);
        }
#pragma unroll
        for (int j = 0; j < QPL; ++j) {
            pr[j] = ld_vec(p4 + j * LANES);
            vr[j] = ld_vec(vs + j * LANES);
        }
        // keep every load above the arithmetic: all of them are in flight together
        __builtin_amdgcn_sched_barrier(0);
        u32x4 red[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            Acc<T> acc;
            acc.first(r[u][0], kt_weight<DEVW>(wts, 0));
#pragma unroll
            for (int k = 1; k < K; ++k) acc.add(r[u][k], kt_weight<DEVW>(wts, k));
            red[u] = acc.finish();
        }
        update_quads<VPT, LANES>(red, lds.red, pr, vr, a, T(0));
        u32x2 *m2 = t.m ? reinterpret_cast<u32x2 *>(t.m) + q0 : nullptr;
        st_quads<QPL, LANES>(p4, v4, m2, pr, vr);
        return;
    }
    fsgd_other_tile<T, K, DEVW, LANES>(lds.table, t_offs, t_numel, tl, g, f, pp, K, wts, a, part, SPLIT);
}

// K = 9..64: full solid tiles take the peers in chunks with the accumulators in registers; every other
// tile as above.  SPLIT workgroups share a tile (fsgd_manyk_shape).  Chunks, not sum_rolling, on quarter tiles: p and
// v are in flight beside them, and the rolling form is 1-5 % slower (K = 9 fp32 19 874 tiles 672 us, 695).
template <typename T, bool DEVW, int SPLIT>
__global__ __launch_bounds__(KT_BLOCK) void kt_fused_sgd_manyk_kernel(const KtTile *tiles, const int64_t *b_elems,
                                                                      const int64_t *t_offs, const void *const *local_ptrs,
                                                                      const void *const *peer_ptrs, void *const *param_ptrs, uint32_t order, int K,
                                                                      void *const *mom_ptrs, void *const *model_ptrs,
                                                                      const int64_t *t_numel, KtSgd a_in,
                                                                      KtWindow win, AllWeights wts)
{
    const FsgdArgs f{local_ptrs, peer_ptrs, param_ptrs, mom_ptrs, model_ptrs};
    constexpr int VE = Elem<T>::VE;
    constexpr int64_t TILE_ELEMS = (int64_t)KT_TILE_VECS * VE;
    constexpr int VPT = KT_TILE_VECS / KT_BLOCK / SPLIT, QPL = VPT * FsgdShape<T>::QPV;
    __shared__ FsgdLds lds;

    const unsigned piece = SPLIT == 1 ? blockIdx.x : kt_piece(order);
    const int part = (int)(piece % SPLIT);
    const KtTile tl = ld_tile(tiles + piece / SPLIT);
    const int64_t b_n = ld_table(b_elems + tl.bucket), t_off = ld_table(t_offs + tl.t0);
    TensorSide<T> t(f, tl.t0);
    const KtSgd a = resolve_sgd(a_in);
    const TileGeom g = tile_geom(tl, b_n, TILE_ELEMS);
    const int tid = threadIdx.x;
    const void *const *pp = f.peer_ptrs + (int64_t)g.bucket * (K - 1);

    if (tl.nt == 0 && g.end - g.start == TILE_ELEMS) {
        t.advance(g.start - t_off);
        const int v0 = part * VPT * KT_BLOCK + tid;       // the lane's first vector in the tile
        const int q0 = part * QPL * KT_BLOCK + tid;       // and its first quad of p, v and the model copy
        u32x4 red[VPT], pr[QPL], vr[QPL];
        u32x4 *p4 = reinterpret_cast<u32x4 *>(t.p) + q0, *v4 = reinterpret_cast<u32x4 *>(t.v) + q0;
        u32x4 *vs = a.first ? p4 : v4;
        auto load_state = [&] {
#pragma unroll
            for (int j = 0; j < QPL; ++j) {
                pr[j] = ld_vec(p4 + j * KT_BLOCK);
                vr[j] = ld_vec(vs + j * KT_BLOCK);
            }
        };
        if (SPLIT > 1) load_state();                      // in flight with the first copies
        Acc<T> acc[VPT];
        sum_in_chunks<T, VPT, DEVW>(acc, [&](int k) { return k == 0 ? t.src : reinterpret_cast<const T *>(ld_table(pp + k - 1)) + g.start; },
                              wts, K, v0);
#pragma unroll
        for (int u = 0; u < VPT; ++u) red[u] = acc[u].finish();
        if (SPLIT == 1) load_state();
        update_quads<VPT, KT_BLOCK>(red, lds.red, pr, vr, a, T(0));
        if (SPLIT == 1) kt_wait_store_window(win);
        st_quads<QPL, KT_BLOCK>(p4, v4, t.m ? reinterpret_cast<u32x2 *>(t.m) + q0 : nullptr, pr, vr);
        return;
    }
    fsgd_other_tile<T, 0, DEVW, KT_BLOCK>(lds.table, t_offs, t_numel, tl, g, f, pp, K, wts, a, part, SPLIT);
}

// Bytes of LDS asked for beyond the kernel's own, to hold the number of workgroups per CU.  Without, registers allow 7 or 8 of
// 256 lanes and LDS 9 of 64 (each keeps the 16 KiB table of a mixed tile).
constexpr unsigned FSGD_LDS_2 = kt_hold_lds(2, sizeof(FsgdLds)), FSGD_LDS_4 = kt_hold_lds(4, sizeof(FsgdLds));

// Workgroups, bytes in flight and order by the size of the launch.  Stores are non-temporal throughout.
//   bf16    2 workgroups of 256 lanes per CU (96 KiB in flight at K = 8) above 2 048 tiles, above 1 024 for one and
//           two copies: K = 4, 21 135 tiles 791 -> 745 us.  Below, the chip is
//           not full long enough to gain (300 to 1 200 tiles, K = 1 to 6: 1-6 % slower with it on aligned sets).
//           Of 3 and more copies from 12 288 tiles on (8 copies: 8 192) workgroups of 64 lanes, 4 per CU for 8 copies (48 KiB in
//           flight), 5 for 5 to 7, 6 for 3 and 4.  Against 2 of 256 lanes, on the buffers of the call before / after 1 GiB of other reads
//           (below): K = 8 9 686 tiles 467 -> 440 / 462 -> 441 us, 39 961 tiles 1 827 -> 1 755 / 1 802 -> 1 750, 1.3B set 7 311 -> 7 160 /
//           7 315 -> 7 059; K = 6 13 725 tiles 576 -> 552 / 570 -> 543; K = 4 39 961 tiles 1 387 -> 1 305 / 1 356 -> 1 283; K = 3 13 725
//           tiles 456 -> 430 / 440 -> 429, 9 686 tiles 304 -> 309 after other reads, which is where the line comes from.  One and two
//           copies: 0-3 % faster, 2-4 % slower after other reads
//   fp32    above 4 096 tiles 2 workgroups per CU for 4 and more copies (K = 8, 21 135 tiles 716 -> 687 us,
//           K = 4, 8 192 tiles 181 -> 179 us), 4 for fewer (K = 2, 21 135 tiles 340 -> 336 us); 6 and more
//           copies from 2 048 tiles on (K = 8, 3 700 tiles 2-5 % over none).  System-scope stores gain 2-12 % up to 2 700
//           tiles where a call finds p and v of the call before in the last-level cache and lose 1-5 % where it does not (1 950
//           tiles, K = 2 and 4, nine sets of buffers in turn), which is the state a training step is called in
// Runs (kt_order) of 64 KiB of gradient per XCD for fp32 of 4 and more copies, else of 128, for launches that hold nothing, from 640
// tiles on: fp32 K = 4 2 587 tiles 58.7 -> 56.8 us on the buffers of the call before, 59.6 -> 59.0 after other reads, bf16 K = 6 1 294 tiles
// 57.0 -> 55.7 / 59.6 -> 57.8.  Held launches gain 1-5 % from runs on the buffers of the call before and lose up to 15 %, for the
// whole launch, after 320 MiB and more of ordinary reads or writes of other data, as a backward pass makes (1.3B set in runs 7 474 / 7 912
// us, in launch order 7 225 / 7 260; fp32 K = 4 19 375 tiles 414 -> 398 / 394 -> 425, K = 7 44 031 tiles 1 313 -> 1 269 / 1 253 -> 1 307; bf16
// K = 6 94 645 tiles 3 856 -> 3 895 / 3 793 -> 4 378); one pass over the set ends that state.  Not below
// 640 tiles, where the few slow tiles that hold many tensors come to lie on one XCD (MobileNetV2, 547 tiles 13.2 -> 13.5 us; 197
// tiles of odd tensors 13.1 -> 13.7).
struct FsgdLaunch {
    unsigned lds;
    int lanes, run;
};
template <typename T> FsgdLaunch fsgd_launch(int K, int64_t ntiles)
{
    if (sizeof(T) == 2) {
        if (K >= 3 && ntiles >= (K >= 8 ? 8192 : 12288))
            return FsgdLaunch{kt_hold_lds(K >= 8 ? 4 : K >= 5 ? 5 : 6, sizeof(FsgdLds)), 64, 0};
        if (ntiles > (K <= 2 ? 1024 : 2048)) return FsgdLaunch{FSGD_LDS_2, KT_BLOCK, 0};
    } else if (ntiles > (K >= 6 ? 2048 : 4096)) {
        return FsgdLaunch{K >= 4 ? FSGD_LDS_2 : FSGD_LDS_4, KT_BLOCK, 0};
    }
    return FsgdLaunch{0u, KT_BLOCK, ntiles < 640 ? 0 : sizeof(T) == 4 && K >= 4 ? 65536 : 131072};
}

// 9 and more copies.  Small launches take quarter tiles (K = 16: 29 tiles fp32 18.9 -> 6.6 us, 249 tiles bf16
// 27.8 -> 19.2, 597 tiles fp32 42.5 -> 36.4; nearly one round of four whole tiles per CU does better with these: K = 9
// from 640 tiles on, K = 12 even at 900), large ones quarter tiles held at two per CU (K = 12 bf16 2 700 tiles
// even, 7 900 tiles 458 -> 422 us, 20 449 tiles 1 208 -> 1 104; K = 16 fp32 20 749 tiles 1 232 -> 1 169).
inline KtShape fsgd_manyk_shape(int K, int64_t nt)
{
    if (nt >= 2560) return {4, 2};
    return {nt <= (K < 12 ? 640 : 896) ? 4 : 1, 0};
}

// Large launches of many copies write little enough (fp32, K = 16: 10 % of the bytes) for the store window of the reduce
// and the fused pass: fp32 from 11 copies on (20 000 tiles: K = 12 924 -> 883 us against held quarter tiles, K = 16
// 1 157 -> 1 066, start 1 221; K = 10 710 us, 740 in the window), bf16 from 14 on with the longest period (K = 16
// with the model copy 1 472 -> 1 411, K = 13 1 262 us against 1 248), smaller ones even or better without (7 900 tiles:
// fp32 K = 12 333 us, 348 in the window, K = 16 429 against 411; bf16 K = 16 561 against 573).
template <typename T> KtWindow fsgd_manyk_window(int K, int64_t nt)
{
    if (K < (sizeof(T) == 2 ? 14 : 11)) return KtWindow{0, 0};
    const int64_t reads = sizeof(T) == 2 ? 196608 : 98304;
    return kt_store_window(sizeof(T) == 2 ? KT_PERIOD_24 : kt_manyk_period(false, K + 2), nt, (reads + K - 1) / K);
}

template <typename T, bool DEVW>
hipError_t launch_fused_sgd_t(const KtDeviceTables &tb, int64_t tile0, int64_t ntiles, const FsgdArgs &f, int K,
                              const KtWeights &w, const KtSgd &a, hipStream_t s)
{
    if (K > 8) {
        const KtWindow win = fsgd_manyk_window<T>(K, ntiles);
        const KtShape sh = win.width ? KtShape{1, 0} : fsgd_manyk_shape(K, ntiles);
        const unsigned lds = kt_shape_lds(sh, (unsigned)sizeof(FsgdLds));
        return launch_in_chunks(tb.tiles + tile0, ntiles, sh.split, [&](const KtTile *tiles, dim3 grid) {
            // runs of 64 KiB per XCD for shared tiles (K = 12 bf16 2 706 tiles 161 -> 153 us, K = 9 bf16 31 528 tiles 1 611 -> 1 534);
            // fp32 of 9 and 10 copies 1 % slower with them (K = 9 19 993 tiles 676 us, 687)
            const uint32_t order = kt_order(grid.x, KT_TILE_BYTES / sh.split, sh.split == 1 || ntiles < 640 || (sizeof(T) == 4 && K < 11) ? 0 : 65536);
#define KT_ARGS \
    tiles, tb.b_elems, tb.t_off, f.local_ptrs, f.peer_ptrs, f.param_ptrs, order, K, f.mom_ptrs, f.model_ptrs, tb.t_numel, a, win, AllWeights(w)
            if (sh.split == 1) kt_fused_sgd_manyk_kernel<T, DEVW, 1><<<grid, dim3(KT_BLOCK), lds, s>>>(KT_ARGS);
            else kt_fused_sgd_manyk_kernel<T, DEVW, 4><<<grid, dim3(KT_BLOCK), lds, s>>>(KT_ARGS);
#undef KT_ARGS
        });
    }
    FsgdLaunch how = fsgd_launch<T>(K, ntiles);
    // nothing held: 64 lanes would still keep 146 KiB of LDS per CU (9 workgroups with the table of a mixed tile each) from kernels
    // beside them, 256 lanes 112-130 (7 or 8)
    if (!kt_may_hold()) how = FsgdLaunch{0u, KT_BLOCK, how.run};
    return launch_in_chunks(tb.tiles + tile0, ntiles, KT_TILE_VECS / how.lanes, [&](const KtTile *tiles, dim3 grid) {
        const uint32_t order = kt_order(grid.x, how.lanes * KT_VEC_BYTES, how.run);
#define KT_LAUNCH(KK, LANES)                                                                                              \
    kt_fused_sgd_kernel<T, KK, DEVW, LANES><<<grid, dim3(LANES), how.lds, s>>>(tiles, tb.b_elems, tb.t_off, f.local_ptrs, \
        f.peer_ptrs, f.param_ptrs, order, f.mom_ptrs, f.model_ptrs, tb.t_numel, a, FewWeights(w))
        switch (K) {
#define KT_CASE(KK)                                                              \
    case KK:                                                                     \
        if constexpr (sizeof(T) == 2 && KK >= 3) {                               \
            if (how.lanes == 64) { KT_LAUNCH(KK, 64); break; }                   \
        }                                                                        \
        KT_LAUNCH(KK, KT_BLOCK);                                                 \
        break;
            KT_CASE(1) KT_CASE(2) KT_CASE(3) KT_CASE(4) KT_CASE(5) KT_CASE(6) KT_CASE(7) KT_CASE(8)
#undef KT_CASE
#undef KT_LAUNCH
        }
    }, how.lanes);
}

}  // namespace

int kt_launch_fused_sgd(const KtDeviceTables &tb, kt_dtype dt, int64_t tile0, int64_t ntiles,
                        const void *const *d_local_ptrs, const void *const *d_peer_ptrs, int K, const KtWeights &w,
                        void *const *d_param_ptrs, void *const *d_mom_ptrs, void *const *d_model_ptrs,
                        const KtSgd &a, void *stream)
{
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const FsgdArgs f{d_local_ptrs, d_peer_ptrs, d_param_ptrs, d_mom_ptrs, d_model_ptrs};
#define KT_FSGD(TT, DD) (int)launch_fused_sgd_t<TT, DD>(tb, tile0, ntiles, f, K, w, a, s)
    if (dt == KT_F32) return w.dev ? KT_FSGD(float, true) : KT_FSGD(float, false);
    return w.dev ? KT_FSGD(uint16_t, true) : KT_FSGD(uint16_t, false);
#undef KT_FSGD
}
