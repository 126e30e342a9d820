// Device-side helpers shared by the kernels: 16-byte global loads/stores,
// bf16 conversion, tile geometry, the tensor-table views of mixed tiles and the
// per-element accumulation of the weighted sum.  Everything is internal to a
// translation unit (anonymous namespace).
#ifndef KT_DEVICE_H
#define KT_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kt_internal.h"

#ifndef KT_NT_LOAD
#define KT_NT_LOAD 1
#endif
#ifndef KT_NT_STORE
#define KT_NT_STORE 1
#endif

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// The same vectors at any element address (2 bytes for bf16, 4 for binary32).  The HSA runtime
// runs kernels in unaligned access mode, so one such access is one global_load/store_dwordx4 at
// any address: a copy loses 1 % (4-byte) to 3.5 % (2-byte) to misaligned loads and 4 % to stores
// that do not start on a 64-byte boundary (512 MiB copied: 6.45 TB/s aligned), where one element
// per lane loses more than half.
typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));

namespace {

template <typename T> struct Elem;
template <> struct Elem<float> { static constexpr int VE = 4; };
template <> struct Elem<uint16_t> { static constexpr int VE = 8; };

// Every data pointer reaches the kernels through a pointer table in memory,
// so the compiler cannot tell that it addresses global memory and would emit
// flat loads/stores.  The data is always in global memory: say so.
#define KT_GLOBAL __attribute__((address_space(1)))

__device__ __forceinline__ u32x4 ld_vec(const void *p)
{
    const KT_GLOBAL u32x4_any *g = (const KT_GLOBAL u32x4_any *)p;
#if KT_NT_LOAD == 2
    return *(const volatile KT_GLOBAL u32x4_any *)g;      // system scope (sc0 sc1), for measurement
#elif KT_NT_LOAD
    return __builtin_nontemporal_load(g);
#else
    return *g;
#endif
}

__device__ __forceinline__ void st_vec(void *p, u32x4 v)
{
    KT_GLOBAL u32x4_any *g = (KT_GLOBAL u32x4_any *)p;
#if KT_NT_STORE == 2
    *(volatile KT_GLOBAL u32x4_any *)g = v;                // system scope (sc0 sc1), for measurement
#elif KT_NT_STORE
    __builtin_nontemporal_store(v, g);
#else
    *g = v;
#endif
}

// Store policy of the kernels that write about as much as they read (pack, unpack, SGD on
// unpack with bf16 gradients: 44-50 % of their bytes are written): a system-scope store, which
// the L2 writes through at once instead of holding the line, measured 1-4 points of 8 TB/s
// better there than the non-temporal store, and 1-3 points worse in the kernels that write a
// quarter of their bytes or less (reduce but for middling launches, reduce_sys; fused pass, K copies -> parameters), which keep
// st_vec.  KT_WT_STORE=0 builds these
// kernels with st_vec as well, for measurement.
#ifndef KT_WT_STORE
#define KT_WT_STORE 1
#endif
template <bool WT> __device__ __forceinline__ void st_vec_copy(void *p, u32x4 v)
{
#if KT_WT_STORE && KT_NT_STORE == 1
    if (WT) {
        *(volatile KT_GLOBAL u32x4_any *)p = v;
        return;
    }
#endif
    st_vec(p, v);
}
// The system-scope store of a tile's vectors as a buffer store (descriptor of `bytes` bytes from a
// uniform base): unlike the volatile store it is not waited for, so a wavefront that has stored
// ends at once and its place goes to the next.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(void *base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}
__device__ __forceinline__ void st_tile_wt(__amdgpu_buffer_rsrc_t rs, int at, u32x4 v)
{
#if KT_WT_STORE && KT_NT_STORE == 1
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, at, 0, 1 | 16);       // sc0 sc1
#else
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, at, 0, 2);            // nt
#endif
}
// The same choice at run time.  The system-scope store wants whole 64-byte pieces: where a
// wavefront's stores start elsewhere it costs 11 % of a copy's rate (5.8 TB/s against 6.58
// aligned), the non-temporal store 4 % (6.28 against 6.45).
__device__ __forceinline__ void st_vec_pick(void *p, u32x4 v, bool wt)
{
    if (wt) st_vec_copy<true>(p, v); else st_vec(p, v);
}

// ---- whole tiles at any address ------------------------------------------------
// The vectors of a full tile are laid out from the destination's 64-byte boundary at or below
// the tile's first byte, so that every store but the first and last of the tile fills whole
// 64-byte pieces wherever the tensor lies; the loads then sit at any address, which costs far
// less (see u32x4_any).  `pos` is a vector's byte position from that boundary and `o` the tile's
// first byte (0..63): positions below `o` belong to the end of the tile, BYTES further on, which
// keeps one vector per lane and the lane numbering.  Where `o` is no multiple of 16 one vector is
// cut in two by the tile's ends; its VE elements are taken one by one (edge_elem).
struct RotVec {
    int at;       // byte offset of the vector from the tile's first byte
    bool whole;   // false: the vector cut in two (`at` is then 0, in bounds)
};
template <int BYTES> __device__ __forceinline__ RotVec rot_vec(int pos, int o)
{
    RotVec r;
    r.whole = pos >= o || pos + KT_VEC_BYTES <= o;
    r.at = r.whole ? (pos >= o ? pos - o : pos + BYTES - o) : 0;
    return r;
}
// Element q (0 <= q < 16 / es) of the cut vector as a byte offset from the tile's first byte.
template <int BYTES> __device__ __forceinline__ int edge_elem(int q, int es, int o)
{
    const int pos = (o & ~(KT_VEC_BYTES - 1)) + q * es;
    return pos >= o ? pos - o : pos + BYTES - o;
}
__device__ __forceinline__ int off64(const void *p) { return (int)(reinterpret_cast<uintptr_t>(p) & 63u); }

// Holds a wave back until the store window opens (KtWindow).  Bounded twice over: the clock
// always advances, so the condition comes true within one period (12 to 24 us), and the
// iteration count ends the loop in any case.  (The low 32 bits of the clock wrap every 43 s at
// 100 MHz; one period is then irregular.)
__device__ __forceinline__ void kt_wait_store_window(const KtWindow &w)
{
    if (w.width) {
        for (int spin = 0; spin < 4096; ++spin) {
            if ((uint32_t)wall_clock64() % w.period < w.width) break;
            __builtin_amdgcn_s_sleep(4);
        }
    }
}

template <typename T> __device__ __forceinline__ T ld_elem(const T *p) { return *(const KT_GLOBAL T *)p; }
template <typename T> __device__ __forceinline__ void st_elem(T *p, T v) { *(KT_GLOBAL T *)p = v; }

// bf16 <-> binary32.  Widening is exact (the bits become the upper half); narrowing is
// round-to-nearest-even, NaN stays quiet NaN with its upper payload bits: two values per
// v_cvt_pk_bf16_f32, which gives the bits of (u + 0x7FFF + ((u >> 16) & 1)) >> 16 for each of the
// 2^32 binary32 patterns (NaN: (u >> 16) | 0x40), in one instruction where the integer form took
// twelve and a branch and made the bf16 kernels three times the size.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t f32_to_bf16x2(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ uint32_t f32_to_bf16(float f) { return f32_to_bf16x2(f, f) & 0xFFFFu; }
// INT: the same bits in integer instructions.  Only for full tiles of the reduce and the fused pass: the
// longer way from the last load to the store spaces the workgroups out.  Launches of 6 and more
// copies that hold their workgroups or use the store window gain 1-5 % (fused, two half tiles per CU: K = 8,
// 21 099 tiles 518 us against 493; K = 6, 24 394 tiles 455 against 431; reduce of the 1.3B set inside the
// windows 3.82 against 3.77 ms), those of whole tiles below 2 048 lose 3-6 %; the fused pass of one
// copy gains 2-5 % from 20 000 tiles on (40 034 tiles of odd tensors 233 us against 224).
__device__ __forceinline__ uint32_t f32_to_bf16_int(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
template <bool INT> __device__ __forceinline__ uint32_t narrow_x2(float lo, float hi)
{
    return INT ? f32_to_bf16_int(lo) | (f32_to_bf16_int(hi) << 16) : f32_to_bf16x2(lo, hi);
}

// scale * x for one element of either storage type
__device__ __forceinline__ float scale_elem(float x, float s) { return __fmul_rn(s, x); }
__device__ __forceinline__ uint16_t scale_elem(uint16_t x, float s)
{
    return (uint16_t)f32_to_bf16(__fmul_rn(s, __uint_as_float((uint32_t)x << 16)));
}

template <typename T, bool INT = false> __device__ __forceinline__ u32x4 scale_vec(u32x4 v, float s)
{
    u32x4 r;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = __float_as_uint(__fmul_rn(s, __uint_as_float(v[c])));
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = narrow_x2<INT>(__fmul_rn(s, bf16_lo(v[c])), __fmul_rn(s, bf16_hi(v[c])));
    }
    return r;
}

// The tables are constant while a kernel runs and every index into them is uniform over the
// workgroup: read through the constant address space they are scalar loads whatever the compiler
// can prove about the stores around them.
#define KT_CONST __attribute__((address_space(4)))
template <typename P> __device__ __forceinline__ P ld_table(const P *p) { return *(const KT_CONST P *)p; }
__device__ __forceinline__ KtTile ld_tile(const KtTile *p)
{
    const u32x4 v = *(const KT_CONST u32x4 *)p;
    return KtTile{(int32_t)v[0], v[1], (int32_t)v[2], (int32_t)v[3]};
}
// Makes a value exist in scalar registers at this point, so that the table loads of a tile are
// issued together and waited for once: the way from the tile record to the first data load is
// two dependent scalar loads (record; lengths and pointers) instead of four.
__device__ __forceinline__ void pin(uint64_t a, uint64_t b, uint64_t c, uint64_t d) { asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d)); }

struct TileGeom {
    int bucket;
    int64_t start;   // first element of the tile inside the bucket
    int64_t end;     // one past the last element (clipped to the bucket length)
};

__device__ __forceinline__ TileGeom tile_geom(const KtTile &tl, int64_t n, int64_t tile_elems)
{
    TileGeom g;
    g.bucket = tl.bucket;
    g.start = (int64_t)tl.tile_in_bucket * tile_elems;
    g.end = g.start + tile_elems < n ? g.start + tile_elems : n;
    return g;
}

// The tile's slice of the tensor table is staged in LDS when it fits, so that
// the per-vector owner search runs on LDS instead of global memory.
struct LdsTable {
    int64_t off[KT_LDS_TENSORS];     // element offset of the tensor in its bucket
    int64_t numel[KT_LDS_TENSORS];   // element count
    uintptr_t ptr[KT_LDS_TENSORS];   // base address (source or destination tensor)
    uintptr_t ptr2[KT_LDS_TENSORS];  // second base address for kernels with two tensor sets
};

// Typed views of the table slice of a mixed tile: in LDS (the usual case) or in
// global memory (more than KT_LDS_TENSORS tensors in one tile).  Keeping the
// address space in the type lets the owner search use LDS instructions.
#define KT_LDS __attribute__((address_space(3)))
struct LdsView {
    const KT_LDS int64_t *off;
    const KT_LDS int64_t *numel;
    const KT_LDS uintptr_t *ptr;
    const KT_LDS uintptr_t *ptr2;
};
struct GlobalView {
    const KT_GLOBAL int64_t *off;
    const KT_GLOBAL int64_t *numel;
    const KT_GLOBAL uintptr_t *ptr;
    const KT_GLOBAL uintptr_t *ptr2;
};

// The table slice of a tile with at most KT_REG_TENSORS tensors (where a large tensor ends and the next begins, with a
// bias or a norm between them) in scalar registers: one more batch of scalar loads behind the tile record's,
// where staging is a vector load, an LDS write, a barrier and a search ahead of the data loads.  Entries from nt on
// repeat the last.  SGD on unpack of bf16 gradients only (kt_sgd.hip): pack, unpack and the fused passes gain 1 % at
// most, small launches of pack lose 10 %.
#define KT_REG_TENSORS 4
template <typename P> struct Regs {
    P a, b, c, d;
    __device__ __forceinline__ P operator[](int i) const
    {
        // all four read first: a choice between their addresses would put them in scratch memory
        const P p = a, q = b, r = c, s = d;
        const P lo = i >= 1 ? q : p, hi = i >= 3 ? s : r;
        return i >= 2 ? hi : lo;
    }
};
struct RegView {
    Regs<int64_t> off, numel;
    Regs<uintptr_t> ptr, ptr2;
};
template <typename P, typename Q> __device__ __forceinline__ Regs<P> ld_regs(const Q *table, int t0, int nt)
{
    const Q *t = table + t0;
    return Regs<P>{(P)ld_table(t), (P)ld_table(t + (nt > 1 ? 1 : 0)), (P)ld_table(t + (nt > 2 ? 2 : nt - 1)), (P)ld_table(t + nt - 1)};
}
__device__ __forceinline__ RegView reg_view(const int64_t *t_off, const int64_t *t_numel, const void *const *first,
                                            const void *const *second, int t0, int nt)
{
    return RegView{ld_regs<int64_t>(t_off, t0, nt), ld_regs<int64_t>(t_numel, t0, nt), ld_regs<uintptr_t>(first, t0, nt),
                   ld_regs<uintptr_t>(second, t0, nt)};
}
__device__ __forceinline__ int find_owner_v(const RegView &tv, int nt, int64_t e)
{
    const int n = (tv.off.a <= e) + (tv.off.b <= e) + (tv.off.c <= e) + (tv.off.d <= e);
    return (n < nt ? n : nt) - 1;
}

template <typename V> __device__ __forceinline__ int find_owner_v(const V &tv, int nt, int64_t e)
{
    int lo = 0, hi = nt;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tv.off[mid] <= e) lo = mid + 1; else hi = mid;
    }
    return lo - 1;
}

// Calls f(q, i, r) for every element e0 + q (0 <= q < N) below `lim` that belongs to a tensor:
// element r of the tile's i-th tensor.  `i` is the owner of e0 (find_owner_v).  Only the owner
// search of successive elements depends on the one before; loads issued by f stay in flight.
template <int N, typename V, typename F>
__device__ __forceinline__ void each_owned(const V &tv, int nt, int i, int64_t e0, int64_t lim, F f)
{
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int64_t e = e0 + q;
        while (i + 1 < nt && tv.off[i + 1] <= e) ++i;
        if (i >= 0 && e < lim) {
            const int64_t r = e - tv.off[i];
            if (r < tv.numel[i]) f(q, i, r);
        }
    }
}

// Calls f(i, r, e) for every element of the tile (length `len`, at bucket element `start`) that lies
// in a vector not wholly inside one tensor: the elements of each tensor before its first whole
// vector of the tile and after its last.  `i` is the tensor, `r` the element in it, `e` the element
// in the tile.  One element per lane and call, so that the few cut vectors of a tile cost one
// memory latency and little code; `first` and `stride` share the work out over the lanes.
// Every tensor takes 2 * VE places that way, whatever its size.  Where these take more turns than
// going through the tile's vectors element by element would (tensors of a few elements: 512 and
// more in a full tile) the vectors are gone through instead.  8 000 tensors of one element, bf16,
// dense: unpack 49 us by places, 10 by vectors; fused pass 236, 43; one-pass SGD 98, 16.
template <int VE, typename V, typename F>
__device__ __forceinline__ void each_cut_elem(const V &tv, int nt, int64_t start, int len, int first, int stride, F f)
{
    const int nvec = (len + VE - 1) / VE;
    if ((nt * 2 * VE + stride - 1) / stride >= VE * ((nvec + stride - 1) / stride)) {
#pragma unroll 1
        for (int v = first; v < nvec; v += stride) {
            const int64_t e0 = start + (int64_t)v * VE;
            int i = find_owner_v(tv, nt, e0);
            if (i >= 0 && e0 - tv.off[i] + VE <= tv.numel[i]) continue;
#pragma unroll 1
            for (int e = v * VE; e < len && e < v * VE + VE; ++e) {
                while (i + 1 < nt && tv.off[i + 1] <= start + e) ++i;
                if (i < 0) continue;
                const int64_t r = start + e - tv.off[i];
                if (r < tv.numel[i]) f(i, r, e);
            }
        }
        return;
    }
    for (int idx = first; idx < nt * 2 * VE; idx += stride) {
        const int i = idx / (2 * VE), slot = idx % (2 * VE);
        const int64_t rel = tv.off[i] - start, last = rel + tv.numel[i];
        const int a = rel > 0 ? (int)(rel < len ? rel : len) : 0;             // the tensor's part of the tile: [a, b)
        const int b = last > 0 ? (int)(last < len ? last : len) : 0;
        const int body = (a + VE - 1) / VE * VE;
        const int e = slot < VE ? a + slot : b / VE * VE + slot - VE;
        if (e < b && (slot < VE ? e < body : e >= body)) f(i, (int64_t)e - rel, e);
    }
}

// VE elements held one per register <-> a 16-byte vector
__device__ __forceinline__ u32x4 join(const float *x)
{
    return u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
}
__device__ __forceinline__ u32x4 join(const uint16_t *x)
{
    u32x4 r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = (uint32_t)x[2 * c] | ((uint32_t)x[2 * c + 1] << 16);
    return r;
}
template <typename T> __device__ __forceinline__ T elem_of(u32x4 v, int q);
template <> __device__ __forceinline__ float elem_of<float>(u32x4 v, int q) { return __uint_as_float(v[q]); }
template <> __device__ __forceinline__ uint16_t elem_of<uint16_t>(u32x4 v, int q)
{
    return (uint16_t)(v[q >> 1] >> (16 * (q & 1)));
}

// The elements [e0, e0 + VE) of a vector that is not wholly inside one tensor, 0 where none owns one.
template <typename T, typename V>
__device__ __forceinline__ u32x4 gather_vec(const V &tv, int nt, int i, int64_t e0, int64_t lim)
{
    constexpr int VE = Elem<T>::VE;
    T x[VE];
#pragma unroll
    for (int q = 0; q < VE; ++q) x[q] = 0;
    each_owned<VE>(tv, nt, i, e0, lim, [&](int q, int t, int64_t r) { x[q] = ld_elem(reinterpret_cast<const T *>(tv.ptr[t]) + r); });
    return join(x);
}
// `second` may be NULL for kernels with one tensor set (ptr2 then mirrors ptr).
template <int LANES = KT_BLOCK>
__device__ __forceinline__ LdsView stage_lds(LdsTable &lds, const int64_t *t_off, const int64_t *t_numel,
                                             const void *const *first, const void *const *second, int t0, int nt)
{
    for (int i = threadIdx.x; i < nt; i += LANES) {
        lds.off[i] = t_off[t0 + i];
        lds.numel[i] = t_numel[t0 + i];
        lds.ptr[i] = reinterpret_cast<uintptr_t>(first[t0 + i]);
        lds.ptr2[i] = reinterpret_cast<uintptr_t>(second ? second[t0 + i] : first[t0 + i]);
    }
    __syncthreads();
    LdsView v;
    v.off = (const KT_LDS int64_t *)lds.off;
    v.numel = (const KT_LDS int64_t *)lds.numel;
    v.ptr = (const KT_LDS uintptr_t *)lds.ptr;
    v.ptr2 = (const KT_LDS uintptr_t *)lds.ptr2;
    return v;
}

__device__ __forceinline__ GlobalView global_view(const int64_t *t_off, const int64_t *t_numel,
                                                  const void *const *first, const void *const *second, int t0)
{
    GlobalView v;
    v.off = (const KT_GLOBAL int64_t *)(t_off + t0);
    v.numel = (const KT_GLOBAL int64_t *)(t_numel + t0);
    v.ptr = (const KT_GLOBAL uintptr_t *)(reinterpret_cast<const uintptr_t *>(first) + t0);
    v.ptr2 = (const KT_GLOBAL uintptr_t *)(reinterpret_cast<const uintptr_t *>(second ? second : first) + t0);
    return v;
}

// The weights as a kernel argument.  Kernels for up to 8 copies take 8 of them: a launch copies its
// argument block to the device, and 340 bytes of it cost the host 3.4 us a launch against 2.8 for 48.
template <int N> struct WeightArgs {
    float w[N];
    const float *dev;
    explicit WeightArgs(const KtWeights &f) : dev(f.dev)
    {
        for (int k = 0; k < N; ++k) w[k] = f.w[k];
    }
};
using FewWeights = WeightArgs<8>;
using AllWeights = WeightArgs<KT_MAX_PEERS>;

// Weight of peer k: from the kernel-argument block, or, when the caller asked for
// the plan's device-resident weights, from device memory (uniform scalar reads).
// (a template parameter, so that launches with weights by value run exactly the code they
// would without this choice.)
template <bool DEVW, typename W> __device__ __forceinline__ float kt_weight(const W &wts, int k)
{
    if (DEVW) return ld_table(wts.dev + k);
    return wts.w[k];
}

// ---- weighted sum of one 16-byte vector per peer ---------------------------
// Per element: acc = w0*x0 (rounded), then acc = fma(wk, xk, acc), ascending k.

template <typename T> struct Acc;
template <> struct Acc<float> {
    float a[4];
    __device__ __forceinline__ void first(u32x4 x, float w)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) a[c] = __fmul_rn(w, __uint_as_float(x[c]));
    }
    __device__ __forceinline__ void add(u32x4 x, float w)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) a[c] = __fmaf_rn(w, __uint_as_float(x[c]), a[c]);
    }
    template <bool INT = false> __device__ __forceinline__ u32x4 finish() const
    {
        u32x4 r;
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = __float_as_uint(a[c]);
        return r;
    }
};
template <> struct Acc<uint16_t> {
    float a[8];
    __device__ __forceinline__ void first(u32x4 x, float w)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            a[2 * c] = __fmul_rn(w, bf16_lo(x[c]));
            a[2 * c + 1] = __fmul_rn(w, bf16_hi(x[c]));
        }
    }
    __device__ __forceinline__ void add(u32x4 x, float w)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            a[2 * c] = __fmaf_rn(w, bf16_lo(x[c]), a[2 * c]);
            a[2 * c + 1] = __fmaf_rn(w, bf16_hi(x[c]), a[2 * c + 1]);
        }
    }
    template <bool INT = false> __device__ __forceinline__ u32x4 finish() const
    {
        u32x4 r;
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = narrow_x2<INT>(a[2 * c], a[2 * c + 1]);
        return r;
    }
};

// ---- K > 8 -------------------------------------------------------------------
// The peers are taken in chunks of at most Chunk<T>::N, ascending, with the
// accumulators of the tile's vectors kept in registers across chunks, so that a
// lane still has (vectors per lane) x (chunk) loads in flight at a time and the
// per-element order of operations is the one of the definition (product for
// k = 0, then one fused multiply-add per peer in ascending k).  `ptr(k)` gives
// peer k's data at the tile start.
template <typename T> struct Chunk;
template <> struct Chunk<float> { static constexpr int N = 8; };       // 148 VGPRs, 3 waves per SIMD
template <> struct Chunk<uint16_t> { static constexpr int N = 6; };    // 8 accumulators per vector: 6 keeps 3 waves per SIMD

template <typename T, int VPT, int KC, bool DEVW, typename P>
__device__ __forceinline__ void sum_chunk(Acc<T> *acc, P ptr, const AllWeights &wts, int k0, int v0)
{
    u32x4 r[VPT][KC];
#pragma unroll
    for (int j = 0; j < KC; ++j) {
        const u32x4 *x = reinterpret_cast<const u32x4 *>(ptr(k0 + j));
#pragma unroll
        for (int u = 0; u < VPT; ++u) r[u][j] = ld_vec(x + u * KT_BLOCK + v0);
    }
#pragma unroll
    for (int j = 0; j < KC; ++j) {
        const float w = kt_weight<DEVW>(wts, k0 + j);
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            if (j == 0 && k0 == 0) acc[u].first(r[u][j], w); else acc[u].add(r[u][j], w);
        }
    }
}

// acc[u] = sum over all K peers of the vectors v0 + u * KT_BLOCK of a full tile.
template <typename T, int VPT, bool DEVW, typename P>
__device__ __forceinline__ void sum_in_chunks(Acc<T> *acc, P ptr, const AllWeights &wts, int K, int v0)
{
    constexpr int CH = VPT == 1 ? 8 : Chunk<T>::N;         // quarter tiles: 32 KB of a workgroup's loads in flight
    int k0 = 0;
#pragma unroll 1
    for (; k0 + CH <= K; k0 += CH) sum_chunk<T, VPT, CH, DEVW>(acc, ptr, wts, k0, v0);
    switch (K - k0) {      // the last, shorter chunk (uniform over the grid)
    case 1: sum_chunk<T, VPT, 1, DEVW>(acc, ptr, wts, k0, v0); break;
    case 2: sum_chunk<T, VPT, 2, DEVW>(acc, ptr, wts, k0, v0); break;
    case 3: sum_chunk<T, VPT, 3, DEVW>(acc, ptr, wts, k0, v0); break;
    case 4: sum_chunk<T, VPT, 4, DEVW>(acc, ptr, wts, k0, v0); break;
    case 5: sum_chunk<T, VPT, 5, DEVW>(acc, ptr, wts, k0, v0); break;
    case 6: if (CH > 6) sum_chunk<T, VPT, 6, DEVW>(acc, ptr, wts, k0, v0); break;
    case 7: if (CH > 7) sum_chunk<T, VPT, 7, DEVW>(acc, ptr, wts, k0, v0); break;
    default: break;
    }
}

// The same for one vector (quarter tiles), rolling: the load of copy k + 8 is issued as copy k is summed, so
// that the number in flight does not sink to 0 between chunks.  Even with chunks from 12 copies on, and
// better where the last chunk is short (reduce of 20 000 tiles, held at two workgroups per CU, K = 9: fp32 532 -> 508 us,
// bf16 547 -> 520).  A sum that starts from -0 is the product of the first copy, zeros' signs included.
template <typename T, int R, bool DEVW, typename P>
__device__ __forceinline__ void roll_tail(Acc<T> &acc, u32x4 *r, P ptr, const AllWeights &wts, int k0, int v0)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        acc.add(r[j], kt_weight<DEVW>(wts, k0 + j));
        if (j < R) r[j] = ld_vec(reinterpret_cast<const u32x4 *>(ptr(k0 + 8 + j)) + v0);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) acc.add(r[j], kt_weight<DEVW>(wts, k0 + 8 + j));
}
template <typename T, bool DEVW, typename P>
__device__ __forceinline__ void sum_rolling(Acc<T> &acc, P ptr, const AllWeights &wts, int K, int v0)
{
    u32x4 r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = ld_vec(reinterpret_cast<const u32x4 *>(ptr(j)) + v0);
#pragma unroll
    for (int c = 0; c < Elem<T>::VE; ++c) acc.a[c] = -0.0f;
    int k0 = 0;
#pragma unroll 1
    for (; k0 + 16 <= K; k0 += 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            acc.add(r[j], kt_weight<DEVW>(wts, k0 + j));
            r[j] = ld_vec(reinterpret_cast<const u32x4 *>(ptr(k0 + 8 + j)) + v0);
        }
    }
    switch (K - k0 - 8) {      // uniform over the grid
    case 0: roll_tail<T, 0, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 1: roll_tail<T, 1, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 2: roll_tail<T, 2, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 3: roll_tail<T, 3, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 4: roll_tail<T, 4, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 5: roll_tail<T, 5, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 6: roll_tail<T, 6, DEVW>(acc, r, ptr, wts, k0, v0); break;
    case 7: roll_tail<T, 7, DEVW>(acc, r, ptr, wts, k0, v0); break;
    default: break;
    }
}

__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }
template <typename T> __device__ __forceinline__ T narrow(float a);
template <> __device__ __forceinline__ float narrow<float>(float a) { return a; }
template <> __device__ __forceinline__ uint16_t narrow<uint16_t>(float a) { return (uint16_t)f32_to_bf16(a); }

// ---- order of the pieces of a launch -------------------------------------------
// Workgroups go to the 8 XCDs in turn: in launch order neighbouring pieces of a bucket are read by different XCDs.
// With an order each XCD takes runs of 2^g pieces instead, the 8 runs of a group side by side, so that the chip still
// sweeps every stream over a front of half a megabyte or one.  The memory system takes a mix of reads and few writes 3-6 %
// faster that way (flat buffers, 8 reads and one write, two workgroups of 4 KiB of each per CU: 5.80 TB/s in
// launch order, 6.12 with runs of 16 KiB, 6.32 with 64 KiB and more); reads alone and copies are even, and which XCD has which
// run makes no difference.  Launches of few bytes in flight are slower with runs instead, for as long as they last, when 320 MiB or more
// of ordinary reads or writes of other data came before them (non-temporal reads do not count; one pass over the same buffers ends
// it): each kernel's rule says where runs hold in both states.  `order`: pieces in whole groups in the upper bits, g in the lower three; 0 is launch
// order.  The remainder of a launch keeps the launch order.
__device__ __forceinline__ unsigned kt_piece(uint32_t order)
{
    const unsigned b = blockIdx.x, g = order & 7u;
    if (b >= (order & ~7u)) return b;
    const unsigned hi = b >> 3;
    return (hi >> g << (3 + g)) | ((b & 7u) << g) | (hi & ((1u << g) - 1));
}
// The order for a launch of `pieces` workgroups of `piece_bytes` each with runs of `run` bytes (powers of two, at most 128
// pieces a run; 0: launch order).
inline uint32_t kt_order(unsigned pieces, int piece_bytes, int run)
{
    uint32_t g = 0;
    while (g < 7 && (piece_bytes << g) < run) ++g;
    return g ? (pieces >> (3 + g) << (3 + g)) | g : 0u;
}

// A grid may not hold 2^32 or more lanes: very large plans go in several launches.  `split`
// workgroups of `lanes` share a tile; launch(tiles, grid) launches one part.
template <typename F> hipError_t launch_in_chunks(const KtTile *tiles, int64_t ntiles, int split, F launch, int lanes = KT_BLOCK)
{
    const int64_t per_launch = (((int64_t)1 << 32) / lanes - 1) / split;
    for (int64_t done = 0; done < ntiles; done += per_launch) {
        const int64_t now = ntiles - done < per_launch ? ntiles - done : per_launch;
        launch(tiles + done, dim3((unsigned)(now * split)));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

#endif
