// gs_kernels.hip -- gfx950 kernels of the per-layer optimizer step and their launchers.
//
// The work is one streaming pass over 2k+26 bytes per parameter (k bf16 gradient streams and
// the fp32 p/m/v streams in, p/m/v and the bf16 weight out) with ~100 VALU lane-ops per
// element: HBM-bound, so there is no MFMA here.  Measured on MI355X, what decides the achieved
// bandwidth of such a many-stream read+write pass is the shape of the memory traffic:
//   * every wave-level memory instruction covers whole, contiguous 128-byte lines.  A lane of the
//     step owns 2 consecutive elements (a 4-byte load per bf16 stream, an 8-byte one per fp32
//     stream): the window of addresses that all resident waves touch together is then half as wide
//     as with 4 elements per lane, and HBM serves it 1-12 % faster;
//   * workgroups are NOT persistent: one 256-element tile per workgroup, dispatched in order, keeps
//     the set of addresses in flight compact, which HBM rewards (a grid-stride loop costs 30-40 %
//     on stores on this part);
//   * the bytes in flight are held to what HBM serves best, by how many workgroups a CU may hold
//     (room_for) and not by making waves wait between their accesses; stores go out back to back and are
//     written through;
//   * ranges that do not fill the chip are bound by the latency of a wave's serial chain instead,
//     and take shapes that put every load in flight (step_shape);
//   * every stream is touched once, so loads and stores carry the non-temporal hint.
// The norm pass is read-only and does best with short contiguous spans of tiles per workgroup.
//
// Partition independence (Sec. 6.5 of the paper: results must not depend on the partition
// ratio): every element goes through the same update function `adamw_element`, compiled with
// floating-point contraction off, whether it is reached through a vector body or through
// the per-element path used for ragged range ends.  Grouping is by ABSOLUTE element index
// (groups of 2 or 4 starting at multiples of their size), and no element's result depends on its
// group, so a range split at any point is processed with bit-identical arithmetic.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gs_internal.h"

#pragma clang fp contract(off)

namespace gs {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The group of EL consecutive elements a lane owns: its fp32 and its bf16 vector.
template <int EL> struct Group;
template <> struct Group<2> { typedef f32x2 F; typedef uint32_t H; };
template <> struct Group<4> { typedef f32x4 F; typedef u32x2 H; };

template <typename T> using global_ptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ global_ptr<T> in_global(T *p) { return (global_ptr<T>)p; }

// ---- memory access helpers: streams are touched exactly once => non-temporal ------------
// KEEP: without the hint, which leaves the line in the memory-side cache.
template <bool KEEP = false, typename T>
__device__ __forceinline__ T ld_stream(const T *p)
{
    if constexpr (KEEP) return *p;
    else return __builtin_nontemporal_load(p);
}
template <bool KEEP = false, typename T>
__device__ __forceinline__ void st_stream(T *p, T v)
{
    if constexpr (KEEP) *p = v;
    else __builtin_nontemporal_store(v, p);
}

// THROUGH: with the hint and past its XCD's L2 too, which otherwise keeps the line dirty and sends it out
// later, in an order of its own (step, 805 M, k = 16, no other change: 7.39 ms against 7.50; 201 M, k = 8: 1289 us
// against 1307).  No builtin gives this pair of cache bits.  A store of more than 64 bits goes on reading its
// registers for up to two cycles, in which none may be written: hence the s_nop.
template <bool THROUGH, typename T>
__device__ __forceinline__ void st_once(T *p, T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "dword, dwordx2 or dwordx4");
    if constexpr (!THROUGH) st_stream(p, v);
    else if constexpr (sizeof(T) == 4) asm volatile("global_store_dword %0, %1, off sc1 nt" ::"v"(p), "v"(v) : "memory");
    else if constexpr (sizeof(T) == 8) asm volatile("global_store_dwordx2 %0, %1, off sc1 nt" ::"v"(p), "v"(v) : "memory");
    else asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

// body(true_type) in a workgroup whose elements are to be kept, else body(false_type): the choice is
// made once for the whole workgroup, around its loop.
template <typename F>
__device__ __forceinline__ void with_keep(bool keep, F body)
{
    if (keep) body(std::true_type{});
    else body(std::false_type{});
}

// s_waitcnt vmcnt(0) (expcnt and lgkmcnt left at their maxima), pinned in place
__device__ __forceinline__ void wait_vm_idle()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// fp32 -> bf16, round to nearest even; NaN stays NaN (quiet bit forced).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    uint32_t nan = (u >> 16) | 0x0040u;
    return ((u & 0x7fffffffu) > 0x7f800000u) ? nan : r;
}

// Clip coefficient from the total squared norm (Sec. 2.1: global L2 norm for clipping).
__device__ __forceinline__ float clip_from(double sqnorm, float max_norm)
{
    float norm = (float)sqrt(sqnorm);
    float c = max_norm / (norm + 1e-6f);
    return c < 1.0f ? c : 1.0f;
}
__device__ __forceinline__ bool clips(const double *d_sqnorm, float max_norm) { return d_sqnorm != nullptr && max_norm > 0.0f; }
__device__ __forceinline__ float clip_coefficient(const double *d_sqnorm, float max_norm)
{
    return clips(d_sqnorm, max_norm) ? clip_from(*d_sqnorm, max_norm) : 1.0f;
}

// *q by a vector load, which other loads overtake and are not held up by: the scalar load that a uniform address
// otherwise gets has to be back before any scalar load after it can be used.
__device__ __forceinline__ double ld_beside(const double *q)
{
    int zero = 0;
    asm volatile("" : "+v"(zero));
    return q[zero];
}

// The element update: clip, moments, master weight (Sec. 2.2: three fp32 states per weight,
// updated element-wise).  One rounding per operation, no fused multiply-add.
__device__ __forceinline__ void adamw_element(float a, float c, const StepConsts &s, float &p, float &m, float &v)
{
    float g = c * a;
    float t1 = s.beta1 * m;
    float t2 = s.omb1 * g;
    float mn = t1 + t2;
    float gg = g * g;
    float t3 = s.beta2 * v;
    float t4 = s.omb2 * gg;
    float vn = t3 + t4;
    float d = __builtin_sqrtf(vn) / s.rsbc2;
    d = d + s.eps;
    float u = mn / d;
    float t5 = p * s.decay;
    float t6 = s.step_size * u;
    p = t5 - t6;
    m = mn;
    v = vn;
}

// k-way accumulation of one group, j ascending from +0 (Sec. 2.1: micro-batch gradients are
// accumulated in full precision).  The loads go out in batches of DEPTH, each batch consumed before
// the next is issued; what is left of k after the whole batches is one batch too.
// APART (DEPTH 4): a batch of its own for each number of streams that can be left.  In the speculative
// kernel the compiler otherwise waits for each of these loads before it issues the next (its registers
// are defined on one side of a branch only), and the whole workgroup waits for them at its sum: k = 11, 201 M
// elements 1662 us against 1529; k = 15 1890 against 1759.  The step has no such wait and is faster
// without (12.6 M, k = 5: 74.7 us against 77.8).  The empty asm statements keep the three from being merged.
__device__ __forceinline__ void add_bf16(float (&a)[4], u32x2 g)
{
    a[0] += bf16_lo(g.x); a[1] += bf16_hi(g.x);
    a[2] += bf16_lo(g.y); a[3] += bf16_hi(g.y);
}
__device__ __forceinline__ void add_bf16(float (&a)[2], uint32_t g)
{
    a[0] += bf16_lo(g); a[1] += bf16_hi(g);
}

// TOGETHER: the addresses of a last, partial batch are read from the argument block together, and not one before
// each load: that is a scalar load and a wait for every stream, in a chain.
template <int N>
__device__ __forceinline__ void all_at_once(global_ptr<const uint16_t> (&p)[N + 1])
{
    if constexpr (N >= 15)
        asm volatile("" : "+s"(p[7]), "+s"(p[8]), "+s"(p[9]), "+s"(p[10]), "+s"(p[11]), "+s"(p[12]), "+s"(p[13]), "+s"(p[14]));
    asm volatile("" : "+s"(p[0]), "+s"(p[1]), "+s"(p[2]), "+s"(p[3]), "+s"(p[4]), "+s"(p[5]), "+s"(p[6]));
}

template <int EL, int DEPTH, bool KEEP = false, bool APART = false, bool TOGETHER = false, typename Table>
__device__ __forceinline__ void accumulate_batches(const Table &gt, int k, int64_t lo, float (&a)[EL])
{
    typedef typename Group<EL>::H H;
#pragma unroll
    for (int e = 0; e < EL; ++e) a[e] = 0.0f;
    int j = 0;
#pragma unroll 1
    for (; j + DEPTH <= k; j += DEPTH) {
        H g[DEPTH];
#pragma unroll
        for (int q = 0; q < DEPTH; ++q) g[q] = ld_stream<KEEP>(reinterpret_cast<const H *>(gt.g[j + q] + lo));
#pragma unroll
        for (int q = 0; q < DEPTH; ++q) add_bf16(a, g[q]);
    }
    const int rest = k - j;
    if constexpr (APART && DEPTH == 4) {
        auto take = [&](auto count) {
            constexpr int N = decltype(count)::value;
            H g[N];
#pragma unroll
            for (int q = 0; q < N; ++q) g[q] = ld_stream<KEEP>(reinterpret_cast<const H *>(gt.g[j + q] + lo));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < N; ++q) add_bf16(a, g[q]);
        };
        if (rest == 3) {
            asm volatile("; 3 streams left");
            take(std::integral_constant<int, 3>{});
        } else if (rest == 2) {
            asm volatile("; 2 streams left");
            take(std::integral_constant<int, 2>{});
        } else if (rest == 1) {
            asm volatile("; 1 stream left");
            take(std::integral_constant<int, 1>{});
        }
    } else if (DEPTH > 1 && rest > 0) {
        H g[DEPTH];
        if constexpr (TOGETHER && DEPTH >= 8) {
            // j is a multiple of DEPTH, so the batch's entries lie in the table; those from k on are not followed
            global_ptr<const uint16_t> from[DEPTH];
#pragma unroll
            for (int q = 0; q < DEPTH - 1; ++q) from[q] = in_global(gt.g[j + q]);
            all_at_once<DEPTH - 1>(from);
#pragma unroll
            for (int q = 0; q < DEPTH - 1; ++q)
                if (q < rest) g[q] = ld_stream<KEEP>(reinterpret_cast<const H *>((const uint16_t *)from[q] + lo));
        } else {
#pragma unroll
            for (int q = 0; q < DEPTH - 1; ++q)
                if (q < rest) g[q] = ld_stream<KEEP>(reinterpret_cast<const H *>(gt.g[j + q] + lo));
        }
#pragma unroll
        for (int q = 0; q < DEPTH - 1; ++q)
            if (q < rest) add_bf16(a, g[q]);
    }
}

// The same sum for the elements [i0,i1) of a group that a range end cuts (the others get 0).  One lane
// works alone here while the rest of the chip runs dry, so its loads go out several streams at a time: at
// 16 streams one load after another took longer than all the whole groups of a small range together.
template <int EL, typename Table>
__device__ __forceinline__ void accumulate_cut(const Table &gt, int k, int64_t lo, int64_t i0, int64_t i1, float (&a)[EL])
{
#pragma unroll
    for (int e = 0; e < EL; ++e) a[e] = 0.0f;
    constexpr int BATCH = 16 / EL;
#pragma unroll 1
    for (int j = 0; j < k; j += BATCH) {
        uint32_t g[BATCH][EL];
#pragma unroll
        for (int q = 0; q < BATCH; ++q)
            if (j + q < k)
#pragma unroll
                for (int e = 0; e < EL; ++e)
                    if (lo + e >= i0 && lo + e < i1) g[q][e] = gt.g[j + q][lo + e];
#pragma unroll
        for (int q = 0; q < BATCH; ++q)
            if (j + q < k)
#pragma unroll
                for (int e = 0; e < EL; ++e)
                    if (lo + e >= i0 && lo + e < i1) a[e] += __uint_as_float(g[q][e] << 16);
    }
}

// ---- block reduction used by the norm kernels ----------------------------------------------
// Per-lane fp64 partial (each square is exact in fp64) -> across the lanes of a wave -> LDS across the
// block's waves -> one partial per block; a second tiny kernel folds the block partials in a
// fixed order, so the result is deterministic.
// A small range waits for every step of this, so lanes are exchanged by DPP moves, a few cycles each, where
// shuffles go through the LDS hardware, and the waves' sums are added across lanes and not one after another
// (norm, 13 k / 200 k elements, k = 4 3.74/4.83 us against 3.99/5.14; fp32 norm, 13 k 2.32 against 2.66; staged norm, 520 k,
// k = 4 5.32 against 5.80).
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double add_dpp(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, false);
    return x + __hiloint2double(hi, lo);       // lanes outside ROWS add 0
}

// the sum of a row of 16 lanes, in all of them
__device__ __forceinline__ double row_sum(double x)
{
    x = add_dpp<0xb1>(x);                      // quad_perm [1,0,3,2]
    x = add_dpp<0x4e>(x);                      // quad_perm [2,3,0,1]
    x = add_dpp<0x141>(x);                     // row_half_mirror
    return add_dpp<0x140>(x);                  // row_mirror
}

// the sum of a wave, in its last lane
__device__ __forceinline__ double wave_sum(double x)
{
    x = row_sum(x);
    x = add_dpp<0x142, 0xa>(x);                // row_bcast:15 into rows 1 and 3
    return add_dpp<0x143, 0xc>(x);             // row_bcast:31 into rows 2 and 3
}

template <int BLOCK>
__device__ __forceinline__ double block_sum(double x, double *lds)
{
    constexpr int NW = BLOCK / 64;
    static_assert(NW >= 1 && NW <= 16, "the waves' sums lie in one row of lanes");
    x = wave_sum(x);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 63) lds[wave] = x;
    __syncthreads();
    double t = 0.0;
    if (wave == 0) t = row_sum(lane < NW ? lds[lane] : 0.0);
    return t;   // valid in thread 0
}

// ---- fused accumulate + clip + AdamW + bf16 emit -----------------------------------------
// A step's arguments in registers, read together as the kernel starts.  Left to themselves they are read where
// each is needed, five times over the life of a wave, and each time is a wait of 0.1-0.3 us in a chain that is
// all there is to a small range (13 k elements, k = 4 / 9 / 32 2.77/2.68/3.01 us against 3.00/3.26/3.52; 400 k, k = 9 / 32
// 4.30/7.78 against 4.74/8.20; 6.5 M, k = 2 / 8 32.8/45.1 against 33.7/46.2; level from 12 M on).
struct StepView {
    const float *p, *m, *v;
    float *po, *mo, *vo;
    uint16_t *w;
    const GradTable &gt;
    int k;
    int64_t begin, end;
    StepConsts c;
    float max_norm;
    const double *d_sqnorm;
    const float *acc;
};
// Where a wave waits between its stores, pinning them all and taking the norm early loses (2 M elements, k = 1 / 4
// 10.9/13.0 us against 10.1/11.9), and so it does in the staged step of a small range (13 k 2.07 against 1.99).  There the
// compiler is left to place the reads: through this view it puts all of them but the streams' addresses and the norm at
// the entry, behind one wait; from the argument block itself (LATE) each where its value is needed (late_arguments says when).
template <bool STAGED, bool LWAIT, bool SWAIT>
constexpr bool reads_early = !STAGED && !LWAIT && !SWAIT;

template <bool EARLY>
__device__ __forceinline__ StepView view_of(const StepArgs &A)
{
    StepView V{A.p, A.m, A.v, A.po, A.mo, A.vo, A.w, A.gt, A.k, A.begin, A.end, A.c, A.max_norm, A.d_sqnorm, A.acc};
    if constexpr (!EARLY) return V;
    // as global addresses, which they are known to be only while they come straight from the argument block
    global_ptr<const float> p = in_global(V.p), m = in_global(V.m), v = in_global(V.v), acc = in_global(V.acc);
    global_ptr<float> po = in_global(V.po), mo = in_global(V.mo), vo = in_global(V.vo);
    global_ptr<uint16_t> w = in_global(V.w);
    global_ptr<const double> sq = in_global(V.d_sqnorm);
    asm volatile("" : "+s"(po), "+s"(mo), "+s"(vo), "+s"(w), "+s"(V.k), "+s"(V.max_norm), "+s"(sq), "+s"(acc), "+s"(V.c.beta1),
                 "+s"(V.c.beta2), "+s"(V.c.omb1), "+s"(V.c.omb2), "+s"(V.c.eps));
    asm volatile("" : "+s"(p), "+s"(m), "+s"(v), "+s"(V.begin), "+s"(V.end), "+s"(V.c.step_size), "+s"(V.c.rsbc2), "+s"(V.c.decay));
    V.p = (const float *)p, V.m = (const float *)m, V.v = (const float *)v, V.acc = (const float *)acc;
    V.po = (float *)po, V.mo = (float *)mo, V.vo = (float *)vo, V.w = (uint16_t *)w, V.d_sqnorm = (const double *)sq;
    return V;
}

template <bool EARLY, bool LATE>
__device__ __forceinline__ decltype(auto) arguments(const StepArgs &A)
{
    static_assert(!(EARLY && LATE), "one of them");
    if constexpr (LATE) return static_cast<const StepArgs &>(A);
    else return view_of<EARLY>(A);
}

// The group of EL elements starting at `lo` (a multiple of EL): vector path when the group lies
// inside [begin,end), per-element path for ragged range ends -- same arithmetic.  States are read
// from A.p/m/v and written to A.po/mo/vo (the same arrays for the in-place entry points).
// STAGED: the gradient sum comes from A.acc instead of the k streams.  NORM: also add the squares
// of the accumulated gradients to acc0/acc1.  DEPTH: gradient loads in flight per batch.  LWAIT:
// the fp32 loads are waited for one by one.  SWAIT: each store waits for the previous one.  THROUGH: the
// stores are written through.
template <int EL, bool STAGED, bool NORM, int DEPTH, bool LWAIT, bool SWAIT, bool THROUGH = false, typename Args>
__device__ __forceinline__ void step_group(const Args &A, int64_t lo, const double *d_sqnorm, double &acc0, double &acc1)
{
    typedef typename Group<EL>::F F;
    typedef typename Group<EL>::H H;
    constexpr bool EARLY = reads_early<STAGED, LWAIT, SWAIT>;
    const StepConsts &s = A.c;
    if (lo >= A.begin && lo + EL <= A.end) {
        float c = 1.0f;
        if constexpr (LWAIT) c = clip_coefficient(d_sqnorm, A.max_norm);
        const F p = ld_stream(reinterpret_cast<const F *>(A.p + lo));
        if constexpr (LWAIT) wait_vm_idle();
        const F m = ld_stream(reinterpret_cast<const F *>(A.m + lo));
        if constexpr (LWAIT) wait_vm_idle();
        const F v = ld_stream(reinterpret_cast<const F *>(A.v + lo));
        if constexpr (LWAIT) wait_vm_idle();
        const bool clip = EARLY && clips(d_sqnorm, A.max_norm);
        double sqnorm = 0.0;
        if (clip) sqnorm = ld_beside(d_sqnorm);
        float a[EL];
        if constexpr (STAGED) {
            const F av = ld_stream(reinterpret_cast<const F *>(A.acc + lo));
#pragma unroll
            for (int e = 0; e < EL; ++e) a[e] = av[e];
        } else {
            accumulate_batches<EL, DEPTH, false, NORM, EARLY>(A.gt, A.k, lo, a);
        }
        if constexpr (!LWAIT && !EARLY) c = clip_coefficient(d_sqnorm, A.max_norm);     // under the loads in flight
        if (clip) {
            asm volatile("" : "+v"(sqnorm));       // here, under the loads in flight, and not where it is loaded
            c = clip_from(sqnorm, A.max_norm);
        }
        F P, M, V;
        uint32_t W[EL];
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            float pe = p[e], me = m[e], ve = v[e];
            if constexpr (NORM) {
                if (e & 1) acc1 = fma((double)a[e], (double)a[e], acc1);
                else acc0 = fma((double)a[e], (double)a[e], acc0);
            }
            adamw_element(a[e], c, s, pe, me, ve);
            P[e] = pe;
            M[e] = me;
            V[e] = ve;
            W[e] = f32_to_bf16_bits(pe);
        }
        H w;
        if constexpr (EL == 2) w = W[0] | (W[1] << 16);
        else w = H{W[0] | (W[1] << 16), W[2] | (W[3] << 16)};
        if constexpr (SWAIT) __builtin_amdgcn_sched_barrier(0);
        st_once<THROUGH>(reinterpret_cast<F *>(A.po + lo), P);
        if constexpr (SWAIT) wait_vm_idle();
        st_once<THROUGH>(reinterpret_cast<F *>(A.mo + lo), M);
        if constexpr (SWAIT) wait_vm_idle();
        st_once<THROUGH>(reinterpret_cast<F *>(A.vo + lo), V);
        if constexpr (SWAIT) wait_vm_idle();
        st_once<THROUGH>(reinterpret_cast<H *>(A.w + lo), w);
    } else {
        const int64_t i0 = lo > A.begin ? lo : A.begin;
        const int64_t i1 = lo + EL < A.end ? lo + EL : A.end;
        float a[EL], p[EL], m[EL], v[EL];
#pragma unroll
        for (int e = 0; e < EL; ++e)
            if (lo + e >= i0 && lo + e < i1) {
                p[e] = A.p[lo + e];
                m[e] = A.m[lo + e];
                v[e] = A.v[lo + e];
                if constexpr (STAGED) a[e] = A.acc[lo + e];
            }
        if constexpr (!STAGED) accumulate_cut<EL>(A.gt, A.k, lo, i0, i1, a);
        const float c = clip_coefficient(d_sqnorm, A.max_norm);
#pragma unroll
        for (int e = 0; e < EL; ++e)
            if (lo + e >= i0 && lo + e < i1) {
                if constexpr (NORM) acc0 = fma((double)a[e], (double)a[e], acc0);
                adamw_element(a[e], c, s, p[e], m[e], v[e]);
                A.po[lo + e] = p[e];
                A.mo[lo + e] = m[e];
                A.vo[lo + e] = v[e];
                A.w[lo + e] = (uint16_t)f32_to_bf16_bits(p[e]);
            }
    }
}

// One element on its own: the same update, all its loads in flight.  One or two streams are simply read:
// the tests for streams that are not there take longer than that (a step of 1 element, k = 1 / 2: 1.8/2.0 us
// against 2.1/2.2).
template <bool STAGED>
__device__ __forceinline__ void step_one(const StepArgs &A, int64_t i)
{
    float p = A.p[i], m = A.m[i], v = A.v[i];
    float a[1];
    if constexpr (STAGED) {
        a[0] = A.acc[i];
    } else if (A.k <= 2) {
        a[0] = 0.0f;
#pragma unroll 1
        for (int j = 0; j < A.k; ++j) a[0] += __uint_as_float((uint32_t)A.gt.g[j][i] << 16);
    } else {
        accumulate_cut<1>(A.gt, A.k, i, i, i + 1, a);
    }
    adamw_element(a[0], clip_coefficient(A.d_sqnorm, A.max_norm), A.c, p, m, v);
    A.po[i] = p;
    A.mo[i] = m;
    A.vo[i] = v;
    A.w[i] = (uint16_t)f32_to_bf16_bits(p);
}

// One workgroup = one tile of BLOCK*EL consecutive elements, one group per lane; which shape a range
// takes is step_shape's choice.  Tiles start at multiples of the tile size counted from element 0 of
// the arrays, not from `begin`: the grouping does not move with the range (partition independence),
// and a wave's accesses stay line-aligned for any `begin` (a split point in the middle of a layer
// would otherwise make every wave straddle two extra lines).
// The elements of groups that a range end cuts (at most EL-1 at each end) are workgroup 0's (`cuts` = 1),
// one lane each: in the wave of their neighbours they come after its whole groups, and the range
// ends one memory latency later (us, k = 1 / 8 / 32: 100 001 elements 2.9/3.0/4.2 against 3.5/4.0/7.2 there, 1 000 001
// elements 5.8/8.9/17.0 against 6.3/9.7/19.9; from 3 M on within 2 %).
template <int BLOCK, int EL, bool STAGED, int DEPTH, bool LWAIT, bool SWAIT, bool THROUGH, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_accum_adamw(StepArgs A, int cuts)
{
    constexpr int TILE = BLOCK * EL;
    decltype(auto) V = arguments<reads_early<STAGED, LWAIT, SWAIT>, LATE>(A);
    const int64_t b = (int64_t)blockIdx.x - cuts;
    if (b < 0) {
        const int64_t head = (A.begin + EL - 1) / EL * EL;         // where the first whole group starts
        const int64_t tail = A.end / EL * EL;                      // where the last one ends
        int64_t i = A.begin + threadIdx.x;
        if (i >= head) i += (tail > head ? tail : head) - head;    // past the first cut group: on to the last
        if (threadIdx.x < 2 * EL && i < A.end) step_one<STAGED>(A, i);
        return;
    }
    const int64_t lo = (V.begin / TILE + b) * TILE + (int64_t)threadIdx.x * EL;
    if (lo < V.begin || lo + EL > V.end) return;
    double unused0 = 0.0, unused1 = 0.0;
    step_group<EL, STAGED, false, DEPTH, LWAIT, SWAIT, THROUGH>(V, lo, V.d_sqnorm, unused0, unused1);
}

// The same for up to eight streams in place, with the arrays given by their distances from p (near_to).  A range of one generation of
// waves is bound by the chain launch, arguments, loads, update, stores: at four bytes an array all that the loads of up to four streams need
// is in registers as a wave starts, the others' distances and the constants arrive under the states' loads, and 112 bytes in all instead of 396
// shorten the host's launch as well (launch_norm_kernel).  us, against addresses in a block: 1 k / 13 k / 100 k, k = 4
// 2.39/2.48/2.67 against 2.55/2.64/2.91; 200 k, k = 1 / 4 / 7 3.10/2.96/3.06 against 3.34/3.25/3.35; 600 k, k = 1 / 5 4.31/5.04 against 4.67/5.81;
// 900 k, k = 2 / 6 / 8 5.4/7.2/7.9 against 5.6/7.6/8.3.  near_args says where not.
// With 4 elements per lane (SWAIT) the memory is busy: there the gradients' loads go first, and from seven streams on only when the states are
// back (states first / gradients first / waited for: 700 k, k = 4 / 6 / 8 5.44/6.18/6.89, 5.41/6.07/6.91, 5.74/5.99/6.58; 550 k, k = 6 / 8
// 4.98/5.47, 4.95/5.39, 5.41/5.67).
// the address `at` units of 2^unit bytes from `base`
template <typename T>
__device__ __forceinline__ T *near_to(float *base, int at, int unit)
{
    return reinterpret_cast<T *>(reinterpret_cast<char *>(base) + ((int64_t)at << unit));
}

template <int K, int BLOCK, int EL, int DEPTH, bool SWAIT, bool THROUGH>
__device__ __forceinline__ void step_near(int64_t begin, int cuts, uint32_t packed, float *p, const double *d_sqnorm, int m_at, int v_at, int g0, int g1,
                                          int g2, int g3, NearRest<K> R)
{
    typedef typename Group<EL>::F F;
    typedef typename Group<EL>::H H;
    constexpr int TILE = BLOCK * EL;
    const int64_t end = begin + (packed % GS_NEAR_CLIP_BIT);
    const bool clip = packed & GS_NEAR_CLIP_BIT;
    const int unit = packed & GS_NEAR_UNIT_BIT ? 8 : 4;
    float *const m = near_to<float>(p, m_at, unit), *const v = near_to<float>(p, v_at, unit);
    const int64_t b = (int64_t)blockIdx.x - cuts;
    if (b < 0) {
        const int64_t head = (begin + EL - 1) / EL * EL;         // where the first whole group starts
        const int64_t tail = end / EL * EL;                      // where the last one ends
        int64_t i = begin + threadIdx.x;
        if (i >= head) i += (tail > head ? tail : head) - head;    // past the first cut group: on to the last
        if (threadIdx.x >= 2 * EL || i >= end) return;
        const int at[8] = {g0, g1, g2, g3, R.g[0], R.g[1], R.g[2], R.g[3]};
        float pe = p[i], me = m[i], ve = v[i], a = 0.0f;
        uint32_t g[K];
#pragma unroll
        for (int q = 0; q < K; ++q) g[q] = near_to<const uint16_t>(p, at[q], unit)[i];
#pragma unroll
        for (int q = 0; q < K; ++q) a += __uint_as_float(g[q] << 16);
        adamw_element(a, clip ? clip_from(*d_sqnorm, R.max_norm) : 1.0f, R.c, pe, me, ve);
        p[i] = pe;
        m[i] = me;
        v[i] = ve;
        near_to<uint16_t>(p, R.w, unit)[i] = (uint16_t)f32_to_bf16_bits(pe);
        return;
    }
    const int64_t lo = ((int64_t)((uint64_t)begin / TILE) + b) * TILE + (int64_t)threadIdx.x * EL;
    if (lo < begin || lo + EL > end) return;
    const int at[8] = {g0, g1, g2, g3, R.g[0], R.g[1], R.g[2], R.g[3]};
    F pv, mv, vv;
    H g[DEPTH];
    double sqnorm = 0.0;
    auto load_states = [&] {
        pv = ld_stream(reinterpret_cast<const F *>(p + lo));
        mv = ld_stream(reinterpret_cast<const F *>(m + lo));
        vv = ld_stream(reinterpret_cast<const F *>(v + lo));
    };
    auto load_batch = [&](int j) {
#pragma unroll
        for (int q = 0; q < DEPTH; ++q)
            if (j + q < K) g[q] = ld_stream(reinterpret_cast<const H *>(near_to<const uint16_t>(p, at[j + q], unit) + lo));
    };
    if constexpr (SWAIT && K < 7) {
        load_batch(0);
        __builtin_amdgcn_sched_barrier(0);
        load_states();
        __builtin_amdgcn_sched_barrier(0);
    } else {
        load_states();
        if (!SWAIT && clip) sqnorm = ld_beside(d_sqnorm);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SWAIT) {
            wait_vm_idle();
        } else {
            // the states' loads are on their way: now the arguments that came through memory, together
            asm volatile("" : "+s"(R.g[0]), "+s"(R.g[1]), "+s"(R.g[2]), "+s"(R.g[3]), "+s"(R.w), "+s"(R.max_norm), "+s"(R.c.beta1), "+s"(R.c.beta2),
                         "+s"(R.c.omb1), "+s"(R.c.omb2), "+s"(R.c.eps), "+s"(R.c.step_size), "+s"(R.c.rsbc2), "+s"(R.c.decay));
            __builtin_amdgcn_sched_barrier(0);
        }
        load_batch(0);
    }
    float a[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) a[e] = 0.0f;
#pragma unroll
    for (int j = 0; j < K; j += DEPTH) {
        if (j > 0) load_batch(j);
#pragma unroll
        for (int q = 0; q < DEPTH; ++q)
            if (j + q < K) add_bf16(a, g[q]);
        if (j + DEPTH < K) __builtin_amdgcn_sched_barrier(0);
    }
    float c = 1.0f;
    if (SWAIT) {
        if (clip) c = clip_from(*d_sqnorm, R.max_norm);
    } else if (clip) {
        asm volatile("" : "+v"(sqnorm));       // here, under the loads in flight, and not where it is loaded
        c = clip_from(sqnorm, R.max_norm);
    }
    F P, M, V;
    uint32_t W[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) {
        float pe = pv[e], me = mv[e], ve = vv[e];
        adamw_element(a[e], c, R.c, pe, me, ve);
        P[e] = pe;
        M[e] = me;
        V[e] = ve;
        W[e] = f32_to_bf16_bits(pe);
    }
    H w;
    if constexpr (EL == 2) w = W[0] | (W[1] << 16);
    else w = H{W[0] | (W[1] << 16), W[2] | (W[3] << 16)};
    if constexpr (SWAIT) __builtin_amdgcn_sched_barrier(0);
    st_once<THROUGH>(reinterpret_cast<F *>(p + lo), P);
    if constexpr (SWAIT) wait_vm_idle();
    st_once<THROUGH>(reinterpret_cast<F *>(m + lo), M);
    if constexpr (SWAIT) wait_vm_idle();
    st_once<THROUGH>(reinterpret_cast<F *>(v + lo), V);
    if constexpr (SWAIT) wait_vm_idle();
    st_once<THROUGH>(reinterpret_cast<H *>(near_to<uint16_t>(p, R.w, unit) + lo), w);
}

// a kernel for each number of streams: told at run time, the compiler waits for each of two or three loads before the next
#define GS_NEAR_STEP(K)                                                                                                                        \
    template <int BLOCK, int EL, bool STAGED, int DEPTH, bool LWAIT, bool SWAIT, bool THROUGH, bool LATE>                                      \
    __global__ __launch_bounds__(BLOCK) void k_accum_adamw(int64_t begin, int cuts, uint32_t packed, float *p, const double *d_sqnorm, int m_at, \
                                                           int v_at, int g0, int g1, int g2, int g3, NearRest<K> R)                            \
    {                                                                                                                                          \
        static_assert(!STAGED && !LWAIT, "waves that do not wait between their loads");                                                        \
        step_near<K, BLOCK, EL, DEPTH, SWAIT, THROUGH>(begin, cuts, packed, p, d_sqnorm, m_at, v_at, g0, g1, g2, g3, R);                       \
    }
GS_NEAR_STEP(1)
GS_NEAR_STEP(2)
GS_NEAR_STEP(3)
GS_NEAR_STEP(4)
GS_NEAR_STEP(5)
GS_NEAR_STEP(6)
GS_NEAR_STEP(7)
GS_NEAR_STEP(8)
#undef GS_NEAR_STEP

// Speculative single pass (Sec. 2.1 of the paper: prior work steps before the global norm is
// known because clipping rarely changes the gradients): the step is applied with c = 1 and the
// squared norm of the same accumulated gradients is reduced on the way, so the gradients are
// read once.  Every workgroup leaves a partial for its `span` consecutive tiles.
template <int BLOCK, int EL, int DEPTH, bool SWAIT, bool THROUGH>
__global__ __launch_bounds__(BLOCK) void k_accum_adamw_spec(StepArgs A, double *partials, int span)
{
    constexpr int TILE = BLOCK * EL;
    __shared__ double lds[BLOCK / 64];
    const int64_t first = (A.begin / TILE + (int64_t)blockIdx.x * span) * TILE + (int64_t)threadIdx.x * EL;
    double acc0 = 0.0, acc1 = 0.0;
    const StepView V = view_of<reads_early<false, false, SWAIT>>(A);
    for (int it = 0; it < span; ++it) {
        const int64_t lo = first + (int64_t)it * TILE;
        if (lo >= V.end) break;
        if (lo + EL <= V.begin) continue;
        step_group<EL, false, true, DEPTH, false, SWAIT, THROUGH>(V, lo, nullptr, acc0, acc1);
    }
    double t = block_sum<BLOCK>(acc0 + acc1, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// ---- squared norm of the accumulated gradient --------------------------------------------
template <int EL>
__device__ __forceinline__ void add_squares(const float (&a)[EL], double &acc0, double &acc1)
{
#pragma unroll
    for (int e = 0; e < EL; e += 2) {
        acc0 = fma((double)a[e], (double)a[e], acc0);
        acc1 = fma((double)a[e + 1], (double)a[e + 1], acc1);
    }
}

// Read-only, 2k bytes per element.  Workgroup b reads `span` consecutive tiles starting at tile
// b*span: a short contiguous run per workgroup is what the read path likes best.  What else bounds
// it is how much a wave has in flight: with up to four streams the same groups of U tiles are loaded together, with more
// of them up to DEPTH streams are.  K: the number of streams, or 0 where it is told at run time (the long runs on some of the CUs).  Told
// at run time, each stream of a partial batch is a test, a scalar load and a wait before its load: with the fold, us, a kernel for each
// number against that, 4 k elements, k = 5 / 17 2.37/3.76 against 2.65/4.33; 13 k, k = 9 / 24 3.91/5.00 against 4.35/5.70; 100 k, k = 12 / 29
// 4.51/5.54 against 4.93/6.23; 1 M, k = 13 / 17 7.75/8.97 against 8.26/9.66; 12 M, k = 11 / 17 46.6/67.2 against 47.6/69.2, 50 M 162.3/244.6
// against 163.7/247.0; level from 200 M on, and everywhere with 8, 16, 24 and 32, whose batches are whole.
// ONE: a single workgroup reads the whole range and leaves the norm itself in `out`.  Workgroups from keep_block on
// leave what they read in the memory-side cache.
template <int K, int U, int BLOCK, bool ONE, int DEPTH, typename Table>
__device__ __forceinline__ void grad_sqnorm(int64_t begin, int span, int keep_block, int64_t end, const Table &gt, int k, double *partials,
                                            double *out, int accumulate)
{
    constexpr int TILE = BLOCK * 4;
    // from five streams on 256 lanes read ranges below GS_KEEP_MANY_MIN, or on some of the CUs
    constexpr bool KEEPS = !ONE && (BLOCK > 256 || (K > 0 && K <= 4));
    static_assert(GS_NORM_256_MAX <= GS_KEEP_MANY_MIN, "else 256 lanes would have to leave lines in the cache");
    // Of several tiles one after the other, each by itself: the sums are then those of workgroups of 256 lanes and their fold, in that order, so
    // that a range has the same norm to the bit whichever of the two it is given to.  That takes 0.05-0.1 us a tile (captured, 7.2 k / 9.6 k, k = 5
    // 3.0/3.8 us against 2.9/3.6; kept in registers and summed beside each other at the end, 10 % in all against 5).
    constexpr bool FOLDS = ONE && K > 4;
    constexpr int TILES = FOLDS ? GS_ONE_MAX_LOADS / K / TILE + 2 : 1, WAVES = BLOCK / 64;
    __shared__ double lds[TILES * WAVES];
    const bool folds = FOLDS && span > 1;
    const int64_t first = (begin / TILE + (int64_t)blockIdx.x * span) * TILE + (int64_t)threadIdx.x * 4;
    double acc0 = 0.0, acc1 = 0.0;
    with_keep(KEEPS && (int)blockIdx.x >= keep_block, [&](auto keep) {
    constexpr bool KEEP = decltype(keep)::value;
    for (int it = 0; it < span; it += U) {
        const int64_t lo = first + (int64_t)it * TILE;
        if (!FOLDS && lo >= end) break;
        if (FOLDS && lo >= end) {
            // all lanes go on to the tile's sum
        } else if (lo >= begin && lo + (int64_t)(U - 1) * TILE + 4 <= end) {
            if constexpr (K > 0) {
                static_assert(K <= DEPTH || U == 1, "tiles are grouped for one batch of streams");
                constexpr int BATCH = K < DEPTH ? K : DEPTH;
                u32x2 g[U][BATCH];
                float a[U][4] = {};
#pragma unroll
                for (int from = 0; from < K; from += BATCH) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int j = 0; j < BATCH; ++j)
                            if (from + j < K) g[u][j] = ld_stream<KEEP>(reinterpret_cast<const u32x2 *>(gt.g[from + j] + lo + (int64_t)u * TILE));
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int j = 0; j < BATCH; ++j)
                            if (from + j < K) add_bf16(a[u], g[u][j]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) add_squares(a[u], acc0, acc1);
            } else {
                static_assert(K > 0 || U == 1, "tiles are grouped for a compile-time K only");
                float a[4];
                accumulate_batches<4, DEPTH, KEEP>(gt, k, lo, a);
                add_squares(a, acc0, acc1);
            }
        } else {
            // a range end lies among these tiles: group by group, and by element in the group it cuts
            for (int u = 0; u < U; ++u) {
                const int64_t l = lo + (int64_t)u * TILE;
                if (l >= begin && l + 4 <= end) {
                    float a[4];
                    accumulate_batches<4, (K == 0 || K > DEPTH ? DEPTH : K), KEEP>(gt, k, l, a);
                    add_squares(a, acc0, acc1);
                    continue;
                }
                const int64_t i0 = l > begin ? l : begin;
                const int64_t i1 = l + 4 < end ? l + 4 : end;
                if (i0 >= i1) continue;
                float a[4];
                accumulate_cut<4>(gt, k, l, i0, i1, a);
                add_squares(a, acc0, acc1);
            }
        }
        if constexpr (FOLDS) {
            if (folds) {
                const double wave = wave_sum(acc0 + acc1);
                if (threadIdx.x % 64 == 63) lds[it * WAVES + threadIdx.x / 64] = wave;
                acc0 = acc1 = 0.0;
            }
        }
    }
    });
    if constexpr (FOLDS) {
        static_assert(BLOCK == 1024 && U == 1 && TILES <= 16, "four workgroups of 256 lanes a tile, in one wave's lanes");
        if (folds) {
            __syncthreads();
            if (threadIdx.x >= 64) return;
            const int part = (int)threadIdx.x + (int)(begin % TILE / 1024);        // the first such workgroup's is lane 0's
            const double *w = lds + 4 * part;
            const double t = wave_sum(part < 4 * span ? (w[0] + w[1]) + (w[2] + w[3]) : 0.0);
            if (threadIdx.x == 63) *out = accumulate ? *out + t : t;
            return;
        }
    }
    double t = block_sum<BLOCK>(acc0 + acc1, lds);
    if (threadIdx.x == 0) {
        if constexpr (ONE) *out = accumulate ? *out + t : t;
        else partials[blockIdx.x] = t;
    }
}

#define GS_NORM_KERNEL(STREAMS)                                                                                                                \
    template <int K, int U, int BLOCK, bool ONE, int DEPTH = 16>                                                                               \
    __global__ __launch_bounds__(BLOCK) void k_grad_sqnorm(int64_t begin, int span, int keep_block, int64_t end, GradTableOf<STREAMS> gt, int k, \
                                                           int accumulate, double *partials, double *out)                                      \
    {                                                                                                                                          \
        grad_sqnorm<K, U, BLOCK, ONE, DEPTH>(begin, span, keep_block, end, gt, K > 0 ? K : k, partials, out, accumulate);                      \
    }
GS_NORM_KERNEL(8)
GS_NORM_KERNEL(16)
GS_NORM_KERNEL(32)
#undef GS_NORM_KERNEL

// up to four (entries of the table beyond K are not read)
template <int K, int U, int BLOCK, bool ONE, int DEPTH = 16>
__global__ __launch_bounds__(BLOCK) void k_grad_sqnorm(int64_t begin, int span, int keep_block, int64_t end, const uint16_t *g0, const uint16_t *g1,
                                                       const uint16_t *g2, const uint16_t *g3, double *partials, double *out, int accumulate)
{
    static_assert(K >= 1 && K <= 4, "streams by compile-time number");
    const GradTableOf<4> gt{{g0, g1, g2, g3}};
    grad_sqnorm<K, U, BLOCK, ONE, DEPTH>(begin, span, keep_block, end, gt, K, partials, out, accumulate);
}

// The same norm that also writes the fp32 sum a_i to A.acc (the staged two-pass variant: the step
// then reads one fp32 stream instead of re-reading k bf16 streams).  Once a store stream is
// involved, runs of tiles per workgroup cost bandwidth (stores want in-order, one-tile workgroups),
// so it uses a span of 1 wherever the partials still fit the workspace.  KEEPS: some of the sum is left
// in the memory-side cache; where none is, the choice alone would cost the one tile of a wave 1-2 %
// (50 M, k = 2, 16 CUs: 741 us against 752).
template <int BLOCK, int EL, int DEPTH, bool KEEPS, typename Table>
__device__ __forceinline__ void grad_accum_sqnorm(int64_t begin, int span, int keep_block, int64_t end, float *acc, const Table &gt, int k, double *partials)
{
    typedef typename Group<EL>::F F;
    constexpr int TILE = BLOCK * EL;
    __shared__ double lds[BLOCK / 64];
    const int64_t first = (begin / TILE + (int64_t)blockIdx.x * span) * TILE + (int64_t)threadIdx.x * EL;
    double acc0 = 0.0, acc1 = 0.0;
    with_keep(KEEPS && (int)blockIdx.x >= keep_block, [&](auto keep) {
    constexpr bool KEEP = decltype(keep)::value;
    for (int it = 0; it < span; ++it) {
        const int64_t lo = first + (int64_t)it * TILE;
        if (lo >= end) break;
        if (lo + EL <= begin) continue;
        float a[EL];
        if (lo >= begin && lo + EL <= end) {
            accumulate_batches<EL, DEPTH>(gt, k, lo, a);
            F sum;
#pragma unroll
            for (int e = 0; e < EL; ++e) sum[e] = a[e];
            st_stream<KEEP>(reinterpret_cast<F *>(acc + lo), sum);
        } else {
            const int64_t i0 = lo > begin ? lo : begin;
            const int64_t i1 = lo + EL < end ? lo + EL : end;
            accumulate_cut<EL>(gt, k, lo, i0, i1, a);
#pragma unroll
            for (int e = 0; e < EL; ++e)
                if (lo + e >= i0 && lo + e < i1) acc[lo + e] = a[e];
        }
        add_squares(a, acc0, acc1);
    }
    });
    double t = block_sum<BLOCK>(acc0 + acc1, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// up to eight streams, and any number
template <int BLOCK, int EL, int DEPTH, bool KEEPS>
__global__ __launch_bounds__(BLOCK) void k_grad_accum_sqnorm(int64_t begin, int span, int keep_block, int64_t end, float *acc, GradTableOf<8> gt, int k,
                                                             double *partials)
{
    grad_accum_sqnorm<BLOCK, EL, DEPTH, KEEPS>(begin, span, keep_block, end, acc, gt, k, partials);
}
template <int BLOCK, int EL, int DEPTH, bool KEEPS>
__global__ __launch_bounds__(BLOCK) void k_grad_accum_sqnorm(int64_t begin, int span, int keep_block, int64_t end, float *acc, GradTable gt, int k,
                                                             double *partials)
{
    grad_accum_sqnorm<BLOCK, EL, DEPTH, KEEPS>(begin, span, keep_block, end, acc, gt, k, partials);
}

// ---- accumulate as you go ------------------------------------------------------------------
// The paper's GPU keeps one full-precision accumulation buffer per layer and each micro-batch's
// backward adds its gradient into it (Sec. 3.4, Sec. 4.3).  acc = (FIRST ? +0 : acc) + widen(g):
// 2 + 4 bytes read and 4 written per element (2 + 4 for the first micro-batch).  NORM: the call
// that adds the last micro-batch also reduces the squared norm of the finished sum.
template <bool FIRST, bool NORM, int BLOCK, int EL, bool LWAIT, bool THROUGH>
__global__ __launch_bounds__(BLOCK) void k_accum_add(AccumAddArgs A, int span)
{
    typedef typename Group<EL>::F F;
    typedef typename Group<EL>::H H;
    constexpr int TILE = BLOCK * EL;
    __shared__ double lds[BLOCK / 64];
    const int64_t first = (A.begin / TILE + (int64_t)blockIdx.x * span) * TILE + (int64_t)threadIdx.x * EL;
    double acc0 = 0.0, acc1 = 0.0;
    with_keep(first - (int64_t)threadIdx.x * EL >= A.keep_from, [&](auto keep) {
    constexpr bool KEEP = decltype(keep)::value;
    for (int it = 0; it < span; ++it) {
        const int64_t lo = first + (int64_t)it * TILE;
        if (lo >= A.end) break;
        if (lo + EL <= A.begin) continue;
        float a[EL];
        if (lo >= A.begin && lo + EL <= A.end) {
            const H g = ld_stream(reinterpret_cast<const H *>(A.g + lo));
            if constexpr (LWAIT && !FIRST) wait_vm_idle();
            F old, sum;
            if constexpr (!FIRST) old = ld_stream<KEEP>(reinterpret_cast<const F *>(A.acc + lo));
#pragma unroll
            for (int e = 0; e < EL; ++e) a[e] = FIRST ? 0.0f : old[e];
            add_bf16(a, g);
#pragma unroll
            for (int e = 0; e < EL; ++e) sum[e] = a[e];
            if constexpr (KEEP) st_stream<true>(reinterpret_cast<F *>(A.acc + lo), sum);
            else st_once<THROUGH>(reinterpret_cast<F *>(A.acc + lo), sum);
        } else {
#pragma unroll
            for (int e = 0; e < EL; ++e) {
                a[e] = 0.0f;
                if (lo + e >= A.begin && lo + e < A.end) {
                    if constexpr (!FIRST) a[e] = A.acc[lo + e];
                    a[e] += __uint_as_float((uint32_t)A.g[lo + e] << 16);
                    A.acc[lo + e] = a[e];
                }
            }
        }
        if constexpr (NORM) add_squares(a, acc0, acc1);
    }
    });
    if constexpr (NORM) {
        double t = block_sum<BLOCK>(acc0 + acc1, lds);
        if (threadIdx.x == 0) A.partials[blockIdx.x] = t;
    }
}

// Norm of a finished fp32 accumulation buffer (the buffer gs_accum_add builds, or one that came
// back from a reduction across devices): 4 bytes read per element, the read-only shape of the
// gradient norm -- U tiles of a short contiguous run in flight together.
template <int U, int BLOCK, bool ONE>
__global__ __launch_bounds__(BLOCK) void k_acc_sqnorm(const float *acc, int64_t begin, int64_t end, int64_t keep_from, double *out, int accumulate, int span)
{
    constexpr int TILE = BLOCK * 4;
    __shared__ double lds[BLOCK / 64];
    const int64_t first = (begin / TILE + (int64_t)blockIdx.x * span) * TILE + (int64_t)threadIdx.x * 4;
    double acc0 = 0.0, acc1 = 0.0;
    with_keep(first - (int64_t)threadIdx.x * 4 >= keep_from, [&](auto keep) {
    constexpr bool KEEP = decltype(keep)::value;
    for (int it = 0; it < span; it += U) {
        const int64_t lo = first + (int64_t)it * TILE;
        if (lo >= end) break;
        if (lo >= begin && lo + (int64_t)(U - 1) * TILE + 4 <= end) {
            f32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = ld_stream<KEEP>(reinterpret_cast<const f32x4 *>(acc + lo + (int64_t)u * TILE));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float a[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                add_squares(a, acc0, acc1);
            }
        } else {
            for (int u = 0; u < U; ++u) {
                const int64_t l = lo + (int64_t)u * TILE;
                if (l >= begin && l + 4 <= end) {
                    const f32x4 v = ld_stream<KEEP>(reinterpret_cast<const f32x4 *>(acc + l));
                    const float a[4] = {v.x, v.y, v.z, v.w};
                    add_squares(a, acc0, acc1);
                    continue;
                }
                const int64_t i0 = l > begin ? l : begin;
                const int64_t i1 = l + 4 < end ? l + 4 : end;
                for (int64_t i = i0; i < i1; ++i) acc0 = fma((double)acc[i], (double)acc[i], acc0);
            }
        }
    }
    });
    double t = block_sum<BLOCK>(acc0 + acc1, lds);
    if (threadIdx.x == 0) {
        if constexpr (ONE) *out = accumulate ? *out + t : t;
        else out[blockIdx.x] = t;        // the workgroup partials
    }
}

// Folding the workgroup partials, in a fixed order (deterministic).  Up to 262144 partials are too
// many for one workgroup to read quickly, so large counts go through GS_FINAL_SLICES workgroups
// that each fold a contiguous slice into the tail of the workspace, then one workgroup folds those.
__global__ __launch_bounds__(GS_FINAL_BLOCK) void k_sqnorm_fold_slices(const double *partials, int nparts, double *slices)
{
    __shared__ double lds[GS_FINAL_BLOCK / 64];
    const int per = (nparts + GS_FINAL_SLICES - 1) / GS_FINAL_SLICES;
    const int lo = blockIdx.x * per;
    const int hi = lo + per < nparts ? lo + per : nparts;
    double x = 0.0;
    for (int i = lo + threadIdx.x; i < hi; i += GS_FINAL_BLOCK) x += partials[i];
    double t = block_sum<GS_FINAL_BLOCK>(x, lds);
    if (threadIdx.x == 0) slices[blockIdx.x] = t;
}

__global__ __launch_bounds__(GS_FINAL_BLOCK) void k_sqnorm_finalize(const double *partials, int nparts, double *out, int accumulate)
{
    __shared__ double lds[GS_FINAL_BLOCK / 64];
    double x = 0.0;
    for (int i = threadIdx.x; i < nparts; i += GS_FINAL_BLOCK) x += partials[i];
    double t = block_sum<GS_FINAL_BLOCK>(x, lds);
    if (threadIdx.x == 0) *out = accumulate ? (*out + t) : t;
}

static hipError_t launch_fold(double *partials, int64_t cap, int nparts, double *d_out, int accumulate, hipStream_t stream)
{
    if (nparts > GS_FINAL_DIRECT_MAX) {
        double *slices = partials + cap;          // the last GS_FINAL_SLICES doubles of the workspace
        k_sqnorm_fold_slices<<<GS_FINAL_SLICES, GS_FINAL_BLOCK, 0, stream>>>(partials, nparts, slices);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_sqnorm_finalize<<<1, GS_FINAL_BLOCK, 0, stream>>>(slices, GS_FINAL_SLICES, d_out, accumulate);
    } else {
        k_sqnorm_finalize<<<1, GS_FINAL_BLOCK, 0, stream>>>(partials, nparts, d_out, accumulate);
    }
    return hipGetLastError();
}

// ---- launchers -----------------------------------------------------------------------------
static int64_t tiles_of(int64_t begin, int64_t end, int64_t tile)
{
    if (end <= begin) return 0;
    return (end - 1) / tile - begin / tile + 1;
}

// HIP launches fewer than 2^32 work items at a time: the workgroups of `block` lanes that is.
static constexpr int64_t max_grid(int block) { return 0xffffffffLL / block; }

// A launch whose arguments are given by reference, each of exactly the kernel's own type.
template <typename... P, typename... V>
static hipError_t launch(void (*kernel)(P...), int grid, int block, uint32_t lds, hipStream_t stream, V &...v)
{
    static_assert((std::is_same_v<P, std::remove_const_t<V>> && ...), "the runtime copies as many bytes as the kernel's arguments have");
    void *args[] = {const_cast<void *>(static_cast<const void *>(&v))...};
    (void)hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block), args, lds, stream);
    return hipGetLastError();
}

// LDS that a launch asks for and does not use, so that a CU holds `workgroups` of them (of the sizes used here
// it would otherwise hold 8 to 32): the fewest pieces of which one workgroup more would not get its share, 55 KB for
// two.  The 512 bytes less leave room for what the kernels do use.
static constexpr uint32_t room_for(int workgroups)
{
    return (uint32_t)((GS_LDS_GRANULES / (workgroups + 1) + 1) * GS_LDS_GRANULE_BYTES - 512);
}

// How a step over `elems` elements is laid out; every line below is where the two sides met when both
// were timed with cold caches (us per launch, k = 1 / 4 / 8 / 16 / 32).  The chip holds 8192 waves
// (256 CUs x 32): up to 2^20 elements the waves of a 2-element shape, and up to 2^21 those of a
// 4-element shape, are resident together.
//   <= 2^19   LATENCY: a wave's chain of dependent loads is the time, so all of them go out at once.
//             100 k elements: 2.9/3.1/3.0/3.2/4.1 against 4.4/5.9/6.6/10.1/17.2 for loads one at a
//             time, and with 2 to 15 streams written through while all loads are back before the stores take the
//             memory (latency_through); at 800 k RESIDENT is level or ahead (5.1/6.1/7.7/9.6/13.2 against 5.6/6.5/7.7/9.6/13.6).
//   <= 2^21   RESIDENT: no second, nearly empty generation of waves: 1.3 M elements 6.7/8.5/10.3/14.7/20.7
//             against 8.8/10.0/12.3/16.0/23.1 with 2 elements per lane and 7.4/9.4/11.8/17.4/27.1 one at a
//             time.  Over the last quarter with few streams the memory is busy enough that SERIAL
//             wins (2.0 M: 10.3/12.8 against 10.3/13.4 for k = 1 / 4).
//   above     2 elements per lane, all stores back to back and written through.
//   <= 7 M    FULL: as many workgroups as a CU holds, four gradient loads in flight, with 5 to 19 streams (FULL_DEEP) eight
//             (with 20 to 24 those are level with the norm and 1-3 % behind without it: 4 M / 5 M, k = 24 2.0/2.1 % slower).
//             norm + step on three sets of tensors in turn, k = 1 / 4 / 8 / 16: 2.3 M 19.1/23.0/29.5/42.8 us against
//             19.4/23.4/30.8/43.7 with the hint alone and four loads, 4.7 M 30.1/36.6/49.9/78.9 against 30.5/37.5/50.6/80.1.
//   above     HBM serves this mix of reads and writes best when a fixed amount of it is asked for: more
//             in flight and it turns between them more often, less and it idles.  A full CU of 32 waves
//             overshoots by a half; waves that wait between their own accesses lower the number too, but leave
//             gaps.  So the waves wait for nothing, and a CU holds as many as make up 50-60 KB of loads:
//   STREAM    four gradient loads in flight, 11 workgroups of two waves (10 where k is a multiple of four).  Against a
//             full CU with its stores one at a time (up to 7 streams, from 2^27 on, each load too), ms: 201 M, k = 1 / 2 /
//             3 / 4 / 8 / 11 / 16 / 24  0.85/0.91/0.97/1.04/1.28/1.47/1.80/2.34 against 0.89/0.94/1.01/1.11/1.31/1.51/1.86/2.44;
//             805 M, k = 16  7.10-7.35 against 7.46-7.56; 402 M, k = 32  5.83-6.00 against 6.11-6.21; norm + step, 12.6 M,
//             k = 1 / 4  64.0/83.8 us against 67.4/85.5.  One workgroup more or less is within 1 %, two cost 2-4 %.
//   DEEP      eight in flight and 9 workgroups, for 5 to 7 streams, which are then one batch (201 M, k = 5 / 6 / 7
//             1.10/1.15/1.22 ms against 1.13/1.16/1.22 in STREAM and 1.16/1.24/1.29 before), and for 8, 16 and 24 up to 2^25
//             elements (norm + step, 12.6 M, k = 8 / 16 113.4/174.0 us against 114.0/174.8 in STREAM and 115.3/175.3 before).
//   9 to 23 streams that are no multiple of 8 leave some over after any batches: FULL up to 2^24 elements (9.4 M,
//             k = 9 / 13 / 17 93.3/116.8/139.6 us against 96.5/118.9/147 in STREAM and 94.2/117.4/141.4 before); then, below
//             20 of them, DEEP up to 2^26 (36 M, k = 11 / 14 382/445 against 383/449 and 387/453; level for k = 9, 10, 12).
//   The staged step reads four fp32 streams: FULL up to 7 M elements (with its norm, 2.5 M / 5 M 19.3/30.9 us against 19.6/31.3
//             with the hint alone), then 4 elements per lane, 10 workgroups of one wave: with its norm, 12.6 M / 36 M 67.2/178
//             us against 69.5/184, alone 617 M 2.72 ms against 2.82, with 2 elements per lane, a full CU and stores one at a
//             time (up to 7 M those are 1 % behind FULL where a range starts in the middle of a line).
enum Shape {
    SHAPE_LATENCY,    // 2 elements per lane, everything in flight at once
    SHAPE_RESIDENT,   // 4 elements per lane, stores one at a time
    SHAPE_SERIAL,     // 4 elements per lane, every load and store of a wave waited for
    SHAPE_FULL,       // 2 elements per lane, four loads in flight, stores written through
    SHAPE_FULL_DEEP,  // the same with eight
    SHAPE_STREAM,     // FULL with fewer workgroups per CU (staged: 4 elements per lane)
    SHAPE_DEEP,       // FULL_DEEP with fewer
    SHAPE_BUDGET      // 4 elements per lane, two gradient loads in flight, stores one at a time
};

// The CUs that `stream` is confined to, or 0 if it may use all of them.  The runtime looks the mask up in the stream's own
// host-side record; a stream it cannot tell about counts as unconfined (only the shape depends on this), and so
// do the null stream and the handles that only name a default stream, which have no record to look up.
static int budget_cus(hipStream_t stream)
{
    if (!stream || stream == hipStreamLegacy || stream == hipStreamPerThread) return 0;
    uint32_t mask[64] = {0};
    int dev = 0, cus = 0, in_mask = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipExtStreamGetCUMask(stream, 64, mask) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    for (uint32_t word : mask) in_mask += __builtin_popcount(word);
    return in_mask < cus ? in_mask : 0;
}

static bool on_cu_budget(hipStream_t stream) { return budget_cus(stream) > 0; }

// Whether launches on `stream` go into a graph (the null stream's cannot, and it is not asked about: beside another
// thread's capture that is an error).
static bool is_captured(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (!stream || stream == hipStreamLegacy) return false;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) (void)hipGetLastError();
    return status != hipStreamCaptureStatusNone;
}

//   A stream confined to some of the CUs (any size over 2^21) takes BUDGET: there the bytes each CU keeps in
//             flight are the bound, and 4 elements per lane hold twice as many (k = 2 / 8, 100 M elements:
//             16 CUs 3.39/4.97 ms against 4.71/5.95 with 2 elements per lane and 4.11/5.83 one load at a time,
//             128 CUs 0.60/0.84 against 0.74/0.95 and 0.67/0.91).
//   States in host memory take LATENCY at every size: the link is the bound, and a wave that waits between
//             its accesses leaves it idle (16 CUs, 12.6 M elements, k = 2 / 8 / 16: 3.23/3.19/3.23 ms against
//             3.26/3.37/3.35 with stores one at a time and 3.35/3.46/3.60 one load at a time; 100 M, k = 8:
//             25.5 ms against 26.4 and 27.3).
// With all of those waves in flight the first generation reads and then writes together, and the link carries one direction at
// a time; with as many as the link needs to be busy both ways, and their stores written through, it does not.  16 CUs, k = 1 / 8 /
// 16: 300 k elements 114/115/121 us against 159/153/156 with the hint and full CUs, 1 M 286/286/291 against 402/324/302, 12.6 M
// 3.12/3.09/3.24 ms against 3.22/3.22/3.23.  Over long ranges full CUs come to be busy both ways by themselves, and alone they are up to 5 % ahead
// where a die has 4 to 15 CUs (50 M, k = 2, 32 / 64 / 112 CUs 12.1/12.1/12.1 ms against 12.3/12.15/12.6; on 16, 24 and all CUs the bound is 0-4 %
// ahead).  But they hold up other work far more: with eight 1 ms GEMMs beside it, a step of 30 M elements on 32 / 64 / 96 / all CUs and they
// take 12.7/15.7/15.7/15.9 ms together unbounded, 11.3/11.1/11.5/11.5 bounded (one after the other 15.5), so the bound holds at every length.
// Work is dealt to the eight dies in turn, and on a die to its four shader engines in turn; so are the CUs of a stream, and the
// engine that got the fewest (once every engine has one) decides what the die takes: that many CUs count (48: 4 a die, not 6).  22
// single-wave workgroups a die are in flight up to 8 such CUs, 64 on more (about half and one and a half times that: 8-15 % slower over
// 12.6 M elements): 1.5 M, 48 / 72 / 136 / 256 CUs 417/407/417/388 us against 510/504/528/529.  Where the dies' shares differ, the smaller
// ones would hold the others back (50 M, 22 / 60 / 92 CUs 6/8/10 % slower alone) and no workgroup is kept off a CU.
static uint32_t link_room(hipStream_t stream)
{
    const auto counting = [](int cus_of_a_die) { return cus_of_a_die < 4 ? cus_of_a_die : cus_of_a_die / 4 * 4; };
    const int budget = budget_cus(stream), cus = budget > 0 ? budget : 256;
    const int share = counting(cus / 8);
    if (share != counting((cus + 7) / 8)) return 0;
    return room_for(share <= 8 ? GS_LINK_WAVES / share : (GS_LINK_WAVES_WIDE + share / 2) / share);
}

// k == 0: the staged step (one fp32 sum instead of gradient streams)
static Shape step_shape(int64_t elems, int k, bool over_link, hipStream_t stream)
{
    if (over_link) return SHAPE_LATENCY;
    if (elems <= GS_LATENCY_MAX) return SHAPE_LATENCY;
    if (elems <= GS_RESIDENT_MAX)
        return k <= GS_SERIAL_MAX_K && elems > GS_RESIDENT_MAX / 4 * 3 ? SHAPE_SERIAL : SHAPE_RESIDENT;
    if (on_cu_budget(stream)) return SHAPE_BUDGET;
    if (k == 0) return elems <= GS_FULL_MAX ? SHAPE_FULL : SHAPE_STREAM;
    if (elems <= GS_FULL_MAX) return k >= 5 && k < 20 ? SHAPE_FULL_DEEP : SHAPE_FULL;
    if (k < 5) return SHAPE_STREAM;
    if (k < 8) return SHAPE_DEEP;
    if (k % 8 == 0) return k <= 24 && elems <= GS_DEEP_MAX ? SHAPE_DEEP : SHAPE_STREAM;
    if (k < 24 && elems <= GS_FULL_ODD_MAX) return SHAPE_FULL;
    return k < 20 && elems <= GS_DEEP_ODD_MAX ? SHAPE_DEEP : SHAPE_STREAM;
}

// Whether a LATENCY step is written through.  Stores that wait in the L2 go out when the kernel ends, others at once, which
// is a gain as long as no wave's loads are held up by them (without the norm, 300 k elements, k = 4 / 6 / 10 / 15 4-5 % faster);
// the more streams, the longer the loads last (500 k, k = 6 / 9 and 450 k, k = 12 9-10 % slower): level at 484/455/435/405/378/357 k
// elements for k = 5/6/7/10/12/15, and ahead over the whole range for 2 to 4 (500 k, k = 3 4 % faster).  8 streams are one whole batch, loaded without the tests of a
// partial one, and meet the line sooner (330 k 2 % faster, 400 k 13 % slower), 16 before 400 k (10 % slower there).  One stream and the
// staged step lose by it from 100 k on (4 %, 5-9 %).
static bool latency_through(int64_t elems, int k)
{
    if (k < 2 || k >= 16) return false;
    if (k < 5) return true;
    return elems <= (k == 8 ? GS_LATENCY_MAX / 2 : GS_LATENCY_MAX - k * GS_LATENCY_THROUGH_STEP);
}

// Whether a step in one generation of waves (RESIDENT, SERIAL) reads its arguments late.  While the range is bound by the
// latency of a wave's chain, each wait more is time (us, view / late, k = 4 / 8 / 16: 700 k 5.9/6.9/8.7 against 6.2/7.2/9.2); once
// the memory is busy, a gap between a wave's state loads and its gradient loads spreads what the waves, which all start
// together, ask for at a time (1 M, k = 7 / 16 8.4/11.3 against 8.2/11.0; 1.3 M, k = 9 / 11 12.3/13.0 against 11.1/11.9).  The memory is busy
// later with few streams (k = 4 1.15 M 7.7 against 7.9, 1.5 M 9.8 against 9.1, and in SERIAL the view is 1 % ahead again; up to three
// streams it wins throughout, 1 M, k = 1 5.8 against 6.5); with many the gain ends where the chip is half full (1.5 M, k = 9 / 16
// 13.4/16.6 against 13.9/16.9).  On some of the CUs the view wins throughout (128 CUs, 1.3 M, k = 9 / 12 15.7/16.4 against 16.0/16.9).
static bool late_arguments(int64_t elems, int k, hipStream_t stream)
{
    if (k < 4 || elems <= GS_LATE_MIN + (k < 7 ? 7 - k : 0) * GS_LATE_MIN_STEP) return false;
    if (elems > (k == 4 ? GS_RESIDENT_MAX / 4 * 3 : k < 8 ? GS_RESIDENT_MAX : GS_LATE_MAX_MANY)) return false;
    return !on_cu_budget(stream);
}

struct NearArgs {
    uint32_t packed;     // elements, whether the norm clips, and the distances' unit
    float *p;
    int m, v, g[8], w;
};

// The arguments of a step in place with up to eight streams as distances from p, if all of its arrays lie within 32 GB of
// it, or within 512 GB and as many bytes beyond multiples of 256 as it does (an allocator deals out such addresses; even in a small process some are
// 32 GB apart).  In LATENCY loads that go out sooner run into the stores of the waves before, where those are written through: level at
// 325/300/310/295/285/270 k elements for 2 to 7 streams (350 k, k = 4 / 7 3.9/4.5 us against 3.8/4.3), at 450 k for one and eight.  In RESIDENT they
// come all at once as the memory gets busy: 2-7 % behind from 1.3 M on for 6 to 8 streams (up to five 1 % ahead there, and level above).
// In full CUs above 2^21 they are ahead again, by less and less (with the norm, k = 2 / 5 / 8: 2.2 M 17.4/20.7/24.6 us against 17.7/21.1/24.9, 3.3 M
// 22.6/27.8/33.9 against 22.9/28.3/34.3, 5 M within 1 %; alone four streams are 0.8 % behind from 6 M on).
// On some of the CUs they are ahead as well (16 / 64 / 128 CUs, 100 k, k = 4 5.9/3.6/2.7 us against 6.8/4.4/3.3, 900 k, k = 2 32.0/10.5/6.8 against
// 32.9/11.8/7.3), but with seven and eight streams in RESIDENT level only: 0.5-1.5 % behind on 16 and 32 CUs (600 k, k = 8 31.3/17.9 against
// 31.0/17.7), from 8 % ahead to 4 % behind on more of them, as the last waves of a range happen to fall (600 k / 1.19 M, k = 8, 64 CUs 11.1/19.9
// against 11.7/19.7, 128 CUs 7.7/13.1 against 8.0/14.3, 192 CUs 7.3/10.9 against 7.6/10.5).  To ask for the stream's CUs takes the host 0.5 us,
// which every call with so many streams would pay.
static bool near_args(const StepArgs &A, NearArgs &N)
{
    const int64_t n = A.end - A.begin;
    if (A.over_link || A.k > 8 || A.po != A.p || A.mo != A.m || A.vo != A.v) return false;
    if (n > GS_NEAR_MAX && !(n > GS_RESIDENT_MAX && n <= GS_NEAR_FULL_MAX)) return false;
    if (n <= GS_LATENCY_MAX && n > (A.k == 1 || A.k == 8 ? GS_NEAR_LATENCY_MAX : GS_NEAR_THROUGH_MAX - A.k * GS_NEAR_THROUGH_STEP)) return false;
    static_assert(GS_NEAR_THROUGH_MAX <= GS_LATENCY_MAX - 7 * GS_LATENCY_THROUGH_STEP, "two to seven streams are written through as long as they are near");
    static_assert(GS_NEAR_MAX < GS_NEAR_FULL_MAX && GS_NEAR_FULL_MAX < GS_NEAR_CLIP_BIT && GS_NEAR_FULL_MAX <= GS_FULL_MAX, "the parts of `packed`");
    const auto bytes_from_p = [&](const void *q) { return (int64_t)(reinterpret_cast<uintptr_t>(q) - reinterpret_cast<uintptr_t>(A.p)); };
    int64_t any = bytes_from_p(A.m) | bytes_from_p(A.v) | bytes_from_p(A.w);
    for (int j = 0; j < A.k; ++j) any |= bytes_from_p(A.gt.g[j]);
    const int unit = any % 256 == 0 ? 8 : 4;
    bool fits = true;
    const auto from_p = [&](const void *q) {
        const int64_t d = bytes_from_p(q) >> unit;
        if (d != (int)d) fits = false;
        return (int)d;
    };
    const bool clip = A.d_sqnorm && A.max_norm > 0.0f;
    N.packed = (uint32_t)n + (clip ? GS_NEAR_CLIP_BIT : 0) + (unit == 8 ? GS_NEAR_UNIT_BIT : 0);
    N.p = A.po;
    N.m = from_p(A.m);
    N.v = from_p(A.v);
    for (int j = 0; j < 8; ++j) N.g[j] = j < A.k ? from_p(A.gt.g[j]) : 0;
    N.w = from_p(A.w);
    return fits;
}

template <int BLOCK, int EL, bool STAGED, int DEPTH, bool LWAIT, bool SWAIT, bool THROUGH = false, bool LATE = false>
static hipError_t launch_step(const StepArgs &A, hipStream_t stream, uint32_t room = 0)
{
    constexpr int64_t TILE = (int64_t)BLOCK * EL;
    int64_t tiles = tiles_of(A.begin, A.end, TILE);
    if (tiles < 1) return hipErrorInvalidValue;
    const int cuts = A.begin % EL != 0 || A.end % EL != 0;
    if (tiles + cuts > max_grid(BLOCK)) {                           // too long for one launch: two, cut where a tile starts
        StepArgs half = A;
        half.end = (A.begin / TILE + tiles / 2) * TILE;
        const hipError_t e = launch_step<BLOCK, EL, STAGED, DEPTH, LWAIT, SWAIT, THROUGH, LATE>(half, stream, room);
        if (e != hipSuccess) return e;
        half.begin = half.end;
        half.end = A.end;
        return launch_step<BLOCK, EL, STAGED, DEPTH, LWAIT, SWAIT, THROUGH, LATE>(half, stream, room);
    }
    if ((A.begin + EL - 1) / EL >= A.end / EL) tiles = 0;           // no whole group
    const int grid = (int)(tiles + cuts);
    if constexpr (!STAGED && !LWAIT && !LATE && (DEPTH == 4 || DEPTH == 8)) {
        NearArgs N;
        if (near_args(A, N)) {
            hipError_t e = hipSuccess;
            const auto go = [&](auto streams) {
                constexpr int K = decltype(streams)::value;
                // the numbers of streams that this shape is taken with; any other is given addresses
                constexpr bool taken = BLOCK == 128 ? (DEPTH == 8) == (K >= 5) : EL == 4 || K == 8 || THROUGH == (K > 1);
                if constexpr (taken) {
                    NearRest<K> R{{N.g[4], N.g[5], N.g[6], N.g[7]}, N.w, A.max_norm, A.c};
                    void (*const kernel)(int64_t, int, uint32_t, float *, const double *, int, int, int, int, int, int, NearRest<K>) =
                        k_accum_adamw<BLOCK, EL, STAGED, DEPTH, LWAIT, SWAIT, THROUGH, LATE>;
                    e = launch(kernel, grid, BLOCK, room, stream, A.begin, cuts, N.packed, N.p, A.d_sqnorm, N.m, N.v, N.g[0], N.g[1], N.g[2], N.g[3], R);
                }
                return taken;
            };
            bool gone = false;
            switch (A.k) {
            case 1: gone = go(std::integral_constant<int, 1>{}); break;
            case 2: gone = go(std::integral_constant<int, 2>{}); break;
            case 3: gone = go(std::integral_constant<int, 3>{}); break;
            case 4: gone = go(std::integral_constant<int, 4>{}); break;
            case 5: gone = go(std::integral_constant<int, 5>{}); break;
            case 6: gone = go(std::integral_constant<int, 6>{}); break;
            case 7: gone = go(std::integral_constant<int, 7>{}); break;
            case 8: gone = go(std::integral_constant<int, 8>{}); break;
            }
            if (gone) return e;
        }
    }
    void (*const kernel)(StepArgs, int) = k_accum_adamw<BLOCK, EL, STAGED, DEPTH, LWAIT, SWAIT, THROUGH, LATE>;
    return launch(kernel, grid, BLOCK, room, stream, A, cuts);
}

template <bool STAGED>
static hipError_t launch_step_shape(const StepArgs &A, hipStream_t stream)
{
    const Shape shape = step_shape(A.end - A.begin, STAGED ? 0 : A.k, A.over_link, stream);
    switch (shape) {
    case SHAPE_LATENCY: {
        if constexpr (!STAGED) {
            const uint32_t room = A.over_link ? link_room(stream) : 0;
            if (A.over_link || latency_through(A.end - A.begin, A.k)) {
                if (A.k > 8) return launch_step<64, 2, false, 16, false, false, true>(A, stream, room);
                return launch_step<64, 2, false, 8, false, false, true>(A, stream, room);
            }
            if (A.k > 8) return launch_step<64, 2, false, 16, false, false>(A, stream);
        }
        return launch_step<64, 2, STAGED, 8, false, false>(A, stream);
    }
    case SHAPE_RESIDENT:
        if constexpr (!STAGED)
            if (late_arguments(A.end - A.begin, A.k, stream)) return launch_step<64, 4, false, 4, false, true, false, true>(A, stream);
        return launch_step<64, 4, STAGED, 4, false, true>(A, stream);
    case SHAPE_SERIAL:
        if constexpr (!STAGED)
            if (late_arguments(A.end - A.begin, A.k, stream)) return launch_step<64, 4, false, 1, true, true, false, true>(A, stream);
        return launch_step<64, 4, STAGED, 1, true, true>(A, stream);
    case SHAPE_BUDGET: return launch_step<64, 4, STAGED, 2, false, true>(A, stream);
    default: break;
    }
    const bool full = shape == SHAPE_FULL || shape == SHAPE_FULL_DEEP;
    if constexpr (STAGED) {
        if (full) return launch_step<128, 2, true, 4, false, false, true>(A, stream);
        return launch_step<64, 4, true, 4, false, false, true>(A, stream, room_for(10));
    } else {
        const bool deep = shape == SHAPE_DEEP || shape == SHAPE_FULL_DEEP;
        if (deep) return launch_step<128, 2, false, 8, false, false, true>(A, stream, full ? 0 : room_for(9));
        return launch_step<128, 2, false, 4, false, false, true>(A, stream, full ? 0 : room_for(A.k % 4 == 0 ? 10 : 11));
    }
}

hipError_t launch_accum_adamw(const StepArgs &A, hipStream_t stream)
{
    return A.acc ? launch_step_shape<true>(A, stream) : launch_step_shape<false>(A, stream);
}

// Partials the workspace can hold (its last GS_FINAL_SLICES doubles serve the folding stage).
static int64_t partial_capacity(size_t workspace_bytes)
{
    return (int64_t)(workspace_bytes / sizeof(double)) - GS_FINAL_SLICES;
}

// The span (tiles per workgroup) that keeps the partials within `cap` and the workgroups of `block` lanes
// within one launch: `span` itself, or the next multiple of U that does.  0: not possible.
static int64_t fit_span(int64_t tiles, int64_t span, int64_t U, int64_t cap, int block)
{
    if (cap > max_grid(block)) cap = max_grid(block);
    if ((tiles + span - 1) / span > cap) span = ((tiles + cap - 1) / cap + U - 1) / U * U;
    return span > 0x7fffffff ? 0 : span;
}

template <int BLOCK, int EL, int DEPTH, bool SWAIT, bool THROUGH>
static hipError_t launch_spec(const StepArgs &A, double *partials, int64_t cap, double *d_out, int accumulate, hipStream_t stream,
                              uint32_t room = 0)
{
    int64_t tiles = tiles_of(A.begin, A.end, (int64_t)BLOCK * EL);
    if (tiles < 1) tiles = 1;
    const int64_t span = fit_span(tiles, 1, 1, cap, BLOCK);
    if (span == 0) return hipErrorInvalidValue;
    const int grid = (int)((tiles + span - 1) / span);
    k_accum_adamw_spec<BLOCK, EL, DEPTH, SWAIT, THROUGH><<<grid, BLOCK, room, stream>>>(A, partials, (int)span);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_fold(partials, cap, grid, d_out, accumulate, stream);
}

// The step with a partial per workgroup.  A wave also reduces its squares, so its chain is longer and a CU holds a few
// workgroups more than in the step.  us or ms per launch and fold, against four loads in flight, a full CU and
// stores one at a time (few streams: one load at a time), k as given:
//   * up to 7 M elements everything in flight, 256 lanes (600 k, k = 3 / 8 / 16: 7.7/8.9/11.0 against 9.7/11.9/16.3);
//     up to 2 streams written through, so that no lines are left for the fold to wait for (k = 1 / 2: 600 k 6.9/7.3
//     against 8.2/8.5, 3 M 18.1/18.7 against 20.6/22.2), and up to 7 streams below 2^21 elements (1.5 M, k = 4 / 6 10.8/12.4
//     against 11.7/13.2; 6.5 M 43.1/47.7 against 41.4/45.3; from 8 streams on level at every size);
//   * then, a partial per 256 elements: single waves of 4 elements per lane, 16 workgroups per CU (14 from 9 streams
//     on): 12.6 M, k = 3 / 8 / 16 69.2/90.4/123.9 against 72.3/91.8/127.6; 50 M, k = 1 / 8 217/335 against 224/342; 201 M,
//     k = 1 / 4 / 8 / 11  867/1051/1289/1469 against 910/1091/1349/1525;
//   * a workspace too small for that: a partial per 512, two waves, 7 workgroups per CU (8 up to 4 streams): 100 M,
//     k = 1 / 4 / 8 / 11 448/553/656/756 against 459/566/698/805;
//   * or runs of 512-element tiles, four waves of 2 elements per lane, 6 workgroups per CU, 5 from 2^28 elements on: 201 M,
//     k = 2 / 8 / 11 0.96/1.33/1.51 against 1.03/1.36/1.56; 402 M, k = 4 / 8 2.30/2.85 against 2.43/2.92; 530 M, k = 16 5.20
//     against 5.53;
//   * from 2^29 elements on (2^28 up to 2 streams, where the two are within 1 %) runs of 4096-element tiles: 700 M,
//     k = 2 / 6 3.59/4.62 against 3.70/4.75, 805 M, k = 8 5.71 against 6.18.
// On a stream confined to some of the CUs it is the bytes that each of them has in flight that bound (step_shape), so
// no workgroup is kept off it (ms on 16 / 64 / 128 CUs, with the small workspace):
//   * a partial per 512, or runs of those with up to 7 streams below 2^28 elements: stores one at a time; 70 M, k = 1
//     2.42/0.73/0.41 against 2.93/0.86/0.47 bounded, k = 8 3.53/1.03/0.61 against 4.31/1.23/0.67; 200 M, k = 2 7.18/2.18/1.25 against
//     9.11/2.65/1.44 in runs of 512-element tiles with bounded CUs;
//   * else runs of those tiles, two elements per lane: 200 M, k = 8 10.67/3.12/1.75 against 11.72/3.40/1.86 bounded; 300 M, k = 2 / 16
//     11.65/3.53/1.95 and 21.92/6.17/3.62 against 14.86/4.01/2.17 in 4096-element tiles and 26.93/7.38/4.11 bounded.
hipError_t launch_accum_adamw_spec(const StepArgs &A, double *partials, size_t workspace_bytes, double *d_out,
                                   int accumulate, hipStream_t stream)
{
    const int64_t cap = partial_capacity(workspace_bytes);
    const int64_t n = A.end - A.begin;
    const bool fits256 = tiles_of(A.begin, A.end, 256) <= cap;
    if (n > GS_RESIDENT_MAX && on_cu_budget(stream)) {
        if (fits256) return launch_spec<64, 4, 2, true, false>(A, partials, cap, d_out, accumulate, stream);
        if (tiles_of(A.begin, A.end, 512) <= cap || (A.k <= GS_SERIAL_MAX_K && n < GS_SPEC_RUN_LONG))
            return launch_spec<128, 4, 4, true, false>(A, partials, cap, d_out, accumulate, stream);
        return launch_spec<256, 2, 4, false, true>(A, partials, cap, d_out, accumulate, stream);
    }
    if (n <= GS_SPEC_FEW_MAX) {
        if (A.k <= 2 || (A.k <= GS_SERIAL_MAX_K && n <= GS_RESIDENT_MAX))
            return launch_spec<256, 4, 16, false, true>(A, partials, cap, d_out, accumulate, stream);
        return launch_spec<256, 4, 16, false, false>(A, partials, cap, d_out, accumulate, stream);
    }
    if (fits256) return launch_spec<64, 4, 4, false, true>(A, partials, cap, d_out, accumulate, stream, room_for(A.k <= 8 ? 16 : 14));
    if (tiles_of(A.begin, A.end, 512) <= cap)
        return launch_spec<128, 4, 4, false, true>(A, partials, cap, d_out, accumulate, stream, room_for(A.k <= 4 ? 8 : 7));
    if (n < (A.k <= 2 ? GS_SPEC_RUN_LONG : GS_SPEC_RUN_MAX))
        return launch_spec<256, 2, 4, false, true>(A, partials, cap, d_out, accumulate, stream, room_for(n < GS_SPEC_RUN_LONG ? 6 : 5));
    return launch_spec<1024, 4, 8, false, true>(A, partials, cap, d_out, accumulate, stream);
}

// Where a pass leaves its lines in the 256 MB memory-side cache.  A step reads again what the norm has
// just read (the gradients, or their fp32 sum), and the adding kernel what it wrote a micro-batch ago.
// Accesses with the non-temporal hint hit lines that are in that cache but put none there, so if only the
// last 256 MB of the re-read stream are accessed without it, they stay until the next pass.  The two passes
// together gain (us, plain against with the hint everywhere):
//   norm + step, k = 1 / 3 / 8 / 16 / 32   6 M 36/42/59/87/143 against 37/45/62/92/155, 50 M 242/290/440/679/1203 against
//                                        250/305/448/692/1221, 805 M k = 16 11.13 ms against 11.23
//   fp32 norm + step                     50 M 255 against 268, 201 M 1031 against 1057
//   8 micro-batches added, then the step   12.6 M 216 against 229, 50 M 766 against 832
// and the first of them pays, which a caller feels who takes only that one or goes on elsewhere:
//   norm alone, k = 8 / 16 / 32            6 M 20.7/36.8/66.4 against 18.9/32.2/61.3, 50 M 127/237/471 against 122/231/466
//   fp32 norm alone                      50 M 37.5 against 34.4;  first micro-batch alone 5 M 8.7 against 7.3, 50 M 51 against 49
// 192 and 320 MB gain less than 256 (norm + step, 201 M: 1749 and 1747 us against 1745).  Not done:
//   * Up to 2^21 elements (the last of several micro-batches: 2^22, launch_accum_add), but for the gradient norm of four streams and more only
//     up to 3 * 2^18, of two and three up to 1.3 M.  The
//     two passes, plain from there on against the hint up to 2^21, k = 4 / 8 / 12 / 32: 800 k 11.0/12.8/14.8/24.3 against 11.1/13.5/15.7/25.6, 1.3 M
//     13.8/16.3/19.3/35.5 against 14.3/17.5/21.9/38.0, 2 M 17.6/23.5/28.4/52.2 against 18.9/25.5/30.2/54.8; k = 2, 1 M / 2 M 10.7/15.6 against
//     10.6/16.3.  Several norms into scalars of their own before their steps gain while their lines fit the cache together, and a little beyond (12 of
//     each, against the tree in which this began at 2^21, 800 k / 1.3 M, k = 16 216/294 against 232/311), and lose where they are several times
//     as long (2 M, k = 16 / 32 433/704 against 433/680).  The norm alone: k = 4 / 8 / 16 / 32 800 k 5.0/5.7/8.2/12.9 against 5.1/5.8/7.8/12.0,
//     2 M 6.2/9.1/14.4/25.4 against 6.5/8.7/13.4/23.2.  Below, the gain goes up and down with the range (600 k, k = 4 / 32 +4/-6 %); the fp32 norm gains from about 2 M on and
//     loses at 800 k (6 %), the staged norm likewise.
//   * accumulate: the norm goes on over other ranges before the step comes, and the next range's lines
//     would push these out again.
//   * On some of the CUs the memory is not the bound, and plain accesses cost 3-7 %.
//   * The staged norm of more than 16 streams: the reads push the sum out again, and its plain stores cost the
//     pass 4-9 % (norm + step, us, with the hint against without, k = 14 / 16 / 20 / 32: 3.3 M 41.9/43.5/47.8/59.1
//     against 41.2/42.4/47.2/62.3; 12.6 M 132/139/155/202 against 133/141/159/209; 50 M 492/523/583/781 against
//     486/520/586/794; 201 M 1940/2070/2328/3115 against 1932/2060/2330/3120).
static int64_t keep_from(int64_t begin, int64_t end, int bytes_per_elem, int accumulate, hipStream_t stream, int64_t upto = GS_RESIDENT_MAX)
{
    if (accumulate || end - begin <= upto || on_cu_budget(stream)) return end;
    return end - GS_KEEP_BYTES / bytes_per_elem;
}

// The first of `grid` workgroups, of `run` elements each from the tile on that `begin` lies in, that starts at keep_from or beyond.
static int first_kept(int64_t begin, int64_t keep_from, int64_t run, int64_t tile, int grid)
{
    const int64_t past = keep_from - begin / tile * tile;
    const int64_t first = past > 0 ? (past + run - 1) / run : 0;
    return first < grid ? (int)first : grid;
}

// A norm's launch.  Its kernels take their arguments one by one and not as a block: leading arguments that fit 14 registers are
// in them as a wave starts (the build asks for that), where a block is fetched from memory by every workgroup before its first load,
// and by all CUs at once as the kernel starts.  Up to four streams everything a load needs is there, from five on all but the streams'
// addresses, in a table no longer than it has to be up to eight.  With the fold, us, against a block of 300 bytes: 13 k, k = 4 3.47 against
// 3.73; 4 k, k = 8 2.88 against 3.15; 3.3 M, k = 3 7.2 against 7.7; 5 M, k = 4 9.9 against 11.1; 7 M, k = 5 16.2 against 17.3; 12.6 M,
// k = 1 / 4 / 8 7.85/19.8/38.0 against 8.04/20.9/38.8; fp32 norm, 5 M / 10 M 6.35/9.1 against 6.8/9.5; within 1 % from 200 M on.  On the
// host a launch with up to 112 bytes of arguments takes 2.28 us, one with more 2.33, and on a core that another program shares 2.7 against 3.3
// (a step, and no slope: 416 bytes 3.35).
template <int K, int U, int BLOCK, bool ONE, int DEPTH = 16>
static hipError_t launch_norm_kernel(SqnormArgs &A, int grid, int span, hipStream_t stream)
{
    const int keep_block = first_kept(A.begin, A.keep_from, (int64_t)span * BLOCK * 4, BLOCK * 4, grid);
    typedef const uint16_t *G;
    G *const g = A.gt.g;
    if constexpr (K >= 1 && K <= 4) {
        void (*const kernel)(int64_t, int, int, int64_t, G, G, G, G, double *, double *, int) = k_grad_sqnorm<K, U, BLOCK, ONE, DEPTH>;
        return launch(kernel, grid, BLOCK, 0, stream, A.begin, span, keep_block, A.end, g[0], g[1], g[2], g[3], A.partials, A.out, A.accumulate);
    } else {
        constexpr int STREAMS = K > 16 ? 32 : K > 8 ? 16 : 8;                 // K == 0: the long runs on some of the CUs, up to seven streams
        GradTableOf<STREAMS> gt;
        for (int j = 0; j < STREAMS; ++j) gt.g[j] = g[j];
        void (*const kernel)(int64_t, int, int, int64_t, GradTableOf<STREAMS>, int, int, double *, double *) = k_grad_sqnorm<K, U, BLOCK, ONE, DEPTH>;
        return launch(kernel, grid, BLOCK, 0, stream, A.begin, span, keep_block, A.end, gt, A.k, A.accumulate, A.partials, A.out);
    }
}

template <int K, int U, int BLOCK, int DEPTH = 16>
static hipError_t launch_norm(SqnormArgs A, int64_t span, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    int64_t tiles = tiles_of(A.begin, A.end, (int64_t)BLOCK * 4);
    if (tiles < 1) tiles = 1;
    span = fit_span(tiles, span, U, cap, BLOCK);
    if (span == 0) return hipErrorInvalidValue;
    const int grid = (int)((tiles + span - 1) / span);
    hipError_t e = launch_norm_kernel<K, U, BLOCK, false, DEPTH>(A, grid, (int)span, stream);
    if (e != hipSuccess) return e;
    return launch_fold(A.partials, cap, grid, d_out, accumulate, stream);
}

// the whole range in one workgroup and one launch
template <int K, int U>
static hipError_t launch_norm_one(SqnormArgs A, double *d_out, int accumulate, hipStream_t stream, int span = U)
{
    A.out = d_out;
    A.accumulate = accumulate;
    return launch_norm_kernel<K, U, GS_ONE_BLOCK, true>(A, 1, span, stream);
}

// From 5 streams on, whether one workgroup reads a range of more than one tile.  Called one after the other, the second launch's host
// time counts (launch_grad_norm).  A captured norm has none, and there it is the GPU's time alone: us in a graph, one workgroup against
// norm and fold, k = 5 / 6 / 7 / 8, 6 k elements 2.7/3.2/3.4/3.8 against 3.7/3.9/3.9/4.0, 8 k, k = 6 3.65 against 3.85, 60 k and 2^16 values, k = 5 / 8
// 4.1/4.55 and 5.3/4.7 against 3.85/4.0 and 4.5/4.0.  The mean over ranges of any begin is 12, 7, 3.5 and 1 % ahead from 24, 32, 36 and 40 k values on and
// 2 % behind from 44 k on.  Each tile is a latency of its own there, so not where the begin lies so late in its tile that the range
// takes one tile more (begin 4093, 4.9 k, k = 10 5.9 against 4.9), and so is a group that a range end cuts, so not where one wave would have both
// (4.2 k, k = 13 8.6 against 6.4).  Both shapes leave the same bits.
static bool one_workgroup(const SqnormArgs &A, int64_t tiles, hipStream_t stream)
{
    constexpr int64_t TILE = GS_ONE_BLOCK * 4, WAVE = 64 * 4;
    const int64_t n = A.end - A.begin;
    if (tiles <= 1) return true;
    if (n * A.k > GS_ONE_MAX_LOADS) return false;
    const bool cuts_meet = A.begin % 4 != 0 && A.end % 4 != 0 && A.begin % TILE / WAVE == A.end % TILE / WAVE;
    const bool one_latency_each = tiles == (n + TILE - 1) / TILE && !cuts_meet;
    return (n * A.k <= GS_ONE_MAX_LOADS_CAPTURED && one_latency_each) || !is_captured(stream);
}

// from 5 streams on
template <int K>
static hipError_t launch_norm_many(const SqnormArgs &A, int64_t run, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    const int64_t n = A.end - A.begin;
    const int64_t tiles = tiles_of(A.begin, A.end, GS_ONE_BLOCK * 4);
    if (one_workgroup(A, tiles, stream)) return launch_norm_one<K, 1>(A, d_out, accumulate, stream, tiles > 1 ? (int)tiles : 1);
    if (n <= GS_NORM_256_MAX) return launch_norm<K, 1, 256>(A, 1, cap, d_out, accumulate, stream);
    if (n <= GS_NORM_512_MAX) return launch_norm<K, 1, 512>(A, 1, cap, d_out, accumulate, stream);
    if constexpr (K < 8)
        if (n <= GS_NORM_1024_MAX) return launch_norm<K, 1, 1024>(A, 2, cap, d_out, accumulate, stream);
    return launch_norm<K, 1, 512>(A, run, cap, d_out, accumulate, stream);
}

template <int K>
static hipError_t launch_norm_by_streams(const SqnormArgs &A, int64_t run, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    if (A.k == K) return launch_norm_many<K>(A, run, cap, d_out, accumulate, stream);
    if constexpr (K < GS_MAX_K) return launch_norm_by_streams<K + 1>(A, run, cap, d_out, accumulate, stream);
    return hipErrorInvalidValue;
}

// Up to four 4096-element tiles a single workgroup reads the range and no fold has to follow (13 k elements, k = 1 / 3: 3.3/3.9 us against
// 5.5/9.4 with the fold), from 5 streams on while there are up to 2^16 values to read, or one tile.  On the GPU alone those 2^16 are too many, 6 k
// elements, k = 5 / 8 2.8/3.35 us against 3.8/3.8 with the fold, 8 k 3.5/4.2 against 3.8/3.9, 13 k, k = 5 4.5 against 4.0; but called one after the other
// the second launch's host time counts too: norm and step, 8 k, k = 8 9.7 against 11.8, 13 k, k = 5 9.7 against 11.7 (one_workgroup has the line for
// captured ones).  The lanes whose groups lie in all four
// tiles have them in flight together; in a range that ends before, the others take them one after another.
// Above that: with up to 4 streams 256 lanes and one group of U tiles up to 4 M elements, 512 lanes and
// two tiles beyond (four from 2^29 elements on, where longer runs win 2-3 %, and always for three streams: 6.3 M / 12.6 M
// / 201 M 9.7/15.2/174 us against 10.3/16.3/180; level at 50 M); one stream is best in 256 lanes at every size, in runs of
// four tiles, and of eight from 2^29 elements on (805 M with the fold 236 against 240) and from 2^23 to 3 * 2^24: there the fold, which takes
// a latency for each 1024 partials and one launch more above 8192 of them, is long beside the reading (with it 8.4 M / 12.6 M / 34 M
// 7.0/8.0/14.9 against 8.1/8.6/16.4; 67 M / 200 M / 400 M 28.3/71.7/126 against 27.8/67.4/124).  On some of the CUs the longer runs
// win at every length from 2^23 on (16 / 64 / 128 CUs, 100 M 321/88.7/54.7 against 363/98.3/55.1; 300 M 942/250/150 against 1068/283/153).
// From 5 streams on a workgroup reads one tile while that makes no more workgroups than the chip holds a few times over, and two
// beyond: 256 lanes up to 3 * 2^18 elements (600 k, k = 11 / 32 6.15/10.7 us against 6.5/11.6 in 512; 900 k 7.1/13.1 against 6.8/12.4), 512 and one
// tile up to 5.5 M (against two tiles of 1024 lanes, with the end of the range left in the cache: 2.2 M, k = 5 / 8 / 16 / 32 7.1/9.9/16.1/28.7
// against 8.1/12.1/20.5/38.3, 3 M 8.7/11.8/19.9/36.1 against 9.2/12.9/22.2/40.9, 5 M 12.5/17.4/30.4/58.3 against 12.4/18.2/33.3/62.6), then two tiles (8 M,
// k = 8 / 16 / 32 24.8/47.3/83.2 against 25.0/46.1/82.5 with one, 10 M 30.3/55.7/103.7 against 31.7/56.5/105.5); 5 to 7 streams read those in 1024 lanes up
// to 2^25 (k = 5, 8 M / 20 M 16.5/36.3 against 17.0/37.6).
// The lines are the same where nothing is left in the cache.  Accumulating, against 256 lanes up to 2^20 and 1024 with two tiles above 2^21 (and a
// number of streams told at run time): 1 M, k = 8 / 32 6.4/15.2 us against 7.2/16.9, 2.2 M 9.3/25.6 against 11.3/33.1, 3 M 11.0/32.6 against 11.9/35.2; 1-2.6 %
// behind at 4 and 5.6 M from eight streams on (k = 32 40.5/57.0 against 39.8/55.5), level at 5.4 and 8 M.  On 16 / 64 / 128 CUs, 2.2 M, k = 8 50.9/16.5/11.3
// against 52.1/19.1/13.8, 5.4 M, k = 16 226/63.8/38.3 against 229/66.7/41.6; where the workgroups happen to leave a last wave nearly empty 1-4 %
// behind (800 k, k = 16 on 16 CUs 38.4 against 37.8; 3 M, k = 32 on 128 44.6 against 42.9).
// us, all with the fold and the last lines left in the cache, against 256 lanes with 8 tiles one after another, without either:
//   100 k  k = 1/3/8/32  4.2/4.3/4.2/5.5 against 3.5/6.3/8.1/38     12.6 M  8.1/16.0/36.1/124 against 8.4/15.8/35.4/151
//   1 M    k = 1/3/8/32  4.3/4.9/6.4/13.6 against 5.8/10.6/8.6/40   201 M   65/176/455/1797 against 89/191/474/1932
//   3 M    k = 1/3/8/32  4.9/6.8/11.3/35 against 6.5/11.5/11.0/51   805 M   236/713/1848/7849 against 347/737/1851/7903
//   On some of the CUs, 4 to 7 streams: once each CU has some tens of thousands of elements to read, 256 lanes,
//   four loads in flight and eight tiles one after another (k = 4 / 5, 50 M elements: 16 CUs 523/694 us against
//   651/860 in the shapes below, 128 CUs 84/110 against 97/122; 3.3 M on 128 CUs, 26 k elements each, 11.6/16.2
//   against 10.9/14.1).  The two meet at 96 k elements per CU for four streams (12.6 M on 128 CUs 29.7 against
//   30.6, 3.3 M on 64 CUs 16.2 against 14.5) and at 48 k above (3.3 M on 64 CUs, k = 5 18.2 against 20.2).
static hipError_t launch_grad_norm(const SqnormArgs &A, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    const int64_t n = A.end - A.begin;
    if (A.k >= 4 && A.k <= 7 && n > GS_LATENCY_MAX) {
        const int cus = budget_cus(stream);
        if (cus > 0 && n / cus >= (A.k == 4 ? 2 : 1) * GS_BUDGET_RUN_MIN)
            return launch_norm<0, 1, 256, 4>(A, 8, cap, d_out, accumulate, stream);
    }
    const bool small = n <= GS_NORM_SMALL_MAX;
    const int64_t run = n < GS_NORM_LONG_MIN ? 2 : 4;
    const int64_t tiles = tiles_of(A.begin, A.end, GS_ONE_BLOCK * 4);
    if (tiles <= 4) {
        switch (A.k) {
        case 1: return launch_norm_one<1, 4>(A, d_out, accumulate, stream);
        case 2: return launch_norm_one<2, 4>(A, d_out, accumulate, stream);
        case 3: return launch_norm_one<3, 4>(A, d_out, accumulate, stream);
        case 4: return launch_norm_one<4, 4>(A, d_out, accumulate, stream);
        }
    }
    switch (A.k) {
    case 1: {
        const bool long_run = n >= GS_NORM_RUN8_MIN && (n <= GS_NORM_RUN8_MAX || n >= GS_NORM_LONG_MIN || on_cu_budget(stream));
        return launch_norm<1, 4, 256>(A, long_run ? 8 : 4, cap, d_out, accumulate, stream);
    }
    case 2:
        if (small) return launch_norm<2, 2, 256>(A, 2, cap, d_out, accumulate, stream);
        return launch_norm<2, 4, 512>(A, 4, cap, d_out, accumulate, stream);
    case 3:
        if (small) return launch_norm<3, 2, 256>(A, 2, cap, d_out, accumulate, stream);
        return launch_norm<3, 2, 512>(A, 4, cap, d_out, accumulate, stream);
    case 4:
        if (small) return launch_norm<4, 2, 256>(A, 2, cap, d_out, accumulate, stream);
        return launch_norm<4, 2, 512>(A, run, cap, d_out, accumulate, stream);
    }
    return launch_norm_by_streams<5>(A, run, cap, d_out, accumulate, stream);
}

// MOST: the streams that a call of this shape has
template <int BLOCK, int EL, int DEPTH, bool KEEPS, int MOST>
static hipError_t launch_staged_kernel(const SqnormArgs &A, int grid, int span, hipStream_t stream)
{
    const int keep_block = first_kept(A.begin, A.keep_from, (int64_t)span * BLOCK * EL, BLOCK * EL, grid);
    if constexpr (MOST > 8) {
        if (A.k > 8) {
            void (*const kernel)(int64_t, int, int, int64_t, float *, GradTable, int, double *) = k_grad_accum_sqnorm<BLOCK, EL, DEPTH, KEEPS>;
            return launch(kernel, grid, BLOCK, 0, stream, A.begin, span, keep_block, A.end, A.acc, A.gt, A.k, A.partials);
        }
    }
    GradTableOf<8> gt;
    for (int j = 0; j < 8; ++j) gt.g[j] = A.gt.g[j];
    void (*const kernel)(int64_t, int, int, int64_t, float *, GradTableOf<8>, int, double *) = k_grad_accum_sqnorm<BLOCK, EL, DEPTH, KEEPS>;
    return launch(kernel, grid, BLOCK, 0, stream, A.begin, span, keep_block, A.end, A.acc, gt, A.k, A.partials);
}

template <int BLOCK, int EL, int DEPTH, bool KEEPS = true, int MOST = GS_MAX_K>
static hipError_t launch_staged(const SqnormArgs &A, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    int64_t tiles = tiles_of(A.begin, A.end, (int64_t)BLOCK * EL);
    if (tiles < 1) tiles = 1;
    const int64_t span = fit_span(tiles, 1, 1, cap, BLOCK);
    if (span == 0) return hipErrorInvalidValue;
    const int grid = (int)((tiles + span - 1) / span);
    const hipError_t e = KEEPS && A.keep_from < A.end ? launch_staged_kernel<BLOCK, EL, DEPTH, KEEPS, MOST>(A, grid, (int)span, stream)
                                                      : launch_staged_kernel<BLOCK, EL, DEPTH, false, MOST>(A, grid, (int)span, stream);
    if (e != hipSuccess) return e;
    return launch_fold(A.partials, cap, grid, d_out, accumulate, stream);
}

// The arguments one by one, as in the norm (launch_norm_kernel): 3 M, k = 2 / 4 / 8 8.4/9.9/12.8 us with the fold against 8.9/10.3/13.2 with a block
// of 330 bytes, 400 k 4.7/5.0/5.6 against 4.85/5.1/5.75; level from 16 M on.
// One tile per workgroup wherever the partials fit.  The plain shape has two gradient loads in flight, 4 elements per
// lane, 64 lanes up to 8 streams and 128 beyond; us per launch, k = 2 / 4 / 8 / 16, against it:
//   <= 2^19  four (below 8 streams) or eight in flight:  300 k  5.0/5.1/5.6/6.4 against 5.1/5.7/6.6/8.7
//   <= 2^22  1024 lanes, four in flight (a sixteenth of the partials):  2 M  7.0/8.4/10.4/15.4 against 9.0/10.3/12.4/16.3.
//            Up to 16 streams also from 4.5 to 10 M elements, with the end of the sum left in the cache: 4.6 M, k = 1 / 4 / 8 / 16
//            10.1/13.6/18.3/30.9 us against 12.3/15.1/20.9/35.2 in the plain shape, 9 M 15.6/22.7/32.5/57.1 against 18.0/23.5/34.4/59.5; with the
//            step 5 M 34.9/38.8/44.1/57.8 against 37.4/40.3/46.6/60.8.  Over 16 M the two are level, above that the plain shape wins.
//            More than 16 streams only up to 2^20 (600 k, k = 20 / 32  9.1/11.7 against 11.0/14.6; 1.5 M 15.9/22.2
//            against 14.9/20.0), and on some of the CUs fewer than 8 streams only up to 48 k elements per CU, from
//            where the many small workgroups win (16 CUs, k = 1 / 2 / 4: 1 M 16.6/18.7/25.6 against 14.9/16.0/22.9,
//            3.3 M 57/64/77 against 51/57/72; 64 CUs, 1 M 7.7/8.2/9.9 against 8.3/8.5/10.5)
//   >= 2^25, 8 streams or more and a multiple of 4: 2 elements per lane, 256 lanes, four in flight: 617 M, k = 8 / 12 /
//            16 / 20  1.92/2.70/3.53/4.39 ms against 1.93/2.75/3.59/4.43.  With streams left over
//            after the batches of four the plain shape wins (k = 9 / 10 / 14  2.14/2.41/3.19 against 2.27/2.60/3.33), and on
//            some of the CUs (100 M, k = 8, 16 CUs 2.78 against 3.39); so it does below 2^25, where 2 elements lose 3-40 %
//   workspace too small for a partial per 512 elements: up to 3 streams runs of 512-element tiles, else 4096-element tiles
//            one after another, two loads in flight either way (500 M, k = 1 / 3 / 8 / 16  0.49/0.80/1.71/3.15 ms in runs,
//            0.67/0.87/1.61/2.99 in wide tiles, 0.68/0.86/1.63/3.13 with four or eight in flight)
static hipError_t launch_staged_norm(const SqnormArgs &A, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    const int64_t n = A.end - A.begin;
    if (n <= GS_LATENCY_MAX) {
        if (A.k < 8) return launch_staged<128, 4, 4, false, 7>(A, cap, d_out, accumulate, stream);
        return launch_staged<64, 4, 8, false>(A, cap, d_out, accumulate, stream);
    }
    if (A.k <= 16 && n >= GS_STAGED_WIDE_AGAIN_MIN && n <= GS_STAGED_WIDE_AGAIN_MAX && !on_cu_budget(stream))
        return launch_staged<1024, 4, 4>(A, cap, d_out, accumulate, stream);
    const int cus = n <= GS_STAGED_WIDE_MAX && A.k < 8 ? budget_cus(stream) : 0;
    if (n <= (A.k <= 16 ? GS_STAGED_WIDE_MAX : GS_STAGED_WIDE_MANY_MAX) && !(cus > 0 && n / cus >= GS_BUDGET_RUN_MIN))
        return launch_staged<1024, 4, 4>(A, cap, d_out, accumulate, stream);
    if (tiles_of(A.begin, A.end, 512) > cap) {
        if (A.k <= 3) return launch_staged<128, 4, 2>(A, cap, d_out, accumulate, stream);
        return launch_staged<1024, 4, 2>(A, cap, d_out, accumulate, stream);
    }
    if (A.k >= 8 && A.k % 4 == 0 && n >= GS_STAGED_PAIR_MIN && !on_cu_budget(stream))
        return launch_staged<256, 2, 4>(A, cap, d_out, accumulate, stream);
    if (A.k <= 8 && tiles_of(A.begin, A.end, 256) <= cap) return launch_staged<64, 4, 2, true, 8>(A, cap, d_out, accumulate, stream);
    return launch_staged<128, 4, 2>(A, cap, d_out, accumulate, stream);
}

hipError_t launch_grad_sqnorm(const SqnormArgs &args, size_t workspace_bytes, double *d_out, int accumulate,
                              hipStream_t stream)
{
    const int64_t cap = partial_capacity(workspace_bytes);
    SqnormArgs A = args;
    const int64_t upto = A.acc || A.k < 2 ? GS_RESIDENT_MAX : A.k < 4 ? GS_KEEP_FEW_MIN : GS_KEEP_MANY_MIN;
    A.keep_from = A.acc && A.k > GS_STAGED_KEEP_MAX_K ? A.end : keep_from(A.begin, A.end, A.acc ? 4 : 2 * A.k, accumulate, stream, upto);
    if (!A.acc) return launch_grad_norm(A, cap, d_out, accumulate, stream);
    return launch_staged_norm(A, cap, d_out, accumulate, stream);
}

template <int U, int BLOCK>
static hipError_t launch_acc_norm(const float *acc, int64_t begin, int64_t end, double *partials, int64_t span, int64_t cap,
                                  double *d_out, int accumulate, hipStream_t stream)
{
    const int64_t tiles = tiles_of(begin, end, (int64_t)BLOCK * 4);
    span = fit_span(tiles, span, U, cap, BLOCK);
    if (span == 0) return hipErrorInvalidValue;
    const int grid = (int)((tiles + span - 1) / span);
    k_acc_sqnorm<U, BLOCK, false><<<grid, BLOCK, 0, stream>>>(acc, begin, end, keep_from(begin, end, 4, accumulate, stream), partials, 0, (int)span);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_fold(partials, cap, grid, d_out, accumulate, stream);
}

// As for the gradient norm: one workgroup, then 256 lanes, then 512 with four tiles in flight (50 M
// elements 34.4 us against 37.1); from 2^27 elements on eight tiles one after another, 256 lanes (805 M:
// 458 us against 477).
hipError_t launch_acc_sqnorm(const float *acc, int64_t begin, int64_t end, double *partials, size_t workspace_bytes,
                             double *d_out, int accumulate, hipStream_t stream)
{
    const int64_t cap = partial_capacity(workspace_bytes);
    const int64_t n = end - begin;
    if (tiles_of(begin, end, GS_ONE_BLOCK * 4) <= 4) {
        k_acc_sqnorm<4, GS_ONE_BLOCK, true><<<1, GS_ONE_BLOCK, 0, stream>>>(acc, begin, end, end, d_out, accumulate, 4);
        return hipGetLastError();
    }
    if (n <= GS_NORM_SMALL_MAX) return launch_acc_norm<4, 256>(acc, begin, end, partials, 4, cap, d_out, accumulate, stream);
    if (n < GS_ACC_NORM_LONG_MIN) return launch_acc_norm<4, 512>(acc, begin, end, partials, 4, cap, d_out, accumulate, stream);
    return launch_acc_norm<1, 256>(acc, begin, end, partials, 8, cap, d_out, accumulate, stream);
}

template <bool FIRST, bool NORM, int BLOCK, int EL, bool LWAIT, bool THROUGH = false>
static hipError_t launch_add_as(const AccumAddArgs &A, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    int64_t tiles = tiles_of(A.begin, A.end, (int64_t)BLOCK * EL);
    if (tiles < 1) tiles = 1;
    const int64_t span = fit_span(tiles, 1, 1, NORM ? cap : tiles, BLOCK);
    if (span == 0) return hipErrorInvalidValue;
    const int grid = (int)((tiles + span - 1) / span);
    k_accum_add<FIRST, NORM, BLOCK, EL, LWAIT, THROUGH><<<grid, BLOCK, 0, stream>>>(A, (int)span);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !NORM) return e;
    return launch_fold(A.partials, cap, grid, d_out, accumulate, stream);
}

template <int BLOCK>
static hipError_t launch_add_norm(const AccumAddArgs &A, int first, int64_t cap, double *d_out, int accumulate, hipStream_t stream)
{
    if (first) return launch_add_as<true, true, BLOCK, 4, false>(A, cap, d_out, accumulate, stream);
    return launch_add_as<false, true, BLOCK, 4, false>(A, cap, d_out, accumulate, stream);
}

// us per launch, each against 64 lanes with the buffer's load after the gradient's:
//   first micro-batch: it is made of stores, and fewer, wider workgroups issue them sooner.  256 lanes up to 900 k elements (1 M 2.6
//                                                       against 3.2), 512 up to 2^21 (2 M 3.5 against 4.6, and 3.85 in 256), then, where the
//                                                       end of the sum stays in the cache and the stores are plain, 128 (5 M / 15 M 7.8/16.9
//                                                       against 8.7/18.0, in 256 8.2/18.0) up to 2^25, where they are level (200 M on 0.3 % behind); 256 on
//                                                       some of the CUs
//   later ones: above 2^21 elements written through where the sum is not left in the cache (805 M 1167 us against 1195,
//   201 M 291 against 294; 64 CUs, 5 M / 20 M 18.2/64.6 against 18.8/66.2; the first micro-batch, which only writes, loses 2-4 % by it).
//   Up to there the L2s hold the sum for the next one: the hint alone (13 k / 800 k 1.97/3.03 against 2.26/3.26 written through; four
//   micro-batches and the step, 0.8 M / 2 M 16.6/28.4 against 18.0/29.4);
//   later ones, <= 2^22 or on some of the CUs only: both loads in flight
//                                                      1 M 3.2 against 3.7, 2 M 4.9 against 5.2; from 200 M on
//                                                       waiting is 0.5 % ahead, level in between
//   with the norm: both loads in flight; 256 lanes up to 2^19, then 1024 where the sum is not left in the cache (fewer partials: 2 M 7.5 against
//                                             9.7), up to 2^23; else, and beyond, 64 (12.6 M 25.1 against 26.2, 201 M 306 against 320).  That
//                                             call on its own takes longer while the partials count (5 M / 8 M 13.1/17.6 against 11.7/16.3 in 1024 lanes
//                                             that leave nothing), and what comes before and after it less: all micro-batches and the step, 5 M / 7 M,
//                                             2 of them 44.5/57.9 against 44.9/58.9, 4 62.0/79.8 against 63.6/82.0, 16 165/211 against 167/214.  Up to
//                                             2^22 that is no gain with two (2.3 M / 3 M 26.7/31.5 against 25.9/30.6) and up to 1 % with four and
//                                             more.  A sum of one micro-batch alone loses that way (5 M 37.4 against 35.8), and wide workgroups that
//                                             leave it in the cache make the fold wait for the write-back (3.3 M 16.6 against 13.3).
//   with a workspace too small for a partial per 256 elements, per 1024 or 4096.
hipError_t launch_accum_add(const AccumAddArgs &args, int first, size_t workspace_bytes, double *d_out, int accumulate,
                            hipStream_t stream)
{
    AccumAddArgs A = args;
    A.keep_from = keep_from(A.begin, A.end, 4, 0, stream);
    const int64_t n = A.end - A.begin;
    if (!d_out) {
        if (first) {
            if (n <= GS_ADD_FIRST_256_MAX || on_cu_budget(stream)) return launch_add_as<true, false, 256, 4, false>(A, 0, nullptr, 0, stream);
            if (n <= GS_RESIDENT_MAX) return launch_add_as<true, false, 512, 4, false>(A, 0, nullptr, 0, stream);
            if (n <= GS_ADD_FIRST_128_MAX) return launch_add_as<true, false, 128, 4, false>(A, 0, nullptr, 0, stream);
            return launch_add_as<true, false, 64, 4, false>(A, 0, nullptr, 0, stream);
        }
        if (n > GS_ADD_SMALL_MAX && !on_cu_budget(stream)) return launch_add_as<false, false, 64, 4, true, true>(A, 0, nullptr, 0, stream);
        if (n > GS_RESIDENT_MAX) return launch_add_as<false, false, 64, 4, false, true>(A, 0, nullptr, 0, stream);
        return launch_add_as<false, false, 64, 4, false>(A, 0, nullptr, 0, stream);
    }
    const int64_t cap = partial_capacity(workspace_bytes);
    if (accumulate || n <= (first ? GS_ADD_WIDE_MAX : GS_ADD_KEEP_MIN)) A.keep_from = A.end;
    const bool keeps = A.keep_from < A.end;
    if ((n > GS_ADD_WIDE_MAX || keeps) && tiles_of(A.begin, A.end, 256) <= cap)
        return launch_add_norm<64>(A, first, cap, d_out, accumulate, stream);
    if (n <= GS_LATENCY_MAX || (n > GS_ADD_WIDE_MAX && tiles_of(A.begin, A.end, 1024) <= cap))
        return launch_add_norm<256>(A, first, cap, d_out, accumulate, stream);
    return launch_add_norm<1024>(A, first, cap, d_out, accumulate, stream);
}

}  // namespace gs
