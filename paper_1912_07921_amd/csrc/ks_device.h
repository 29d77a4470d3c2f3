// Device-side building blocks shared by the gfx950 kernel files of the
// real-time TDDFT hot path: complex helpers, streaming loads and stores,
// reductions, Bloch phases, the H.psi work item and the projector gather /
// apply work items.
//
// H.psi = -1/2 Lap psi + (v + |A|^2/2) psi - i A.grad psi + V_NL psi on a
// uniform grid (section "Periodic systems": finite-difference Laplacian and
// gradient; eq. Hamiltonian_dipole: one-body potential; section
// "Magneto-optics": non-local pseudopotentials; section "t-SURFF": uniform
// vector potential), applied to batches of resident states (sections "Memory
// layout" and "GPUs").
//
// Stencil design (HBM bound: 32 B moved per point and state in FP64):
//  - a workgroup owns a tile of full x-rows (nx x TY) of one state and marches
//    along z over a chunk of planes;
//  - each thread keeps the z-neighbours' share of its points in registers, so
//    every value is loaded from memory once per pass (plus the y-halo rows);
//  - the current xy plane (with 4 halo rows on each side) is staged in LDS for
//    the x and y neighbours; x-rows are read as consecutive 16-byte complex
//    values across the wavefront (coalesced);
//  - the KB term V_NL psi, formed on the projector hull rows by the apply
//    work item, is read at hull points and added before the single store
//    of the output; the Taylor recurrence scale, the final Taylor sum, the
//    ETRS predictor and the density/norm partial sums are fused into the
//    epilogue.
#pragma once

#include "ks_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

namespace ks {

// Half-width-4 central weights: Laplacian (c0..c4) and gradient (d1..d4).
constexpr double kLap[5] = {-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0,
                            -1.0 / 560.0};
constexpr double kGrad[5] = {0.0, 4.0 / 5.0, -1.0 / 5.0, 4.0 / 105.0,
                             -1.0 / 280.0};

template <class R> struct Cplx;
template <> struct Cplx<double> { using T = double2; };
template <> struct Cplx<float> { using T = float2; };

template <class V> __device__ __forceinline__ V czero()
{
    V r;
    r.x = 0;
    r.y = 0;
    return r;
}
template <class V> __device__ __forceinline__ V cmk(double a, double b)
{
    V r;
    r.x = a;
    r.y = b;
    return r;
}
template <class V> __device__ __forceinline__ V cadd(V a, V b)
{
    V r;
    r.x = a.x + b.x;
    r.y = a.y + b.y;
    return r;
}
template <class V> __device__ __forceinline__ V csub(V a, V b)
{
    V r;
    r.x = a.x - b.x;
    r.y = a.y - b.y;
    return r;
}
template <class V, class S> __device__ __forceinline__ V cscale(V a, S s)
{
    V r;
    r.x = a.x * s;
    r.y = a.y * s;
    return r;
}
template <class V> __device__ __forceinline__ V cmul(V a, V b)
{
    V r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}
// a * conj(b)
template <class V> __device__ __forceinline__ V cmulc(V a, V b)
{
    V r;
    r.x = a.x * b.x + a.y * b.y;
    r.y = a.y * b.x - a.x * b.y;
    return r;
}

// Fused multiply-adds written out, so that every kernel that forms a value
// rounds it alike; acc + s a for a complex a.
__device__ __forceinline__ double rfma(double a, double b, double c)
{
    return __builtin_fma(a, b, c);
}
__device__ __forceinline__ float rfma(float a, float b, float c)
{
    return __builtin_fmaf(a, b, c);
}
template <class V, class S> __device__ __forceinline__ V cfma(S s, V a, V acc)
{
    acc.x = rfma(s, a.x, acc.x);
    acc.y = rfma(s, a.y, acc.y);
    return acc;
}
// a b with its roundings fixed (every kernel that applies a phase gets the
// same bits)
template <class V> __device__ __forceinline__ V cmulf(V a, V b)
{
    V r;
    r.x = rfma(a.x, b.x, -(a.y * b.y));
    r.y = rfma(a.y, b.x, a.x * b.y);
    return r;
}
// |a|^2 with its roundings fixed
__device__ __forceinline__ double abs2f(double re, double im)
{
    return rfma(im, im, re * re);
}
// A copy the optimiser cannot trace: what is computed from it inside a loop
// stays in the loop (the LDS addresses of the H.psi kernel would otherwise be
// hoisted into tens of vector registers and spill).
__device__ __forceinline__ int fresh(int s)
{
    asm volatile("" : "+s"(s));
    return s;
}
// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ float uni(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uni(double v)
{
    typedef int i2 __attribute__((ext_vector_type(2)));
    i2 b = __builtin_bit_cast(i2, v);
    b.x = __builtin_amdgcn_readfirstlane(b.x);
    b.y = __builtin_amdgcn_readfirstlane(b.y);
    return __builtin_bit_cast(double, b);
}

// Every buffer the kernels touch is global memory.  Accesses go through an
// explicitly global pointer, so that pointers read from memory (the job
// table of the batched form) compile to global, not flat, instructions.
template <class T> using gptr_t = __attribute__((address_space(1))) T *;
template <class T> __device__ __forceinline__ gptr_t<T> gp(T *p)
{
    return (gptr_t<T>)p;
}

// Loads and stores of the HIP vector classes through global pointers go by
// the compiler's native vector types.
typedef double gd2_t __attribute__((ext_vector_type(2)));
typedef float gf2_t __attribute__((ext_vector_type(2)));
typedef double gd4_t __attribute__((ext_vector_type(4)));
typedef int gi4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 gld(const double2 *p)
{
    const gd2_t v = *gp(reinterpret_cast<const gd2_t *>(p));
    return make_double2(v.x, v.y);
}
__device__ __forceinline__ float2 gld(const float2 *p)
{
    const gf2_t v = *gp(reinterpret_cast<const gf2_t *>(p));
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ double4 gld(const double4 *p)
{
    const gd4_t v = *gp(reinterpret_cast<const gd4_t *>(p));
    return make_double4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ int4 gld(const int4 *p)
{
    const gi4_t v = *gp(reinterpret_cast<const gi4_t *>(p));
    return make_int4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void gst(double2 *p, double2 v)
{
    *gp(reinterpret_cast<gd2_t *>(p)) = gd2_t{v.x, v.y};
}
__device__ __forceinline__ void gst(float2 *p, float2 v)
{
    *gp(reinterpret_cast<gf2_t *>(p)) = gf2_t{v.x, v.y};
}

template <class R, class T> __device__ __forceinline__ typename Cplx<R>::T
ldc(const T *p, long i)
{
    T v = gld(p + i);
    typename Cplx<R>::T r;
    r.x = (R)v.x;
    r.y = (R)v.y;
    return r;
}

// Streaming stores and loads of data touched once per pass (the H.psi
// outputs, the Taylor terms read by the final pass): non-temporal, so they
// do not evict the plane and halo lines that neighbouring workgroups reuse
// from L2.
#ifndef KS_NT_STORE
#define KS_NT_STORE 1
#endif
#ifndef KS_NT_LOAD
#define KS_NT_LOAD 1
#endif
typedef double nd2_t __attribute__((ext_vector_type(2)));
typedef float nf2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void st_stream(double2 *p, double x, double y)
{
#if KS_NT_STORE
    nd2_t v = {x, y};
    __builtin_nontemporal_store(v, gp(reinterpret_cast<nd2_t *>(p)));
#else
    gst(p, make_double2(x, y));
#endif
}
__device__ __forceinline__ void st_stream(float2 *p, float x, float y)
{
#if KS_NT_STORE
    nf2_t v = {x, y};
    __builtin_nontemporal_store(v, gp(reinterpret_cast<nf2_t *>(p)));
#else
    gst(p, make_float2(x, y));
#endif
}
__device__ __forceinline__ void st_stream(double *p, double x)
{
#if KS_NT_STORE
    __builtin_nontemporal_store(x, gp(p));
#else
    *gp(p) = x;
#endif
}
__device__ __forceinline__ double2 ld_stream(const double2 *p)
{
#if KS_NT_LOAD
    const nd2_t v =
        __builtin_nontemporal_load(gp(reinterpret_cast<const nd2_t *>(p)));
    return make_double2(v.x, v.y);
#else
    return gld(p);
#endif
}
__device__ __forceinline__ float2 ld_stream(const float2 *p)
{
#if KS_NT_LOAD
    const nf2_t v =
        __builtin_nontemporal_load(gp(reinterpret_cast<const nf2_t *>(p)));
    return make_float2(v.x, v.y);
#else
    return gld(p);
#endif
}

// a state value at a sphere point for the gather (non-temporal with
// KS_GATHER_NT: the states are larger than the MALL and the next pass
// streams them again anyway, while the point tables are re-read by every
// state group)
#ifndef KS_GATHER_NT
#define KS_GATHER_NT 1
#endif
template <class R, class T>
__device__ __forceinline__ typename Cplx<R>::T ldc_g(const T *p, long i)
{
    const T v = KS_GATHER_NT ? ld_stream(p + i) : gld(p + i);
    typename Cplx<R>::T r;
    r.x = (R)v.x;
    r.y = (R)v.y;
    return r;
}

// Raw buffer accesses (gfx9 buffer descriptor, no stride): an offset at or
// beyond the buffer's size reads zero and drops a store, so an access with
// nothing to move needs no branch around it.
typedef __amdgpu_buffer_rsrc_t BufRes;
__device__ __forceinline__ BufRes buf_res(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0,
                                             bytes, 0x00020000);
}
// A buffer of any size below 2 GiB whose accesses keep their own bounds
// (kBufNone: nothing to move), or an empty one (use == false).
constexpr unsigned kBufNone = 0x80000000u;
__device__ __forceinline__ BufRes buf_any(const void *p, bool use)
{
    return buf_res(p, use ? 0x7fffffff : 0);
}
// off is the per-thread byte offset (range checked against the buffer's
// size), soff a byte offset uniform over the wavefront (added to the address
// past the check).
template <class T>
__device__ __forceinline__ T bld_raw(BufRes r, unsigned off, int soff);
template <>
__device__ __forceinline__ double2 bld_raw<double2>(BufRes r, unsigned off,
                                                    int soff)
{
    return __builtin_bit_cast(
        double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}
template <>
__device__ __forceinline__ float2 bld_raw<float2>(BufRes r, unsigned off,
                                                  int soff)
{
    return __builtin_bit_cast(
        float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
}
// the same with the non-temporal hint (streams read once)
template <class T>
__device__ __forceinline__ T bld_raw_nt(BufRes r, unsigned off, int soff);
template <>
__device__ __forceinline__ double2 bld_raw_nt<double2>(BufRes r, unsigned off,
                                                       int soff)
{
    return __builtin_bit_cast(
        double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 2));
}
template <>
__device__ __forceinline__ float2 bld_raw_nt<float2>(BufRes r, unsigned off,
                                                     int soff)
{
    return __builtin_bit_cast(
        float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 2));
}
// complex value of storage type T, in precision R
template <class R, class T>
__device__ __forceinline__ typename Cplx<R>::T bld(BufRes r, unsigned off,
                                                   int soff)
{
    const T v = bld_raw<T>(r, off, soff);
    typename Cplx<R>::T o;
    o.x = (R)v.x;
    o.y = (R)v.y;
    return o;
}
template <class R, class T>
__device__ __forceinline__ typename Cplx<R>::T bld_nt(BufRes r, unsigned off,
                                                      int soff)
{
    const T v = bld_raw_nt<T>(r, off, soff);
    typename Cplx<R>::T o;
    o.x = (R)v.x;
    o.y = (R)v.y;
    return o;
}
__device__ __forceinline__ double bld_d(BufRes r, unsigned off, int soff)
{
    return __builtin_bit_cast(
        double, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
}
// Non-temporal stores (the outputs are read by the next pass only).  No
// scalar offset: the compiler leaves no wait state between a 16-byte store
// that has one and the next write of its data registers, and on gfx950 such
// a store was seen to take the overwritten data; the plane goes into the
// buffer's base address instead.
template <class T>
__device__ __forceinline__ void bst(BufRes r, unsigned off, double x,
                                    double y);
template <>
__device__ __forceinline__ void bst<double2>(BufRes r, unsigned off,
                                             double x, double y)
{
    typedef int i4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(
        __builtin_bit_cast(i4, make_double2(x, y)), r, off, 0, 2);
}
template <>
__device__ __forceinline__ void bst<float2>(BufRes r, unsigned off, double x,
                                            double y)
{
    typedef int i2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(i2, make_float2((float)x, (float)y)), r, off, 0,
        2);
}
__device__ __forceinline__ void bst_d(BufRes r, unsigned off, double v)
{
    typedef int i2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i2, v), r, off,
                                          0, 2);
}

__device__ __forceinline__ int floordiv(int a, int n)
{
    return a >= 0 ? a / n : -((-a + n - 1) / n);
}

template <class T> __device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// Deterministic block reduction of NV values; result valid in thread 0.
template <class T, int NV>
__device__ __forceinline__ void block_sum(T (&v)[NV], T *sbuf)
{
    const int tid = threadIdx.x;
    const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i)
        v[i] = wave_sum(v[i]);
    if ((tid & 63) == 0)
#pragma unroll
        for (int i = 0; i < NV; ++i)
            sbuf[(tid >> 6) * NV + i] = v[i];
    __syncthreads();
    if (tid == 0)
        for (int i = 0; i < NV; ++i) {
            T s = 0;
            for (int w = 0; w < nw; ++w)
                s += sbuf[w * NV + i];
            v[i] = s;
        }
}


// ---------------------------------------------------------------------------
// Bloch phases.  kph[k][a] = exp(i k_a L_a) is tabulated on the host; a wrap
// by w cells along axis a multiplies by kph[k][a]^w (|w| is 1 except on
// axes shorter than the stencil).
// ---------------------------------------------------------------------------
template <class V>
__device__ __forceinline__ V phase_pow(const double2 *kph, int axis, int w)
{
    const double2 kv = gld(kph + axis);
    V ph = cmk<V>(kv.x, kv.y);
    if (w < 0) {
        ph.y = -ph.y;
        w = -w;
    }
    V r = ph;
    for (int i = 1; i < w; ++i)
        r = cmul(r, ph);
    return r;
}

template <class V>
__device__ __forceinline__ V shift_phase(const double2 *kph, int code)
{
    // lattice shift packed as three signed bytes (x, y, z)
    V r = cmk<V>(1.0, 0.0);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int t = (int)(signed char)((code >> (8 * ax)) & 0xff);
        if (t)
            r = cmul(r, phase_pow<V>(kph, ax, t));
    }
    return r;
}

__device__ __forceinline__ double axis_coord(int n, double h, int per, int i)
{
    return per ? i * h : (i - 0.5 * (n - 1)) * h;
}

// ---------------------------------------------------------------------------
// Workgroups are handed to the 8 XCDs round robin in launch order; remap the
// launch index so that each XCD receives a contiguous range of work items
// (neighbouring y-tiles of the same state, which share halo rows in that
// XCD's L2).
// ---------------------------------------------------------------------------
#ifndef KS_XCD_REMAP
#define KS_XCD_REMAP 1
#endif
__device__ __forceinline__ int xcd_remap(int L, int nblk)
{
    if (!KS_XCD_REMAP)
        return L;
    constexpr int X = 8;
    const int per = nblk / X, rem = nblk % X;
    const int x = L % X, i = L / X;
    return x * per + min(x, rem) + i;
}

// ---------------------------------------------------------------------------
// H.psi with a fused epilogue.  R: arithmetic precision; InT: storage type of
// the input states; TT: storage type of t-terms (t1, t2, term outputs);
// GRAD: the velocity-gauge term -i A.grad (0: none, 1: every axis, 2: A along
// z only); HM: halo loads per thread and plane; RPT: rows per thread.
//
// A workgroup marches its tile of full x-rows along z.  LDS holds the current
// xy plane padded by 4 rows above and below and 4 columns left and right: the
// neighbours' values, zeros (zero boundary; written once) or Bloch-wrapped
// values, so the x and y taps are branch-free LDS reads; two plane buffers
// alternate, one barrier per plane.  A thread owns RPT adjacent rows, whose y
// taps overlap: 9 + RPT - 1 reads serve all of them.
// Along z the FP64 kernels split the star: plane z adds its x, y, centre and
// z-4 .. z-1 taps to the output of plane z and its own z+m taps to the pending
// outputs of planes z-1 .. z-4, the last of which is then complete and stored.
// Four previous values and four pending outputs per point live in registers,
// their slots fixed by unrolling the march by four, and a plane's own rows and
// its halo rows are loaded at the same time, so that neighbouring tiles find
// them in the L2 (128^3, 64 states: 4.9 -> 3.9 GB fetched per term pass).
// Every tap is one FMA with a coefficient that carries -1/2 c_m / h^2, from
// the smallest weight to the largest: half the rounding error of pairwise
// sums.  The FP32 kernels keep a column of nine values and the order of their
// sums.  So do FP64 tiles of one row (rows above 256 points; eight or more halo
// loads per thread), with the split star's order of sums: their neighbours are
// all halo rows, which the split star asks for while the tiles that own them
// do, where the column has asked four planes before (400 x 24 x 30 x 6 with A
// along every axis 60.4 -> 51.3 us a pass, 512 x 20 x 40 x 8 78 -> 69, 300 x 90
// x 64 x 16 640 -> 562).  Every access is a raw buffer access with a constant
// per-thread offset and the plane in the scalar offset.
// What bounds it: large launches memory (128^3 x 64 states FP64 term pass, 6.0
// GB through the L2 in 1.05 ms = 5.7 TB/s, where a plain copy reaches 6.6;
// without the x taps 1.02 ms), launches of few states the chain of barrier,
// LDS reads, FMAs and loads of each plane (~0.6 us with one row per thread,
// whatever is loaded), which is why those get short chunks of low tiles.
// Loads run PF planes ahead of their use: 2, or 1 in the FP64 kernels with
// two rows per thread or the column, whose registers hold no second set (64^3 x
// 32, one row: 80 -> 72 us with 2; two rows: 70 -> 127 us, spilled; the column
// 52 -> 85 us).  The KB term V_NL in is precomputed on the hull rows
// (k_kbapply) and added with one coalesced read.
// ---------------------------------------------------------------------------
extern __shared__ double2 smem_d2[];

// One work item of the H.psi pass described by `a`: work item w is
// (launch state, z-chunk, y-tile).  The whole workgroup takes part.  Avec
// holds the vector potential (x, y, z) and |A|^2 / 2 of the pass.  Thread
// t owns column x = t % nx of the rows base .. base + rpt - 1 with base =
// rpt * (t / nx) (the last pair of an odd tile is shifted up by one and its
// first row left to its neighbour).
template <class R, class InT, class TT, int MODE, int GRAD, int HM, int RPT>
__device__ __forceinline__ void hpsi_item(const HArgs &a, const int w,
                                          const double4 Avec)
{
    using V = typename Cplx<R>::T;
    unsigned char *smem_raw = reinterpret_cast<unsigned char *>(smem_d2);
    constexpr bool FIN = MODE == kFinal || MODE == kFinalPred;
    constexpr bool CUR = MODE == kCurrent;
    constexpr bool ENE = MODE == kEnergy;

    const int nx = a.geo.nx, ny = a.geo.ny, nz = a.geo.nz;
    const int P = nx * ny;
    const long N = a.geo.N;
    const int ntiles = a.ntile_y * a.nzc;
    const int sl = w / ntiles;
    const int tile = w - sl * ntiles;
    const int zc = tile / a.ntile_y;
    const int tile_y = tile - zc * a.ntile_y;
    const int sg = a.sg0 + sl;
    const int kk = sg / a.nstates;
    const double2 *kph = a.kph + 3 * kk;
    const int perx = a.geo.per[0], pery = a.geo.per[1], perz = a.geo.per[2];

    const int TY = a.TY;
    // rows per thread of this item's shape (the launch's RPT is the most
    // any item of it uses)
    const int rpt = RPT > 1 ? min(a.rpt, TY) : 1;
    const int TYh = (TY + rpt - 1) / rpt;
    const int y0 = tile_y * TY;
    const int rows = min(TY, ny - y0);
    const int tid = threadIdx.x;
    const int nthr = blockDim.x;
    const int x = tid % nx;
    const int yl = tid / nx;
    const int RS = nx + 2 * kHalf;                  // LDS row stride
    const int row0 = yl < TYh ? min(yl * rpt, TY - rpt) : 0;
    const int own = (row0 + kHalf) * RS + x + kHalf;  // LDS slot of row 0
    // byte offsets within a plane of 16, 8 and 4-byte elements.  A row that
    // two threads hold is stored by both, with the same value, and counted
    // by the one that owns it (act).
    bool valid[RPT], act[RPT];
    unsigned p16[RPT], p8[RPT], p4[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        valid[r] = r < rpt && yl < TYh && row0 + r < rows;
        act[r] = valid[r] && row0 + r >= yl * rpt;
        const unsigned p = (unsigned)((y0 + row0 + r) * nx + x);
        p16[r] = valid[r] ? p * 16u : kBufNone;
        p8[r] = valid[r] ? p * 8u : kBufNone;
        p4[r] = valid[r] ? p * 4u : kBufNone;
    }
    const int z0 = zc * a.zchunk;
    const int z1 = min(nz, z0 + a.zchunk);
    // FP64 scatters plane z's z taps to pending outputs; FP32, and FP64 tiles
    // of one row, gather them from a column of nine values (below)
    constexpr bool F64 = sizeof(R) == 8;
    constexpr bool SC = F64 && !(RPT == 1 && HM >= 8 && !CUR && !ENE);
    constexpr bool COL64 = F64 && !SC;
    const int zend = SC && !CUR ? z1 + 4 : z1;      // planes marched

    const int plane = (TY + 2 * kHalf) * RS;
    V *buf0 = reinterpret_cast<V *>(smem_raw);
    V *buf1 = buf0 + plane;
    V *sPh = buf1 + plane;        // x/y wrap phases, 81 entries
    V *sPz = sPh + 81;            // z wrap phases, 9 entries
    int2 *sRow = reinterpret_cast<int2 *>(sPz + 9);   // hull rows of tile

    // ---- buffers.  Every per-plane access is a raw buffer access whose
    // per-thread offset is out of range where there is nothing to move, and
    // whose buffer is empty for a plane outside the grid or the chunk (the
    // hardware then returns zero, or drops the store), so no memory
    // instruction sits behind a branch and the compiler knows exactly how
    // many are in flight.  The range check covers the per-thread offset, the
    // plane rides in the scalar offset. ----
    const InT *in = reinterpret_cast<const InT *>(a.in) + (size_t)sl * N;
    const bool proj = !CUR && a.rowinfo != nullptr;
    const V *Wst = reinterpret_cast<const V *>(a.W) + (size_t)sl * a.nhull;
    const size_t sN = (size_t)sl * N;
    // the potential: FP64, or its FP32 copy in the FP32 kernels (half the
    // bytes of the stream every state re-reads)
    constexpr bool V32 = sizeof(R) == 4;
    constexpr unsigned VB = V32 ? 4u : 8u;
    const void *vptr = CUR ? nullptr
                           : (V32 ? (const void *)a.v32 : (const void *)a.v);
    using OutT = typename std::conditional<MODE == kTerm, TT, double2>::type;
    OutT *out = CUR || ENE ? nullptr : reinterpret_cast<OutT *>(a.out) + sN;
    const BufRes rw = buf_any(Wst, proj);
    auto off_of = [&](int r, size_t elem) -> unsigned {
        return elem == 16 ? p16[r] : (elem == 8 ? p8[r] : p4[r]);
    };

    // plane of the grid that plane zq maps to (-1: none); the own rows are
    // needed on planes z0 - 4 .. z1 + 3
    auto wrap_z = [&](int zq) -> int {
        if (perz) {
            while (zq < 0)
                zq += nz;
            while (zq >= nz)
                zq -= nz;
        }
        return zq >= 0 && zq < nz ? zq : -1;
    };
    auto own_ld = [&](int r, int zz) -> V {
        return bld<R, InT>(buf_any(in, zz >= 0), off_of(r, sizeof(InT)),
                           max(zz, 0) * P * (int)sizeof(InT));
    };
    // the own rows of plane zq as loaded, with their Bloch phase
    auto own_fix = [&](V v, int zq) -> V {
        if (perz && (zq < 0 || zq >= nz)) {
            int wz = 0;
            for (; zq < 0; zq += nz)
                --wz;
            for (; zq >= nz; zq -= nz)
                ++wz;
            v = cmulf(v, sPz[wz + 4]);
        }
        return v;
    };
    // the first planes of the column: they are in flight during the setup.
    // Split star: p[r][s] holds plane z < z0 with (z - z0) & 3 == s; column:
    // q[r][m] holds plane z + m - 4.
    V p[RPT][4], q[RPT][9], c[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        if constexpr (SC) {
#pragma unroll
            for (int m = 1; m <= 4; ++m)
                p[r][4 - m] = own_ld(r, wrap_z(z0 - m));
            c[r] = own_ld(r, z0);
        } else {
#pragma unroll
            for (int m = 0; m <= 8; ++m)
                q[r][m] = own_ld(r, wrap_z(z0 - 4 + m));
        }
    }

    // ---- Bloch phases of x/y wraps by -4..4 cells: sPh[(wy+4)*9 + wx+4],
    // of z wraps: sPz[wz+4]; hull rows of this tile: sRow[(z-z0)*TY + row] =
    // (first x | (count - 1) << 16, hull index of x = 0), none: first x
    // beyond the row ----
    if (perx || pery || perz)
        for (int t = tid; t < 81 + 9; t += nthr) {
            V ph;
            if (t < 81) {
                const int wx = t % 9 - 4, wy = t / 9 - 4;
                ph = cmk<V>(1.0, 0.0);
                if (wx)
                    ph = cmulf(ph, phase_pow<V>(kph, 0, wx));
                if (wy)
                    ph = cmulf(ph, phase_pow<V>(kph, 1, wy));
            } else {
                const int wz = t - 81 - 4;
                ph = wz ? phase_pow<V>(kph, 2, wz) : cmk<V>(1.0, 0.0);
            }
            sPh[t] = ph;
        }
    if (proj)
        for (int t = tid; t < (z1 - z0) * TY; t += nthr) {
            const int zz = z0 + t / TY, r = t % TY;
            int2 ri = make_int2(0xffff, 0);
            if (r < rows) {
                const int4 g = gld(a.rowinfo + zz * ny + y0 + r);
                if (g.x <= g.y)
                    ri = make_int2(g.x | (g.y - g.x) << 16, g.z - g.x);
            }
            sRow[t] = ri;
        }

    // ---- halo of the padded plane: 8 rows of nx and 8 columns of the
    // tile's rows (the star never reads the corners).  Both buffers start
    // zeroed, which holds every entry outside a zero-boundary axis for all
    // planes.  The in-grid (or wrapped) halo rows are loaded per plane; the
    // wrapped columns of a periodic x axis are copies of the tile's own
    // values, written by the threads that hold them, or loaded where a row
    // is shorter than both halves of the halo.  Loaded entry d goes to this
    // thread when d = tid + i * nthr, i < HM.  hof: byte offset within a
    // plane; hpk: LDS slot | phase id << 20 (id 40: no wrap) ----
    for (int t = tid; t < 2 * plane; t += nthr)
        buf0[t] = czero<V>();
    const bool xcopy = perx && nx >= 2 * kHalf;
    const int u0 = pery ? 0 : max(0, kHalf - y0);   // first dynamic top row
    const int nup = kHalf - u0;
    const int nlow = pery ? kHalf : max(0, min(kHalf, ny - (y0 + rows)));
    const int ndy = (nup + nlow) * nx;
    const int ndyn = ndy + (perx && !xcopy ? rows * 2 * kHalf : 0);
    unsigned hof[HM];
    int hpk[HM];
#pragma unroll
    for (int i = 0; i < HM; ++i) {
        const int d = tid + i * nthr;
        hof[i] = kBufNone;
        hpk[i] = 40 << 20;
        if (d >= ndyn)
            continue;
        int r, xs, slot;
        if (d < ndy) {
            const int q = d / nx, hx = d - q * nx;
            r = q < nup ? u0 + q : rows + kHalf + (q - nup);
            xs = hx;
            slot = r * RS + hx + kHalf;
        } else {
            const int d2 = d - ndy;
            const int cc = d2 % (2 * kHalf);
            r = kHalf + d2 / (2 * kHalf);
            xs = cc < kHalf ? cc - kHalf : nx + cc - kHalf;
            slot = r * RS + (cc < kHalf ? cc : nx + cc);
        }
        int ys = y0 - kHalf + r;
        int wy = 0, wx = 0;
        if (ys < 0 || ys >= ny) {
            wy = floordiv(ys, ny);
            ys -= wy * ny;
        }
        if (xs < 0 || xs >= nx) {
            wx = floordiv(xs, nx);
            xs -= wx * nx;
        }
        hof[i] = (unsigned)(ys * nx + xs) * (unsigned)sizeof(InT);
        hpk[i] = slot | (((wy + 4) * 9 + wx + 4) << 20);
    }
    auto halo_ld = [&](int i, int zq) -> V {
        const bool ok = zq < z1;
        return bld<R, InT>(buf_any(in, ok), hof[i],
                           (ok ? zq * P : 0) * (int)sizeof(InT));
    };
    using VV = typename std::conditional<V32, float, double>::type;
    auto v_ld = [&](int r, int zq) -> VV {
        const bool ok = zq >= z0 && zq < z1;
        const BufRes rv = buf_any(vptr, ok);
        const int so = (ok ? zq * P : 0) * (int)VB;
        if constexpr (V32)
            return __builtin_bit_cast(
                float,
                __builtin_amdgcn_raw_buffer_load_b32(rv, p4[r], so, 0));
        else
            return bld_d(rv, p8[r], so);
    };
    auto kb_ld = [&](int r, int zq) -> V {
        unsigned off = kBufNone;
        if (proj && zq >= z0 && zq < z1) {
            // (an item of one row per thread in a launch of two has no
            // second row: past the tile, in its last plane past the table)
            const int2 ri =
                sRow[(zq - z0) * TY + row0 + min(r, rpt - 1)];
            const unsigned d = (unsigned)x - (unsigned)(ri.x & 0xffff);
            if (valid[r] && d <= (unsigned)ri.x >> 16)
                off = (unsigned)(ri.y + x) * (unsigned)sizeof(V);
        }
        return bld_nt<R, V>(rw, off, 0);
    };
    // own values and halo of one plane into an LDS buffer
    auto put_own = [&](V *buf) {
        const int rs = COL64 ? RS : fresh(RS);
#pragma unroll
        for (int r = 0; r < RPT; ++r)
            if (valid[r])
                buf[own + r * rs] = c[r];
        if (xcopy && (x < kHalf || x >= nx - kHalf)) {
            // wrap by +1 (phase 41) to the right of the row, by -1 (39) to
            // its left
            const int w = COL64 ? nx : fresh(nx);
            const bool left = x < kHalf;
            const V ph = sPh[left ? 41 : 39];
            V *d = buf + own + (left ? w : -w);
#pragma unroll
            for (int r = 0; r < RPT; ++r)
                if (valid[r])
                    d[r * rs] = cmulf(c[r], ph);
        }
    };
    auto put_halo = [&](V *buf, int i, V v) {
        const int o = COL64 ? 0 : fresh(0);
        if (hof[i] != kBufNone) {
            const int pid = hpk[i] >> 20;
            if (pid != 40)
                v = cmulf(v, sPh[pid + o]);
            buf[(hpk[i] & 0xfffff) + o] = v;
        }
    };

    // ---- plane z0: halo, potential, KB term; with two planes of lead also
    // plane z0 + 1 ----
    constexpr int PF = !F64 || (SC && RPT == 1) ? 2 : 1;
    constexpr int NS = SC ? PF : 2 * PF;   // sets of potential and KB term
    // plane of the own rows loaded for plane zq of the column (-1: none)
    auto ahead = [&](int zq) -> int {
        return zq < z1 + (CUR ? 0 : 4) ? wrap_z(zq) : -1;
    };
    V shv[PF][HM], snq[PF][RPT], skb[NS][RPT];
    VV sv[NS][RPT];
    {
        V hv0[HM];
#pragma unroll
        for (int i = 0; i < HM; ++i)
            hv0[i] = halo_ld(i, z0);
        __syncthreads();   // zeroed buffers, phase tables, hull rows ready
        if constexpr (!SC) {
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                sv[0][r] = v_ld(r, z0);
                skb[0][r] = kb_ld(r, z0);
#pragma unroll
                for (int m = 0; m <= 8; ++m)
                    q[r][m] = own_fix(q[r][m], z0 - 4 + m);
                c[r] = q[r][4];
            }
        }
        if constexpr (PF == 2) {
#pragma unroll
            for (int i = 0; i < HM; ++i)
                shv[1][i] = halo_ld(i, z0 + 1);
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                snq[1][r] = own_ld(r, SC ? wrap_z(z0 + 1) : ahead(z0 + 5));
                if constexpr (SC) {   // no output is complete before z0 + 4
                    sv[1][r] = 0;
                    skb[1][r] = czero<V>();
                } else {
                    sv[1][r] = v_ld(r, z0 + 1);
                    skb[1][r] = kb_ld(r, z0 + 1);
                }
            }
        }
        put_own(buf0);
#pragma unroll
        for (int i = 0; i < HM; ++i)
            put_halo(buf0, i, hv0[i]);
        if constexpr (SC)
#pragma unroll
            for (int r = 0; r < RPT; ++r)
#pragma unroll
                for (int m = 1; m <= 4; ++m)
                    p[r][4 - m] = own_fix(p[r][4 - m], z0 - m);
    }

    // ---- coefficients, uniform over the workgroup.  FP64: CL[axis][m] =
    // -c_m / (2 h^2) (from the host, with c0 the centre), CG[axis][m] =
    // A d_m / h (or d_m / h in mode kCurrent).  FP32: the weights and, apart,
    // 1 / h^2 and A / h ----
    R CL[3][5], CG[3][5];
    R LC[5], GD[5];
#pragma unroll
    for (int m = 1; m <= 4; ++m) {
        if constexpr (F64) {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                CL[ax][m] = a.cl[ax][m - 1];
                const double A =
                    ax == 0 ? Avec.x : (ax == 1 ? Avec.y : Avec.z);
                CG[ax][m] = uni((R)((CUR ? 1.0 : A) * a.cg[ax][m - 1]));
            }
        } else {
            LC[m] = (R)kLap[m];
            GD[m] = (R)kGrad[m];
        }
    }
    const R c0 = F64 ? (R)a.c0 : (R)0;
    const R ih2x = (R)(1.0 / (a.geo.h[0] * a.geo.h[0]));
    const R ih2y = (R)(1.0 / (a.geo.h[1] * a.geo.h[1]));
    const R ih2z = (R)(1.0 / (a.geo.h[2] * a.geo.h[2]));
    const R c0sum = (R)kLap[0] * (ih2x + ih2y + ih2z);
    const R Ax = (R)(Avec.x / a.geo.h[0]), Ay = (R)(Avec.y / a.geo.h[1]),
            Az = (R)(Avec.z / a.geo.h[2]);
    const R sc = uni((R)a.cim);
    const double w_occ = FIN ? gp(a.wocc)[sg] : 0.0;
    double nrm = 0.0;
    double jc[3] = {0.0, 0.0, 0.0};   // kCurrent: Im(conj psi [H, r_a] psi)
    // pending outputs of planes z-1 .. z-4 (slots as p)
    V o[RPT][4];
#pragma unroll
    for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int m = 0; m < 4; ++m)
            o[r][m] = czero<V>();

    auto plane_step = [&](auto Pc, const int z) {
        constexpr int PH = decltype(Pc)::value;    // (z - z0) % 4
        constexpr int LS = PF == 2 ? PH & 1 : 0;   // set loaded now
        constexpr int CS = PF == 2 ? 1 - (PH & 1) : 0;   // set of plane z+1
        const V *cur = (PH & 1) == 0 ? buf0 : buf1;
        V *nxt = (PH & 1) == 0 ? buf1 : buf0;
        constexpr int LV = SC ? LS : (PH + PF) & (NS - 1);
        constexpr int UV = SC ? CS : PH & (NS - 1);
        const int zo = SC ? z - 4 : z;             // output plane completed
        const bool emit = zo >= z0;
        const int so = (emit ? zo : 0) * P;
        // the final pass's other inputs at plane zo, then plane z + PF
        double2 fb[RPT];
        TT f1[RPT], f2[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            if constexpr (FIN) {
                const unsigned ot = off_of(r, sizeof(TT));
                fb[r] = bld_raw_nt<double2>(buf_any(a.base + sN, emit),
                                            p16[r], so * 16);
                f1[r] = bld_raw_nt<TT>(
                    buf_any(reinterpret_cast<const TT *>(a.t1) + sN, emit),
                    ot, so * (int)sizeof(TT));
                f2[r] = bld_raw_nt<TT>(
                    buf_any(reinterpret_cast<const TT *>(a.t2) + sN, emit),
                    ot, so * (int)sizeof(TT));
            }
        }
#pragma unroll
        for (int i = 0; i < HM; ++i)
            shv[LS][i] = halo_ld(i, z + PF);
        const int zn = ahead(SC ? z + PF : z + 4 + PF);
        // FP64 uses them at the end of the step that completes their plane
        const int zv = SC ? zo + PF - 1 : z + PF;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            snq[LS][r] = own_ld(r, zn);
            if constexpr (!CUR) {
                sv[LV][r] = v_ld(r, zv);
                skb[LV][r] = kb_ld(r, zv);
            }
        }
        // FP64: plane z's share of the pending outputs, their z+m taps
        V done[RPT], cdone[RPT];
        if constexpr (SC)
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
#pragma unroll
                for (int m = 1; m <= 4; ++m) {
                    V &t = o[r][(PH + 4 - m) & 3];
                    t = cfma(CL[2][m], c[r], t);
                    if constexpr (GRAD) {
                        t.x = rfma(CG[2][m], c[r].y, t.x);
                        t.y = rfma(-CG[2][m], c[r].x, t.y);
                    }
                }
                done[r] = o[r][PH];
                cdone[r] = p[r][PH];
            }
        if (z < z1) {
            __syncthreads();
            const int rs = COL64 ? RS : fresh(RS);
            const V *rp = cur + own;
            V yv[RPT + 8];        // y neighbours of all rows: rows -4 ..
#pragma unroll
            for (int j = 0; j <= 8; ++j)
                yv[j] = j == 4 ? c[0] : rp[(j - 4) * rs];
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                if (r > 0 && r >= rpt)
                    continue;
                if (r > 0)
                    yv[r + 8] = rp[(r + 4) * rs];
                const V *rx = rp + r * rs;
                const V cc = c[r];
                V sx = czero<V>(), sy = czero<V>(), sz = czero<V>();
                V g = czero<V>();
                if constexpr (CUR) {
                    // [H, r_a] has the taps -+d_m / h_a - i A_a m d_m at
                    // displacement +-m h_a (the kinetic taps -c_m / (2 h^2)
                    // times m h, m c_m = 2 d_m for these weights); both ends
                    // of a pair of points give the same Im(conj psi [H, r_a]
                    // psi), so the lower neighbours count twice and the
                    // upper ones are not read
                    auto axis = [&](auto Ax, double A, auto nb) {
                        constexpr int ax = decltype(Ax)::value;
                        V G = czero<V>(), U = czero<V>();
#pragma unroll
                        for (int m = 4; m >= 1; --m)
                            G = cfma(CG[ax][m], nb(m), G);
                        jc[ax] += act[r] ? 2.0 * (cc.x * G.y - cc.y * G.x)
                                         : 0.0;
                        if (A != 0.0) {
#pragma unroll
                            for (int m = 4; m >= 1; --m)
                                U = cfma(m * CG[ax][m], nb(m), U);
                            jc[ax] -= act[r] ? 2.0 * A * a.geo.h[ax] *
                                                   (cc.x * U.x + cc.y * U.y)
                                             : 0.0;
                        }
                    };
                    axis(std::integral_constant<int, 0>{}, Avec.x,
                         [&](int m) { return rx[-m]; });
                    axis(std::integral_constant<int, 1>{}, Avec.y,
                         [&](int m) { return rx[-m * rs]; });
                    axis(std::integral_constant<int, 2>{}, Avec.z,
                         [&](int m) { return p[r][(PH + 4 - m) & 3]; });
                    continue;
                }
                if constexpr (!F64) {
                    // the FP32 sums keep their order, and so their bits:
                    // pairs of taps, the weights apart from 1 / h^2
                    V gx = czero<V>(), gy = czero<V>(), gz = czero<V>();
#pragma unroll
                    for (int m = 1; m <= 4; ++m) {
                        const V xp = rx[m], xn = rx[-m];
                        const V yp = yv[r + 4 + m], yn = yv[r + 4 - m];
                        const V zp = q[r][4 + m], zn = q[r][4 - m];
                        sx = cfma(LC[m], cadd(xp, xn), sx);
                        sy = cfma(LC[m], cadd(yp, yn), sy);
                        sz = cfma(LC[m], cadd(zp, zn), sz);
                        if constexpr (GRAD == 1) {
                            gx = cfma(GD[m], csub(xp, xn), gx);
                            gy = cfma(GD[m], csub(yp, yn), gy);
                        }
                        if constexpr (GRAD)
                            gz = cfma(GD[m], csub(zp, zn), gz);
                    }
                    V lap = cfma(ih2x, sx, cscale(sy, ih2y));
                    lap = cfma(ih2z, sz, lap);
                    lap = cfma(c0sum, cc, lap);
                    const R vv = (R)((double)sv[UV][r] + Avec.w);
                    V hp = cfma(vv, cc, cscale(lap, (R)-0.5));
                    if constexpr (GRAD) {
                        // -i A.grad
                        V gr = cfma(Ax, gx, cscale(gy, Ay));
                        gr = cfma(Az, gz, gr);
                        hp.x += gr.y;
                        hp.y -= gr.x;
                    }
                    done[r] = cadd(hp, skb[UV][r]);
                    cdone[r] = cc;
                    continue;
                }
#pragma unroll
                for (int m = 4; m >= 1; --m) {
                    const V xn = rx[-m], xp = rx[m];
                    const V yn = yv[r + 4 - m], yp = yv[r + 4 + m];
                    const V zn = SC ? p[r][(PH + 4 - m) & 3] : q[r][4 - m];
                    sx = cfma(CL[0][m], xn, sx);
                    sy = cfma(CL[1][m], yn, sy);
                    sz = cfma(CL[2][m], zn, sz);
                    sx = cfma(CL[0][m], xp, sx);
                    sy = cfma(CL[1][m], yp, sy);
                    if constexpr (GRAD == 1) {
                        g = cfma(CG[0][m], xp, g);
                        g = cfma(-CG[0][m], xn, g);
                        g = cfma(CG[1][m], yp, g);
                        g = cfma(-CG[1][m], yn, g);
                    }
                }
                V h = cadd(cadd(sx, sy), sz);
                h = cfma(c0, cc, h);
                if constexpr (GRAD) {
                    // -i A.grad
#pragma unroll
                    for (int m = 4; m >= 1; --m)
                        g = cfma(-CG[2][m],
                                 SC ? p[r][(PH + 4 - m) & 3] : q[r][4 - m], g);
                    h.x += g.y;
                    h.y -= g.x;
                }
                if constexpr (!SC) {
                    // the upper z taps from the column, in the order in which
                    // the split star adds them
#pragma unroll
                    for (int m = 1; m <= 4; ++m) {
                        const V zp = q[r][4 + m];
                        h = cfma(CL[2][m], zp, h);
                        if constexpr (GRAD) {
                            h.x = rfma(CG[2][m], zp.y, h.x);
                            h.y = rfma(-CG[2][m], zp.x, h.y);
                        }
                    }
                    done[r] = h;
                    cdone[r] = cc;
                    continue;
                }
                o[r][PH] = h;
            }
        }
        // output of plane zo
        if constexpr (!CUR) {
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const BufRes rout = buf_any(out + so, emit && !ENE);
                const unsigned off = off_of(r, sizeof(OutT));
                // FP64: potential and KB term of the finished point
                V hp = done[r];
                if constexpr (F64)
                    hp = cadd(cfma((R)(sv[UV][r] + Avec.w), cdone[r], hp),
                              skb[UV][r]);
                if constexpr (ENE) {
                    if (act[r] && emit)
                        nrm += cdone[r].x * hp.x + cdone[r].y * hp.y;
                } else if constexpr (MODE == kApply) {
                    bst<double2>(rout, off, (double)hp.x, (double)hp.y);
                } else if constexpr (MODE == kTerm) {
                    bst<TT>(rout, off, -sc * hp.y, sc * hp.x);
                } else {
                    const V t4 = cmk<V>(-sc * hp.y, sc * hp.x);
                    const V t3 = cdone[r];
                    const double2 bb = fb[r];
                    const TT u1 = f1[r], u2 = f2[r];
                    const double re = bb.x + (double)u1.x + (double)u2.x +
                                      (double)t3.x + (double)t4.x;
                    const double im = bb.y + (double)u1.y + (double)u2.y +
                                      (double)t3.y + (double)t4.y;
                    bst<double2>(rout, off, re, im);
                    double part;
                    if constexpr (MODE == kFinalPred) {
                        const double pr = bb.x + 2.0 * u1.x + 4.0 * u2.x +
                                          8.0 * t3.x + 16.0 * (double)t4.x;
                        const double pi = bb.y + 2.0 * u1.y + 4.0 * u2.y +
                                          8.0 * t3.y + 16.0 * (double)t4.y;
                        part = w_occ * abs2f(pr, pi);
                    } else {
                        const double sq = abs2f(re, im);
                        part = w_occ * sq;
                        if (act[r] && emit)
                            nrm += sq;
                    }
                    bst_d(buf_any(a.npart + sN + so, emit && a.npart),
                          p8[r], part);
                }
            }
        }
        // plane z + 1 into the other buffer (free: its last readers passed
        // this plane's barrier)
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            if constexpr (SC) {
                p[r][PH] = c[r];
                c[r] = z + 1 < zend ? own_fix(snq[CS][r], z + 1) : c[r];
            } else {
#pragma unroll
                for (int m = 0; m < 8; ++m)
                    q[r][m] = q[r][m + 1];
                q[r][8] = z + 5 < z1 + 4 ? own_fix(snq[CS][r], z + 5)
                                         : snq[CS][r];
                c[r] = q[r][4];
            }
        }
        if (z + 1 < z1) {
            put_own(nxt);
#pragma unroll
            for (int i = 0; i < HM; ++i)
                put_halo(nxt, i, shv[CS][i]);
        }
    };
    // planes z1 .. z1 + 3 only complete the last outputs
    for (int z = z0; z < zend; z += 4) {
        plane_step(std::integral_constant<int, 0>{}, z);
        if (z + 1 < zend)
            plane_step(std::integral_constant<int, 1>{}, z + 1);
        if (z + 2 < zend)
            plane_step(std::integral_constant<int, 2>{}, z + 2);
        if (z + 3 < zend)
            plane_step(std::integral_constant<int, 3>{}, z + 3);
    }
    if constexpr (MODE == kFinal || ENE) {
        if (!a.normpart)
            return;
        __syncthreads();
        double vals[1] = {nrm};
        block_sum<double, 1>(vals, reinterpret_cast<double *>(smem_raw));
        if (tid == 0)
            gp(a.normpart)[(size_t)sl * ntiles + tile] = vals[0];
    }
    if constexpr (CUR) {
        __syncthreads();
        block_sum<double, 3>(jc, reinterpret_cast<double *>(smem_raw));
        if (tid == 0)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
                gp(a.normpart)[((size_t)sl * ntiles + tile) * 3 + ax] =
                    jc[ax];
    }
}

// ---------------------------------------------------------------------------
// KB projectors.  p_j(r) = N_j P_j(r) rad(r) with the real solid harmonics
// P = (1; x, y, z; xy, yz, zx, x^2 - y^2, 3z^2 - r^2) and
// rad = exp(-r^2 / (2 sigma^2)) (1 - r^2 / rc^2)^2, evaluated here without
// N_j (which the coefficients carry).
// ---------------------------------------------------------------------------
// NP: the projectors formed, 4 (s and p) where no atom has more, or 9.
template <class R, int NP = kMaxProj>
__device__ __forceinline__ void proj_shape(double dx, double dy, double dz,
                                           double r2, double2 ar, int np,
                                           R p[NP])
{
    const double wv = 1.0 - r2 * ar.y;
    const R rad = (R)(exp(-r2 * ar.x) * wv * wv);
    const R X = (R)dx, Y = (R)dy, Z = (R)dz;
    p[0] = rad;
    p[1] = rad * X;
    p[2] = rad * Y;
    p[3] = rad * Z;
    if constexpr (NP > 4) {
        p[4] = rad * X * Y;
        p[5] = rad * Y * Z;
        p[6] = rad * Z * X;
        p[7] = rad * (X * X - Y * Y);
        p[8] = rad * ((R)3 * Z * Z - (X * X + Y * Y + Z * Z));
    }
    for (int j = np; j < NP; ++j)
        p[j] = 0;
}

// Stage 1 of the gather: S_j = sum_pt P_j(r) rad(r) exp(i k.T) in(pt) over
// chunks of kGatherChunk sphere points.  A workgroup takes one atom, one
// chunk and 4 * kGatherSPW states: wavefront w handles kGatherSPW states,
// each lane a point, so the projector shape is evaluated once per point and
// wavefront.
#ifndef KS_GATHER_CHUNK
#define KS_GATHER_CHUNK 512
#endif
#ifndef KS_GATHER_SPW
#define KS_GATHER_SPW 2
#endif
constexpr int kGatherChunk = KS_GATHER_CHUNK;
constexpr int kGatherSPW = KS_GATHER_SPW;   // states per wavefront
constexpr int kGatherStates = 4 * kGatherSPW;

template <class R, class InT, int NP>
__device__ __forceinline__ void gather_item(const GArgs &a, const int at,
                                            const int grp, const int ch)
{
    using V = typename Cplx<R>::T;
    constexpr int U = kGatherChunk / 64;      // points per lane
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s0 = grp * kGatherStates + wave * kGatherSPW;
    const int np = gp(a.pj.nproj)[at];
    const int npt = gp(a.pj.npts)[at];
    const long io = gp(a.pj.ioff)[at];
    const double4 ap = gld(a.pj.apos + at);
    const double2 ar = gld(a.pj.arad + at);
    const int nx = a.geo.nx, ny = a.geo.ny, nz = a.geo.nz;
    const double Lx = nx * a.geo.h[0], Ly = ny * a.geo.h[1],
                 Lz = nz * a.geo.h[2];
    const int p0 = ch * kGatherChunk;
    const int p1 = min(npt, p0 + kGatherChunk);
    // all loads of the chunk are issued before any is used: the point
    // tables first, then the states at those points
    int gi[U], pk[U], code[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int pt = p0 + lane + 64 * u;
        const bool ok = pt < p1;
        gi[u] = ok ? gp(a.pj.sidx)[io + pt] : -1;
        pk[u] = ok ? gp(a.pj.sxyz)[io + pt] : 0;
        code[u] = ok ? gp(a.pj.sshift)[io + pt] : 0;
    }
    V val[U][kGatherSPW];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < kGatherSPW; ++q) {
            const int sl = s0 + q;
            val[u][q] = (gi[u] >= 0 && sl < a.ns)
                            ? ldc_g<R>(reinterpret_cast<const InT *>(a.in) +
                                         (size_t)sl * a.geo.N, gi[u])
                            : czero<V>();
        }
    R acc[kGatherSPW][2 * NP];
#pragma unroll
    for (int q = 0; q < kGatherSPW; ++q)
#pragma unroll
        for (int j = 0; j < 2 * NP; ++j)
            acc[q][j] = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (gi[u] < 0)
            continue;
        const int ix = pk[u] & 0x3ff, iy = (pk[u] >> 10) & 0x3ff,
                  iz = pk[u] >> 20;
        const int tx = (int)(signed char)(code[u] & 0xff);
        const int ty = (int)(signed char)((code[u] >> 8) & 0xff);
        const int tz = (int)(signed char)((code[u] >> 16) & 0xff);
        const double dx = axis_coord(nx, a.geo.h[0], a.geo.per[0], ix) +
                          tx * Lx - ap.x;
        const double dy = axis_coord(ny, a.geo.h[1], a.geo.per[1], iy) +
                          ty * Ly - ap.y;
        const double dz = axis_coord(nz, a.geo.h[2], a.geo.per[2], iz) +
                          tz * Lz - ap.z;
        const double r2 = dx * dx + dy * dy + dz * dz;
        R p[NP];
        proj_shape<R, NP>(dx, dy, dz, r2, ar, np, p);
#pragma unroll
        for (int q = 0; q < kGatherSPW; ++q) {
            const int sl = s0 + q;
            if (sl >= a.ns)
                break;
            V v = val[u][q];
            if (code[u]) {
                const int kk = (a.sg0 + sl) / a.nstates;
                v = cmul(v, shift_phase<V>(a.kph + 3 * kk, code[u]));
            }
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                acc[q][2 * j] += p[j] * v.x;
                acc[q][2 * j + 1] += p[j] * v.y;
            }
        }
    }
    // sum over the 64 lanes by a transpose through LDS: column c of the
    // workgroup (wave, state, projector, re/im) gets the lanes' values as
    // rows; thread c then adds its column in lane order (deterministic)
    constexpr int kCols = 4 * kGatherSPW * 2 * NP;
    static_assert(kCols <= 256, "one thread of the workgroup per column");
    __shared__ R red[kCols][65];
    __syncthreads();               // the previous item's reads are done
#pragma unroll
    for (int q = 0; q < kGatherSPW; ++q)
#pragma unroll
        for (int j = 0; j < 2 * NP; ++j)
            red[(wave * kGatherSPW + q) * 2 * NP + j][lane] = acc[q][j];
    __syncthreads();
    const int c = threadIdx.x;
    if (c < kCols) {
        R sum = 0;
        for (int r = 0; r < 64; ++r)
            sum += red[c][r];
        const int w = c / (2 * NP * kGatherSPW);
        const int q = (c / (2 * NP)) % kGatherSPW;
        const int jj = c % (2 * NP);
        const int sl = grp * kGatherStates + w * kGatherSPW + q;
        if (sl < a.ns) {
            R *part = reinterpret_cast<R *>(a.Dpart) +
                      2 * ((((size_t)sl * a.pj.natoms + at) * a.nchunk + ch) *
                           kMaxProj);
            gp(part)[jj] = sum;    // (j, re/im) interleaved as in V
        }
    }
}

// Stage 2: D[s][a][j] = N_j^2 h^3 E_{a,l(j)} sum over chunks (in order).
template <class R>
__device__ __forceinline__ void gather_finalize_item(const GArgs &a,
                                                     const long i)
{
    using V = typename Cplx<R>::T;
    const long total = (long)a.ns * a.pj.natoms * kMaxProj;
    if (i >= total)
        return;
    const int j = (int)(i % kMaxProj);
    const long sa = i / kMaxProj;           // s * natoms + atom
    const int at = (int)(sa % a.pj.natoms);
    const int nch = (gp(a.pj.npts)[at] + kGatherChunk - 1) / kGatherChunk;
    const V *part = reinterpret_cast<const V *>(a.Dpart) +
                    (size_t)sa * a.nchunk * kMaxProj + j;
    R re = 0, im = 0, e = 0;
    if (j < gp(a.pj.nproj)[at]) {
        for (int c = 0; c < nch; ++c) {
            const V v = gld(part + (size_t)c * kMaxProj);
            re += v.x;
            im += v.y;
        }
        e = (R)gp(a.pj.EjN2)[at * kMaxProj + j];
    }
    gst(reinterpret_cast<V *>(a.D) + i, cmk<V>(e * re, e * im));
}

// Both stages for one atom and one state in one workgroup, for launches of
// few states, which the latency of a launch and of its dependent loads bounds:
// wavefront w takes the chunks w, w + W, .. of the sphere (W
// wavefronts), the chunk sums meet in LDS and the coefficients are written
// at once, without partials and a second launch.  The points, the lanes and
// the chunks are summed in the order of the two stages, so the bits are the
// same.  smem: W * sphere_row(NP) reduction rows, then nchunk * 2 * kMaxProj
// sums.
__host__ __device__ constexpr int sphere_row(int np) { return 2 * np * 65; }

template <class R, class InT, int NP>
__device__ __forceinline__ void gather_sphere_item(const GArgs &a,
                                                   const int at, const int sl,
                                                   R *smem)
{
    using V = typename Cplx<R>::T;
    constexpr int U = kGatherChunk / 64;      // points per lane
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = blockDim.x >> 6;
    R *red = smem + wave * sphere_row(NP);
    R *sums = smem + W * sphere_row(NP);
    const int np = gp(a.pj.nproj)[at];
    const int npt = gp(a.pj.npts)[at];
    const long io = gp(a.pj.ioff)[at];
    const double4 ap = gld(a.pj.apos + at);
    const double2 ar = gld(a.pj.arad + at);
    const int nx = a.geo.nx, ny = a.geo.ny, nz = a.geo.nz;
    const double Lx = nx * a.geo.h[0], Ly = ny * a.geo.h[1],
                 Lz = nz * a.geo.h[2];
    const int nch = (npt + kGatherChunk - 1) / kGatherChunk;
    const double2 *kph = a.kph + 3 * ((a.sg0 + sl) / a.nstates);
    const InT *in = reinterpret_cast<const InT *>(a.in) +
                    (size_t)sl * a.geo.N;
    for (int ch = wave; ch < nch; ch += W) {
        const int p0 = ch * kGatherChunk;
        const int p1 = min(npt, p0 + kGatherChunk);
        int gi[U], pk[U], code[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int pt = p0 + lane + 64 * u;
            const bool ok = pt < p1;
            gi[u] = ok ? gp(a.pj.sidx)[io + pt] : -1;
            pk[u] = ok ? gp(a.pj.sxyz)[io + pt] : 0;
            code[u] = ok ? gp(a.pj.sshift)[io + pt] : 0;
        }
        V val[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            val[u] = gi[u] >= 0 ? ldc_g<R>(in, gi[u]) : czero<V>();
        R acc[2 * NP];
#pragma unroll
        for (int j = 0; j < 2 * NP; ++j)
            acc[j] = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (gi[u] < 0)
                continue;
            const int ix = pk[u] & 0x3ff, iy = (pk[u] >> 10) & 0x3ff,
                      iz = pk[u] >> 20;
            const int tx = (int)(signed char)(code[u] & 0xff);
            const int ty = (int)(signed char)((code[u] >> 8) & 0xff);
            const int tz = (int)(signed char)((code[u] >> 16) & 0xff);
            const double dx = axis_coord(nx, a.geo.h[0], a.geo.per[0], ix) +
                              tx * Lx - ap.x;
            const double dy = axis_coord(ny, a.geo.h[1], a.geo.per[1], iy) +
                              ty * Ly - ap.y;
            const double dz = axis_coord(nz, a.geo.h[2], a.geo.per[2], iz) +
                              tz * Lz - ap.z;
            const double r2 = dx * dx + dy * dy + dz * dz;
            R p[NP];
            proj_shape<R, NP>(dx, dy, dz, r2, ar, np, p);
            V v = val[u];
            if (code[u])
                v = cmul(v, shift_phase<V>(kph, code[u]));
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                acc[2 * j] += p[j] * v.x;
                acc[2 * j + 1] += p[j] * v.y;
            }
        }
        // the lanes in order, through this wavefront's own LDS rows
#pragma unroll
        for (int j = 0; j < 2 * NP; ++j)
            red[j * 65 + lane] = acc[j];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < 2 * NP) {
            R sum = 0;
            for (int r = 0; r < 64; ++r)
                sum += red[lane * 65 + r];
            sums[ch * 2 * kMaxProj + lane] = sum;
        }
        // the rows are read before the next chunk's values go there
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    const int j = threadIdx.x;
    if (j < kMaxProj) {
        R re = 0, im = 0, e = 0;
        if (j < np) {
            for (int c = 0; c < nch; ++c) {
                re += sums[(2 * c) * kMaxProj + 2 * j];
                im += sums[(2 * c) * kMaxProj + 2 * j + 1];
            }
            e = (R)gp(a.pj.EjN2)[at * kMaxProj + j];
        }
        gst(reinterpret_cast<V *>(a.D) +
                ((size_t)sl * a.pj.natoms + at) * kMaxProj + j,
            cmk<V>(e * re, e * im));
    }
}

// V_NL in on the hull: W[s][h] = sum over atoms a whose sphere holds hull
// point h of sum_j P_j(r) rad(r) D[s][a][j] exp(-i k.T).  A workgroup takes
// a chunk of 64 hull points (one per lane) and kApplyWaves * SPW states
// (SPW per wavefront).  The wavefront walks the chunk's atoms in a uniform
// loop; for atom i every lane whose hull point lies in its sphere (the
// lane's next hull entry has slot i: entries are in atom order, so each
// lane still adds its terms in atom order, deterministically) adds the
// atom's term.  The projector values come from a per-grid table of the
// entries (evaluated once at creation), the coefficients of the atom and
// the wavefront's states through scalar loads (one address for the whole
// wavefront): no LDS staging, no barrier, no per-lane coefficient read.
// (Staging the coefficients in LDS and reading them per lane cost 23 %
// more at 128^3 x 256, 26 % more in the FP32 kernels.)
// States per wavefront: for launches of many states 8 in FP64 and 16 in
// FP32 (fewer hull-entry walks and table reads per state), 4 for few (more
// workgroups): 128^3 x 256 FP64 1.02 -> 0.92 ms with 8 (1.01 ms with 16),
// FP32 0.74 -> 0.68 ms with 16; 64^3 x 32 12.3 -> 16.6 us with 8.
#ifndef KS_APPLY_SPW_SMALL
#define KS_APPLY_SPW_SMALL 4
#endif
#ifndef KS_APPLY_SPW_LARGE
#define KS_APPLY_SPW_LARGE 8
#endif
#ifndef KS_APPLY_SPW_LARGE32
#define KS_APPLY_SPW_LARGE32 16
#endif
#ifndef KS_APPLY_LARGE_NS
#define KS_APPLY_LARGE_NS 128
#endif
#ifndef KS_APPLY_WAVES
#define KS_APPLY_WAVES 4
#endif
constexpr int kApplyWaves = KS_APPLY_WAVES;
constexpr int kApplyThreads = 64 * kApplyWaves;
// states per wavefront of a single-grid launch of ns states in FP64 or
// FP32 (the batched launch, whose jobs are small, takes the small count)
__host__ __device__ constexpr int apply_spw(int ns, bool fp32)
{
    return ns < KS_APPLY_LARGE_NS
               ? KS_APPLY_SPW_SMALL
               : (fp32 ? KS_APPLY_SPW_LARGE32 : KS_APPLY_SPW_LARGE);
}
// state groups of the apply for ns states at spw states per wavefront
__host__ __device__ constexpr int apply_groups(int ns, int spw)
{
    return (ns + kApplyWaves * spw - 1) / (kApplyWaves * spw);
}
template <class T> using kptr_t = __attribute__((address_space(4))) const T *;

template <class R, int SPW, int NP>
__device__ __forceinline__ void kbapply_item(const GArgs &a, const int chunk,
                                             const int grp)
{
    using V = typename Cplx<R>::T;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s0 = (grp * kApplyWaves + wave) * SPW;
    const int h = chunk * kHullChunk + lane;
    const bool valid = h < a.pj.nhull;
    int e = valid ? gp(a.pj.he_off)[h] : 0;
    const int e1 = valid ? gp(a.pj.he_off)[h + 1] : 0;
    const int c0 = __builtin_amdgcn_readfirstlane(gp(a.pj.hc_off)[chunk]);
    const int c1 =
        __builtin_amdgcn_readfirstlane(gp(a.pj.hc_off)[chunk + 1]);
    V acc[SPW];
#pragma unroll
    for (int q = 0; q < SPW; ++q)
        acc[q] = czero<V>();
    int slot = e < e1 ? gp(a.pj.he_slot)[e] : -1;
    const kptr_t<R> Dall = (kptr_t<R>)reinterpret_cast<const R *>(a.D);
    for (int i = 0; i < c1 - c0; ++i) {
        const int at =
            __builtin_amdgcn_readfirstlane(gp(a.pj.hc_atoms)[c0 + i]);
        if (slot != i)
            continue;
        const int code = gp(a.pj.he_code)[e];
        R p[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j)
            p[j] = (R)gp(a.pj.he_p)[(size_t)e * kMaxProj + j];
        // all NP projectors: past the atom's count both the coefficients
        // and the tabulated values are zero
#pragma unroll
        for (int q = 0; q < SPW; ++q) {
            const int sl = s0 + q;
            if (sl < a.ns) {
                const kptr_t<R> D =
                    Dall + 2 * ((size_t)sl * a.pj.natoms + at) * kMaxProj;
                R d[2 * NP];
#pragma unroll
                for (int j = 0; j < 2 * NP; ++j)
                    d[j] = D[j];
                V t = czero<V>();
#pragma unroll
                for (int j = 0; j < NP; ++j)
                    t = cadd(t, cscale(cmk<V>(d[2 * j], d[2 * j + 1]), p[j]));
                if (code) {
                    const int kk = (a.sg0 + sl) / a.nstates;
                    t = cmul(t, shift_phase<V>(a.kph + 3 * kk, code));
                }
                acc[q] = cadd(acc[q], t);
            }
        }
        ++e;
        slot = e < e1 ? gp(a.pj.he_slot)[e] : -1;
    }
    // W is read once, by the next H.psi pass, and is larger than the MALL:
    // non-temporal stores
    if (valid)
#pragma unroll
        for (int q = 0; q < SPW; ++q) {
            const int sl = s0 + q;
            if (sl < a.ns)
                st_stream(reinterpret_cast<V *>(a.W) +
                              (size_t)sl * a.pj.nhull + h,
                          acc[q].x, acc[q].y);
        }
}

}  // namespace ks
