// Projector, density, dipole, norm, kick, Gram and exchange kernels and
// their launchers.
#include "ks_device.h"

#include <algorithm>

namespace ks {

// NP: projectors per atom, 4 where every atom has s and p at most (half the
// sums, the reduction and the coefficients of the nine) or 9.
template <class R, class InT, int NP>
__global__ __launch_bounds__(256) void k_gather(GArgs a)
{
    gather_item<R, InT, NP>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The same work in the plane order of the work items: workgroup -> (state
// group, work item), consecutive work items (the chunks of one range of
// planes) of one state group on one XCD.  Used for launches large enough
// that the chunks of overlapping spheres would otherwise miss the L2.
template <class R, class InT, int NP>
__global__ __launch_bounds__(256) void k_gather_planes(GArgs a)
{
    const int L = xcd_remap(blockIdx.x, gridDim.x);
    const int grp = L / a.pj.ngpairs;
    const int *it = reinterpret_cast<const int *>(a.pj.gpairs) +
                    2 * (L - grp * a.pj.ngpairs);
    gather_item<R, InT, NP>(a, gp(it)[0], grp, gp(it)[1]);
}

template <class R>
__global__ __launch_bounds__(256) void k_gather_finalize(GArgs a)
{
    gather_finalize_item<R>(a, (long)blockIdx.x * blockDim.x + threadIdx.x);
}

extern __shared__ double smem_proj[];

// (768 threads: three FP64 wavefronts per SIMD without spills)
constexpr int kSphereWaves = 12;

template <class R, class InT, int NP>
__global__ __launch_bounds__(64 * kSphereWaves) void k_gather_sphere(GArgs a)
{
    gather_sphere_item<R, InT, NP>(a, blockIdx.x, blockIdx.y,
                               reinterpret_cast<R *>(smem_proj));
}

template <class R, int SPW, int NP>
__global__ __launch_bounds__(kApplyThreads) void k_kbapply(GArgs a)
{
    kbapply_item<R, SPW, NP>(a, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------
// density: rho(g) = sum over sources in fixed order (density partials or
// weighted |psi|^2); optional v = v_ion + v_x(rho); optional dipole partials
// ---------------------------------------------------------------------------
constexpr int kDensThreads = 256;
#ifndef KS_DENS_U
#define KS_DENS_U 8
#endif
#ifndef KS_DENS_NT
#define KS_DENS_NT 1
#endif

// block blk of the density launch of `a` (sbuf: 3 doubles per wavefront)
__device__ __forceinline__ void density_block(const DArgs &a, long blk,
                                              double *sbuf)
{
    const Geo G = a.geo;
    const long g = blk * kDensThreads + threadIdx.x;
    double rho = 0.0;
    if (g < G.N) {
        // sources in order; U loads issued before their adds (the
        // partials are read once: non-temporal)
        constexpr int U = KS_DENS_U;
        int s = 0;
        if (a.npart) {
            const double *p = a.npart + g;
            for (; s + U <= a.nsrc; s += U) {
                double v[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = KS_DENS_NT ? __builtin_nontemporal_load(
                                            gp(p + (size_t)(s + u) * G.N))
                                      : p[(size_t)(s + u) * G.N];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    rho += v[u];
            }
            for (; s < a.nsrc; ++s)
                rho += p[(size_t)s * G.N];
        } else {
            const double2 *p = a.psi + g;
            for (; s + U <= a.nsrc; s += U) {
                double2 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = p[(size_t)(s + u) * G.N];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    rho += a.wocc[s + u] * (v[u].x * v[u].x + v[u].y * v[u].y);
            }
            for (; s < a.nsrc; ++s) {
                const double2 v = p[(size_t)s * G.N];
                rho += a.wocc[s] * (v.x * v.x + v.y * v.y);
            }
        }
        if (a.rho)
            a.rho[g] = rho;
        if (a.vout) {
            double vx = a.xc ? -cbrt(3.0 * rho / M_PI) : 0.0;
            a.vout[g] = a.vion[g] + vx;
        }
    }
    if (a.dpart) {
        double d[3] = {0.0, 0.0, 0.0};
        if (g < G.N) {
            int x = (int)(g % G.nx);
            int y = (int)((g / G.nx) % G.ny);
            int z = (int)(g / ((long)G.nx * G.ny));
            d[0] = axis_coord(G.nx, G.h[0], G.per[0], x) * rho;
            d[1] = axis_coord(G.ny, G.h[1], G.per[1], y) * rho;
            d[2] = axis_coord(G.nz, G.h[2], G.per[2], z) * rho;
        }
        block_sum<double, 3>(d, sbuf);
        if (threadIdx.x == 0)
            for (int c = 0; c < 3; ++c)
                a.dpart[(size_t)blk * 3 + c] = d[c];
    }
}

__global__ __launch_bounds__(kDensThreads) void k_density(DArgs a)
{
    __shared__ double sbuf[(kDensThreads / 64) * 3];
    density_block(a, blockIdx.x, sbuf);
}

// The densities of several grids in one launch: launch block L is block
// L - off[j] of job j (off[j] <= L < off[j + 1]), each computed exactly as
// k_density computes it.
__global__ __launch_bounds__(kDensThreads) void k_density_batch(
    const DArgs *args, const int *off, int njobs, int total)
{
    __shared__ double sbuf[(kDensThreads / 64) * 3];
    for (int L = blockIdx.x; L < total; L += gridDim.x) {
        int j = 0;
        while (j + 1 < njobs && L >= off[j + 1])
            ++j;
        const DArgs a = args[j];
        density_block(a, L - off[j], sbuf);
        __syncthreads();   // sbuf is reused by the next block
    }
}

// sum of nblocks dipole partials in fixed order, times h^3; with a device
// step counter, into out[3 * (step + 1) ...]
__device__ __forceinline__ void dipole_finalize_job(const double *dpart,
                                                    int nblocks, double h3,
                                                    double *out,
                                                    const int *step,
                                                    double *sbuf)
{
    if (step)
        out += 3 * (*step + 1);
    double d[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x)
        for (int c = 0; c < 3; ++c)
            d[c] += dpart[(size_t)b * 3 + c];
    block_sum<double, 3>(d, sbuf);
    if (threadIdx.x == 0)
        for (int c = 0; c < 3; ++c)
            out[c] = h3 * d[c];
}

__global__ __launch_bounds__(256) void k_dipole_finalize(const double *dpart,
                                                         int nblocks,
                                                         double h3,
                                                         double *out,
                                                         const int *step)
{
    __shared__ double sbuf[4 * 3];
    dipole_finalize_job(dpart, nblocks, h3, out, step, sbuf);
}

// one workgroup per job
__global__ __launch_bounds__(256) void k_dipole_finalize_batch(
    const DipJob *jobs)
{
    __shared__ double sbuf[4 * 3];
    const DipJob J = jobs[blockIdx.x];
    dipole_finalize_job(J.dpart, J.nblocks, J.h3, J.out, J.step, sbuf);
}

// per-state partial sums of |psi|^2 over chunks of the grid
__global__ __launch_bounds__(256) void k_norm_partial(Geo G,
                                                      const double2 *psi,
                                                      int nchunks,
                                                      double *part)
{
    __shared__ double sbuf[4];
    const int s = blockIdx.y;
    const long chunk = (G.N + nchunks - 1) / nchunks;
    const long b = (long)blockIdx.x * chunk;
    const long e = min(G.N, b + chunk);
    const double2 *p = psi + (size_t)s * G.N;
    double acc[1] = {0.0};
    for (long g = b + threadIdx.x; g < e; g += blockDim.x) {
        double2 v = p[g];
        acc[0] += v.x * v.x + v.y * v.y;
    }
    block_sum<double, 1>(acc, sbuf);
    if (threadIdx.x == 0)
        part[(size_t)s * nchunks + blockIdx.x] = acc[0];
}

__device__ __forceinline__ void norm_finalize_state(const double *part,
                                                    int ns, int ntiles,
                                                    double h3, double *out,
                                                    const int *step, int s,
                                                    double *sbuf, int *flag)
{
    if (step)
        out += (size_t)ns * (*step + 1);
    double acc[1] = {0.0};
    for (int t = threadIdx.x; t < ntiles; t += blockDim.x)
        acc[0] += part[(size_t)s * ntiles + t];
    block_sum<double, 1>(acc, sbuf);
    if (threadIdx.x == 0) {
        const double v = h3 * acc[0];
        out[s] = v;
        // every writer stores the same value, so the order does not matter
        if (flag && !isfinite(v))
            *flag = 1;
    }
}

__global__ __launch_bounds__(64) void k_norm_finalize(const double *part,
                                                      int ntiles, double h3,
                                                      double *out,
                                                      const int *step)
{
    __shared__ double sbuf[1];
    norm_finalize_state(part, gridDim.x, ntiles, h3, out, step, blockIdx.x,
                        sbuf, nullptr);
}

// state blockIdx.x of job blockIdx.y
__global__ __launch_bounds__(64) void k_norm_finalize_batch(
    const NormJob *jobs)
{
    __shared__ double sbuf[1];
    const NormJob J = jobs[blockIdx.y];
    if ((int)blockIdx.x >= J.ns)
        return;
    norm_finalize_state(J.part, J.ns, J.ntiles, J.h3, J.out, J.step,
                        blockIdx.x, sbuf, J.flag);
}

// The norm partials of the tiles a grid's own H.psi launches take: a
// workgroup sums a tile with the threads, rows and planes in the order of the
// final pass (hpsi_item), so that partials and norms have the same bits
// whatever shape a batch runs.  One read of the states, after eight passes.
__global__ __launch_bounds__(512) void k_norm_tiles_batch(
    const NormTiles *jobs, int nblocks)
{
    __shared__ double sbuf[8];
    int j = 0;
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        while (b >= jobs[j + 1].first)
            ++j;
        const NormTiles J = jobs[j];
        const int ntiles = J.ntile_y * J.nzc;
        const int w = b - J.first;
        const int sl = w / ntiles, tile = w - sl * ntiles;
        const int zc = tile / J.ntile_y, y0 = (tile - zc * J.ntile_y) * J.TY;
        const int rpt = min(J.rpt, J.TY);
        const int rows = min(J.TY, J.ny - y0);
        const int x = threadIdx.x % J.nx, yl = threadIdx.x / J.nx;
        const int row0 = min(yl * rpt, J.TY - rpt);
        const long P = (long)J.nx * J.ny;
        const int z0 = zc * J.zchunk, z1 = min(J.nz, z0 + J.zchunk);
        double acc[1] = {0.0};
        if (yl < (J.TY + rpt - 1) / rpt) {
            // this thread's rows that no lower thread counts
            const int r0 = yl * rpt - row0, r1 = min(rpt, rows - row0);
            const double2 *p = J.psi + ((size_t)sl * J.nz + z0) * P +
                               (long)(y0 + row0) * J.nx + x;
#pragma unroll 4
            for (int z = z0; z < z1; ++z, p += P)
                for (int r = r0; r < r1; ++r) {
                    const double2 v = gld(p + r * J.nx);
                    acc[0] += abs2f(v.x, v.y);
                }
        }
        block_sum<double, 1>(acc, sbuf);
        if (threadIdx.x == 0)
            J.part[(size_t)sl * ntiles + tile] = acc[0];
        __syncthreads();
    }
}

// psi <- exp(i kappa z) psi
__global__ __launch_bounds__(256) void k_kick(Geo G, double2 *psi,
                                              double kappa)
{
    const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G.N)
        return;
    const int z = (int)(g / ((long)G.nx * G.ny));
    double s, c;
    sincos(kappa * axis_coord(G.nz, G.h[2], G.per[2], z), &s, &c);
    double2 *p = psi + (size_t)blockIdx.y * G.N + g;
    double2 v = *p;
    double2 o;
    o.x = v.x * c - v.y * s;
    o.y = v.x * s + v.y * c;
    *p = o;
}

// ---------------------------------------------------------------------------
// Gram matrix partials on the FP64 matrix cores: part[ks][k][i][j] = sum
// over the ks-th slice of the grid of conj(psi_ki) psi_kj for j >= i (the
// rest is its conjugate).  A workgroup (four wavefronts) owns a T x T tile of
// (i, j), ti <= tj (T = 64, or 32 for few states), as blocks of 16 x 16
// accumulated by v_mfma_f64_16x16x4f64 (D[16][16] += A[16][4] B[4][16], four
// grid points per instruction): Re G = Ar^T Ar + Ai^T Ai and Im G = Ar^T Ai -
// Ai^T Ar, with A the states' values at the points.  32 points of the tile's
// states are staged through LDS per round (coalesced rows of 512 bytes).
// A tile off the diagonal gives each wavefront a quarter; a tile on it has
// one set of states (half the loads and the LDS) and only the blocks on and
// above the diagonal, which every wavefront accumulates over its quarter of
// the points (10 of 16 blocks at T = 64); the four sums meet in LDS.
// The matrix pipe and the stage loads (one round in flight) bound it: 48^3, 4
// k x 64 states 408 + 71 us with every block computed, both copies of a
// diagonal tile staged and one thread per element of the 512 slices' sum, 281
// + 11 us so.
// Operand layout on gfx950: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; D[4 r + l / 16][l % 16] is element r of lane l's
// accumulator.
// ---------------------------------------------------------------------------
constexpr int kGK = 32;          // points per LDS stage

__device__ __forceinline__ void gram_block(double2 a, double2 b, gd4_t &re,
                                           gd4_t &im)
{
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.x, im, 0, 0, 0);
}

// the states st .. st + kGT - 1 at kGK points from g0 (zero past the ends)
template <int kGT>
__device__ __forceinline__ void gram_stage(double2 (&s)[kGT][kGK + 1],
                                           const double2 *pk, long N, int st,
                                           int ns, long g0, long ge)
{
#pragma unroll
    for (int u = 0; u < kGT / 8; ++u) {
        const int r = (threadIdx.x >> 5) + 8 * u, c = threadIdx.x & 31;
        const long g = g0 + c;
        s[r][c] = (st + r < ns && g < ge) ? pk[(size_t)(st + r) * N + g]
                                          : make_double2(0.0, 0.0);
    }
}

template <int kGT>
__global__ __launch_bounds__(256) void k_gram_partial(Geo G,
                                                      const double2 *psi,
                                                      int ns, int ksplit,
                                                      double2 *part)
{
    constexpr int B = kGT / 32;      // 16 x 16 blocks per wavefront side
    constexpr int D = kGT / 16;      // and per tile side
    constexpr int ND = D * (D + 1) / 2;
    __shared__ double2 sa[kGT][kGK + 1];
    __shared__ double2 sb[kGT][kGK + 1];
    const int ntile = (ns + kGT - 1) / kGT;
    // tile pair blockIdx.x of the upper triangle, row by row
    int ti = 0, rest = blockIdx.x;
    while (rest >= ntile - ti) {
        rest -= ntile - ti;
        ++ti;
    }
    const int tj = ti + rest;
    const int kk = blockIdx.y;
    const int ks = blockIdx.z;
    const long slice = (G.N + ksplit - 1) / ksplit;
    const long gb = ks * slice, ge = min(G.N, gb + slice);
    const double2 *pk = psi + (size_t)kk * ns * G.N;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    double2 *out = part + ((size_t)ks * gridDim.y + kk) * ns * ns;
    if (ti == tj) {
        gd4_t re[ND], im[ND];
#pragma unroll
        for (int b = 0; b < ND; ++b)
            re[b] = im[b] = gd4_t{0.0, 0.0, 0.0, 0.0};
        for (long g0 = gb; g0 < ge; g0 += kGK) {
            gram_stage<kGT>(sa, pk, G.N, ti * kGT, ns, g0, ge);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kGK / 16; ++q) {
                const int k4 = 8 * wave + 4 * q;
                double2 v[D];
#pragma unroll
                for (int u = 0; u < D; ++u)
                    v[u] = sa[16 * u + li][k4 + lk];
                int b = 0;
#pragma unroll
                for (int u = 0; u < D; ++u)
#pragma unroll
                    for (int w = u; w < D; ++w, ++b)
                        gram_block(v[u], v[w], re[b], im[b]);
            }
            __syncthreads();
        }
        // the wavefronts' sums in order; sb holds one block of each
        double2 *sum = &sb[0][0];
        int b = 0;
#pragma unroll
        for (int u = 0; u < D; ++u)
#pragma unroll
            for (int w = u; w < D; ++w, ++b) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    sum[wave * 256 + r * 64 + lane] =
                        make_double2(re[b][r], im[b][r]);
                __syncthreads();
                const int t = threadIdx.x;         // element r * 64 + lane
                double2 s = sum[t];
                for (int q = 1; q < 4; ++q) {
                    const double2 v = sum[q * 256 + t];
                    s.x += v.x;
                    s.y += v.y;
                }
                const int i = ti * kGT + 16 * u + 4 * (t >> 6) +
                              ((t & 63) >> 4);
                const int j = ti * kGT + 16 * w + (t & 15);
                if (i < ns && j < ns && i <= j)
                    out[(size_t)i * ns + j] = s;
                __syncthreads();
            }
        return;
    }
    const int r0 = (wave >> 1) * (kGT / 2), c0 = (wave & 1) * (kGT / 2);
    gd4_t re[B][B], im[B][B];
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
        for (int w = 0; w < B; ++w)
            re[u][w] = im[u][w] = gd4_t{0.0, 0.0, 0.0, 0.0};
    for (long g0 = gb; g0 < ge; g0 += kGK) {
        gram_stage<kGT>(sa, pk, G.N, ti * kGT, ns, g0, ge);
        gram_stage<kGT>(sb, pk, G.N, tj * kGT, ns, g0, ge);
        __syncthreads();
#pragma unroll
        for (int k4 = 0; k4 < kGK; k4 += 4) {
            double2 a[B], b[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                a[u] = sa[r0 + 16 * u + li][k4 + lk];
                b[u] = sb[c0 + 16 * u + li][k4 + lk];
            }
#pragma unroll
            for (int u = 0; u < B; ++u)
#pragma unroll
                for (int w = 0; w < B; ++w)
                    gram_block(a[u], b[w], re[u][w], im[u][w]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
        for (int w = 0; w < B; ++w)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = ti * kGT + r0 + 16 * u + 4 * r + lk;
                const int j = tj * kGT + c0 + 16 * w + li;
                if (i < ns && j < ns)
                    out[(size_t)i * ns + j] =
                        make_double2(re[u][w][r], im[u][w][r]);
            }
}

// G[k][i][j], j >= i, and its mirror: PARTS threads share the slices of an
// element (in order, then in order over the threads).
constexpr int kGfThreads = 256, kGramParts = 16;

template <int PARTS>
__global__ __launch_bounds__(kGfThreads) void k_gram_finalize(
    const double2 *part, int ns, long count, int ksplit, double h3,
    double2 *out)
{
    constexpr int kElems = kGfThreads / PARTS;
    __shared__ double2 s[PARTS][kElems];
    const int e = threadIdx.x % kElems, q = threadIdx.x / kElems;
    const long i = (long)blockIdx.x * kElems + e;
    const int row = (int)(i / ns % ns), col = (int)(i % ns);
    const bool on = i < count && row <= col;
    double2 a = make_double2(0.0, 0.0);
    const int per = (ksplit + PARTS - 1) / PARTS;
    if (on)
        for (int k = q * per; k < min(ksplit, (q + 1) * per); ++k) {
            const double2 v = part[(size_t)k * count + i];
            a.x += v.x;
            a.y += v.y;
        }
    if constexpr (PARTS > 1) {
        s[q][e] = a;
        __syncthreads();
    }
    if (q != 0 || !on)
        return;
    for (int p = 1; p < PARTS; ++p) {
        a.x += s[p][e].x;
        a.y += s[p][e].y;
    }
    a.x *= h3;
    a.y *= h3;
    out[i] = a;
    if (row < col)
        out[i + (long)(col - row) * ns - (col - row)] =
            make_double2(a.x, -a.y);
}

// partial sums of rho^(4/3) (exchange energy)
__global__ __launch_bounds__(256) void k_exchange_partial(Geo G,
                                                          const double *rho,
                                                          double *part)
{
    __shared__ double sbuf[4];
    const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
    double acc[1] = {0.0};
    if (g < G.N)
        acc[0] = pow(rho[g], 4.0 / 3.0);
    block_sum<double, 1>(acc, sbuf);
    if (threadIdx.x == 0)
        part[blockIdx.x] = acc[0];
}

int gather_chunks(int max_npts)
{
    return std::max(1, (max_npts + kGatherChunk - 1) / kGatherChunk);
}

int gather_chunk_points() { return kGatherChunk; }

// Gather launches of at least this many workgroups run in plane order
// (128^3 x 256 states, 64 atoms: 45k workgroups, 0.91 -> 0.83 ms; at 2.5k
// and 96 workgroups the plain order is 2-10 % faster).
constexpr long kGatherPlaneOrderMin = 8192;
// Launches of at most this many (atom, state, chunk) wavefronts give each atom
// and state one workgroup (k_gather_sphere).  Nine projectors: 24^3 x 4 states,
// 72 wavefronts, 8.7 + 4.4 us in two launches -> 8.6; 64^3 x 32, 2304, 13.1 +
// 5.3 -> 13.6 (FP32 13.3 + 5.1 -> 11.5); 48^3 x 64, 3072, 15.6 + 4.6 -> 18.6;
// 72x60x66 x 40, 3600, 16.1 + 5.3 -> 22.0.  Four projectors: 7.5, 11.5 (FP32
// 10.1), 13.7 us; by events, two launches against one: 60^3 x 12, 3348, 20.7
// and 21.0, 64^3 x 56, 4032, 22.0 and 21.2, 48^3 x 36, 5184, 24.3 and 27.3.
// (Nine projectors on spheres of 16 chunks, two rounds of the workgroup's
// wavefronts, still gain at 6144: 32.7 and 30.2.)
constexpr long kGatherSphereMax = 3072, kGatherSphereMax4 = 4096;

template <int NP>
static hipError_t go_gather(bool mixed, bool in_is_f64, const GArgs &a, int ns,
                         hipStream_t st)
{
    if (ns <= 0 || a.pj.natoms <= 0)
        return hipSuccess;
    GArgs b = a;
    b.ns = ns;
    // few (atom, state, chunk) wavefronts: one workgroup per atom and state
    // sums the whole sphere and needs no second launch
    const int W = std::min(a.nchunk, kSphereWaves);
    const size_t rs = mixed ? 4 : 8;
    const size_t lds = rs * ((size_t)W * sphere_row(NP) +
                             (size_t)a.nchunk * 2 * kMaxProj);
    if ((long)a.pj.natoms * ns * a.nchunk <=
            (NP <= 4 ? kGatherSphereMax4 : kGatherSphereMax) &&
        lds <= kLdsBudget && ns <= 65535) {
        dim3 grid(a.pj.natoms, ns), blk(64 * W);
        if (!mixed)
            hipLaunchKernelGGL((k_gather_sphere<double, double2, NP>), grid, blk,
                               lds, st, b);
        else if (in_is_f64)
            hipLaunchKernelGGL((k_gather_sphere<float, double2, NP>), grid, blk,
                               lds, st, b);
        else
            hipLaunchKernelGGL((k_gather_sphere<float, float2, NP>), grid, blk,
                               lds, st, b);
        return hipGetLastError();
    }
    const int ngrp = (ns + kGatherStates - 1) / kGatherStates;
    const long nblk = (long)a.pj.ngpairs * ngrp;
    dim3 blk(256);
    if (nblk >= kGatherPlaneOrderMin && nblk <= 0x7fffffffL) {
        dim3 grid((unsigned)nblk);
        if (!mixed)
            hipLaunchKernelGGL((k_gather_planes<double, double2, NP>), grid, blk,
                               0, st, b);
        else if (in_is_f64)
            hipLaunchKernelGGL((k_gather_planes<float, double2, NP>), grid, blk,
                               0, st, b);
        else
            hipLaunchKernelGGL((k_gather_planes<float, float2, NP>), grid, blk,
                               0, st, b);
    } else {
        dim3 grid(a.pj.natoms, ngrp, a.nchunk);
        if (!mixed)
            hipLaunchKernelGGL((k_gather<double, double2, NP>), grid, blk, 0, st,
                               b);
        else if (in_is_f64)
            hipLaunchKernelGGL((k_gather<float, double2, NP>), grid, blk, 0, st,
                               b);
        else
            hipLaunchKernelGGL((k_gather<float, float2, NP>), grid, blk, 0, st,
                               b);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const long total = (long)ns * a.pj.natoms * kMaxProj;
    dim3 g2((unsigned)((total + 255) / 256));
    if (!mixed)
        hipLaunchKernelGGL((k_gather_finalize<double>), g2, dim3(256), 0, st,
                           b);
    else
        hipLaunchKernelGGL((k_gather_finalize<float>), g2, dim3(256), 0, st,
                           b);
    return hipGetLastError();
}

template <int NP>
static hipError_t go_kbapply(bool mixed, const GArgs &a, int ns,
                             hipStream_t st)
{
    if (ns <= 0 || a.pj.natoms <= 0 || a.pj.nhull <= 0)
        return hipSuccess;
    GArgs b = a;
    b.ns = ns;
    const int spw = apply_spw(ns, mixed);
    dim3 grid(a.pj.nhchunk, apply_groups(ns, spw));
    constexpr int SL = KS_APPLY_SPW_LARGE, SS = KS_APPLY_SPW_SMALL,
                  SL32 = KS_APPLY_SPW_LARGE32;
    if (!mixed && spw == SL)
        hipLaunchKernelGGL((k_kbapply<double, SL, NP>), grid,
                           dim3(kApplyThreads), 0, st, b);
    else if (!mixed)
        hipLaunchKernelGGL((k_kbapply<double, SS, NP>), grid,
                           dim3(kApplyThreads), 0, st, b);
    else if (spw == SL32)
        hipLaunchKernelGGL((k_kbapply<float, SL32, NP>), grid,
                           dim3(kApplyThreads), 0, st, b);
    else
        hipLaunchKernelGGL((k_kbapply<float, SS, NP>), grid, dim3(kApplyThreads),
                           0, st, b);
    return hipGetLastError();
}

hipError_t launch_gather(bool mixed, bool in_is_f64, const GArgs &a, int ns,
                         hipStream_t st)
{
    return a.pj.npmax <= 4 ? go_gather<4>(mixed, in_is_f64, a, ns, st)
                           : go_gather<kMaxProj>(mixed, in_is_f64, a, ns, st);
}

hipError_t launch_kbapply(bool mixed, const GArgs &a, int ns, hipStream_t st)
{
    return a.pj.npmax <= 4 ? go_kbapply<4>(mixed, a, ns, st)
                           : go_kbapply<kMaxProj>(mixed, a, ns, st);
}

// he_p[e][j] = p_j (without N_j) of entry e's atom at its sphere point, by
// the gather's own evaluation (the same point image, the same shapes).
__global__ __launch_bounds__(256) void k_hull_table(ProjDev pj, Geo G,
                                                    const int2 *ent,
                                                    long nent, double *he_p)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nent)
        return;
    const int2 ai = ent[e];
    const int at = ai.x;
    const long ip = gp(pj.ioff)[at] + ai.y;
    const int pk = gp(pj.sxyz)[ip];
    const int code = gp(pj.sshift)[ip];
    const int ix = pk & 0x3ff, iy = (pk >> 10) & 0x3ff, iz = pk >> 20;
    const int tx = (int)(signed char)(code & 0xff);
    const int ty = (int)(signed char)((code >> 8) & 0xff);
    const int tz = (int)(signed char)((code >> 16) & 0xff);
    const double4 ap = gld(pj.apos + at);
    const double2 ar = gld(pj.arad + at);
    const double dx = axis_coord(G.nx, G.h[0], G.per[0], ix) +
                      tx * (G.nx * G.h[0]) - ap.x;
    const double dy = axis_coord(G.ny, G.h[1], G.per[1], iy) +
                      ty * (G.ny * G.h[1]) - ap.y;
    const double dz = axis_coord(G.nz, G.h[2], G.per[2], iz) +
                      tz * (G.nz * G.h[2]) - ap.z;
    double p[kMaxProj];
    proj_shape<double>(dx, dy, dz, dx * dx + dy * dy + dz * dz, ar,
                       gp(pj.nproj)[at], p);
#pragma unroll
    for (int j = 0; j < kMaxProj; ++j)
        he_p[e * kMaxProj + j] = p[j];
}

hipError_t launch_hull_table(const ProjDev &pj, const Geo &g,
                             const int2 *ent, long nent, double *he_p,
                             hipStream_t st)
{
    if (nent <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_hull_table, dim3((unsigned)((nent + 255) / 256)),
                       dim3(256), 0, st, pj, g, ent, nent, he_p);
    return hipGetLastError();
}

// out[g] = sum_j w[j] src[j][g], j = 0 .. h-1 in order (potential
// extrapolation of the CFM4 propagator).
struct VComb {
    const double *src[4];
    double w[4];
};

__global__ __launch_bounds__(256) void k_vcombine(long N, int h, VComb c,
                                                  double *out)
{
    const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= N)
        return;
    double s = 0.0;
    for (int j = 0; j < h; ++j)
        s += c.w[j] * c.src[j][g];
    out[g] = s;
}

hipError_t launch_vcombine(long N, int h, const double *const src[4],
                           const double w[4], double *out, hipStream_t st)
{
    if (h < 1 || h > 4)
        return hipErrorInvalidValue;
    VComb c;
    for (int j = 0; j < 4; ++j) {
        c.src[j] = j < h ? src[j] : nullptr;
        c.w[j] = j < h ? w[j] : 0.0;
    }
    hipLaunchKernelGGL(k_vcombine, dim3((unsigned)((N + 255) / 256)),
                       dim3(256), 0, st, N, h, c, out);
    return hipGetLastError();
}

int density_blocks(long N)
{
    return (int)((N + kDensThreads - 1) / kDensThreads);
}

hipError_t launch_density(const DArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_density, dim3(density_blocks(a.geo.N)),
                       dim3(kDensThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_density_batch(const DArgs *args, const int *blk_off,
                                int njobs, int nblocks, hipStream_t st)
{
    if (njobs <= 0 || nblocks <= 0)
        return hipSuccess;
    const int grid = std::min(nblocks, 1 << 22);
    hipLaunchKernelGGL(k_density_batch, dim3(grid), dim3(kDensThreads), 0, st,
                       args, blk_off, njobs, nblocks);
    return hipGetLastError();
}

hipError_t launch_dipole_finalize_batch(const DipJob *jobs, int njobs,
                                        hipStream_t st)
{
    if (njobs <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_dipole_finalize_batch, dim3(njobs), dim3(256), 0, st,
                       jobs);
    return hipGetLastError();
}

hipError_t launch_norm_finalize_batch(const NormJob *jobs, int njobs,
                                      int max_ns, hipStream_t st)
{
    if (njobs <= 0 || max_ns <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_norm_finalize_batch, dim3(max_ns, njobs), dim3(64), 0,
                       st, jobs);
    return hipGetLastError();
}

hipError_t launch_norm_tiles_batch(const NormTiles *jobs, int njobs,
                                   int nblocks, int nthr, hipStream_t st)
{
    if (njobs <= 0 || nblocks <= 0)
        return hipSuccess;
    // (2^22 workgroups of 512 threads at most)
    hipLaunchKernelGGL(k_norm_tiles_batch, dim3(std::min(nblocks, 1 << 22)),
                       dim3(nthr), 0, st, jobs, nblocks);
    return hipGetLastError();
}

hipError_t launch_dipole_finalize(const double *dpart, int nblocks,
                                  double h3, double *out, hipStream_t st,
                                  const int *step)
{
    hipLaunchKernelGGL(k_dipole_finalize, dim3(1), dim3(256), 0, st, dpart,
                       nblocks, h3, out, step);
    return hipGetLastError();
}

hipError_t launch_norm_partial(const Geo &g, const double2 *psi, int ns,
                               int nchunks, double *normpart, hipStream_t st)
{
    if (ns <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_norm_partial, dim3(nchunks, ns), dim3(256), 0, st, g,
                       psi, nchunks, normpart);
    return hipGetLastError();
}

hipError_t launch_norm_finalize(const double *normpart, int ns, int ntiles,
                                double h3, double *out, hipStream_t st,
                                const int *step)
{
    if (ns <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_norm_finalize, dim3(ns), dim3(64), 0, st, normpart,
                       ntiles, h3, out, step);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_to_f32(const double *in, float *out,
                                               long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = (float)in[i];
}

hipError_t launch_to_f32(const double *in, float *out, long n,
                         hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((n + 255) / 256)), dim3(256),
                       0, st, in, out, n);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_to_f32_batch(const F32Copy *copies,
                                                     const int *blk_off,
                                                     int ncopies)
{
    int j = 0;
    while (j + 1 < ncopies && (int)blockIdx.x >= blk_off[j + 1])
        ++j;
    const F32Copy c = copies[j];
    const long i = (long)(blockIdx.x - blk_off[j]) * blockDim.x + threadIdx.x;
    if (i < c.n)
        c.dst[i] = (float)c.src[i];
}

hipError_t launch_to_f32_batch(const F32Copy *copies, const int *blk_off,
                               int ncopies, int nblocks, hipStream_t st)
{
    if (ncopies <= 0 || nblocks <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_to_f32_batch, dim3((unsigned)nblocks), dim3(256), 0,
                       st, copies, blk_off, ncopies);
    return hipGetLastError();
}

hipError_t launch_kick(const Geo &g, double2 *psi, int ns, double kappa,
                       hipStream_t st)
{
    if (ns <= 0)
        return hipSuccess;
    dim3 grid((unsigned)((g.N + 255) / 256), ns);
    hipLaunchKernelGGL(k_kick, grid, dim3(256), 0, st, g, psi, kappa);
    return hipGetLastError();
}

hipError_t launch_gram(const Geo &g, const double2 *psi, int nk, int ns,
                       double2 *part, int ksplit, double2 *out,
                       hipStream_t st)
{
    const int T = gram_tile(ns);
    const int ntile = (ns + T - 1) / T;
    dim3 grid(ntile * (ntile + 1) / 2, nk, ksplit);
    if (T == 64)
        hipLaunchKernelGGL((k_gram_partial<64>), grid, dim3(256), 0, st, g,
                           psi, ns, ksplit, part);
    else
        hipLaunchKernelGGL((k_gram_partial<32>), grid, dim3(256), 0, st, g,
                           psi, ns, ksplit, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const long count = (long)nk * ns * ns;
    double h3 = g.h[0] * g.h[1] * g.h[2];
    // one thread per element where the slices are few, as they are for many
    // states: sixteen would idle there, and from 2^14 states on pass the 2^32
    // threads of a launch
    const int parts = ksplit >= kGramParts ? kGramParts : 1;
    const long blocks = (count * parts + kGfThreads - 1) / kGfThreads;
    if (parts > 1)
        hipLaunchKernelGGL(k_gram_finalize<kGramParts>, dim3((unsigned)blocks),
                           dim3(kGfThreads), 0, st, part, ns, count, ksplit,
                           h3, out);
    else
        hipLaunchKernelGGL(k_gram_finalize<1>, dim3((unsigned)blocks),
                           dim3(kGfThreads), 0, st, part, ns, count, ksplit,
                           h3, out);
    return hipGetLastError();
}

hipError_t launch_exchange_partial(const Geo &g, const double *rho,
                                   double *part, hipStream_t st)
{
    hipLaunchKernelGGL(k_exchange_partial, dim3(density_blocks(g.N)),
                       dim3(256), 0, st, g, rho, part);
    return hipGetLastError();
}

}  // namespace ks
