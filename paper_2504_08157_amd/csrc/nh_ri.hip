// gfx950 kernels of the RI-velocity diagnostic (paper, section on the RI
// velocity): the speed-weighted centre of each level, the mean tangential
// speed over open annuli (strips) around it, and the maximum of those means
// over strips and levels, with the maximum horizontal speed alongside.
//
// Every level is cut into nb contiguous chunks of lattice columns, one
// workgroup per (chunk, level): a reduction pass for the centre, then a
// histogram pass (strip sums and counts in LDS) for the means.  Partial
// results per workgroup are combined in a fixed order by small final
// kernels; only the LDS histogram additions are unordered.  Neighbouring
// threads take neighbouring columns and walk rows of the chunk, so that no index is
// divided per node, and a lane adds the nodes of one strip up in registers
// until the strip changes: neighbouring rows mostly share it.  (Summing the
// lanes of one strip across the wavefront before each LDS update was 2.8x
// slower than one LDS atomic per node: neighbouring lanes span about a dozen
// strips at the benchmark's resolution.)
#include "nh_internal.h"

namespace nh {

constexpr int kRiThreads = 256;

constexpr int kRiRows = 2;   // rows whose loads are in flight together

// sum over the workgroup: a butterfly per wave, the waves in order (every thread gets it)
__device__ __forceinline__ double ri_block_sum(double v, double *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < kRiThreads / 64; ++w) r += red[w];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double ri_block_max(double v, double *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int w = 1; w < kRiThreads / 64; ++w) r = fmax(r, red[w]);
    __syncthreads();
    return r;
}

// Groups of rows that a chunk is cut into.  Its tasks, a column of a group each,
// take the threads ceil(columns groups / threads) rounds of ceil(rows / groups) rows,
// and about one and a half rows' worth of start and end each; tried are the groups that
// fill 1 to 16 rounds.
static int ri_row_groups(int nx, int ny, int nb)
{
    const long nxy = (long)nx * ny, chunk = (nxy + nb - 1) / nb, nc = chunk < nx ? chunk : nx;
    const long nr = (chunk + nx - 1) / nx;
    double best = 1e300;
    long rg = 1;
    for (int k = 1; k <= 16; ++k) {
        long g = k * (long)kRiThreads / nc;
        g = g < 1 ? 1 : g > nr ? nr : g;
        const double t = (double)((nc * g + kRiThreads - 1) / kRiThreads) * ((double)((nr + g - 1) / g) + 1.5);
        if (t < best) {
            best = t;
            rg = g;
        }
    }
    return (int)rg;
}

// The columns of chunk b of a level: rows of nx consecutive columns from
// the chunk's first one, cut into p.rg groups of rows.  For each column of a
// group that is the thread's: begin(ix) with its x index, rows(i, iy, n) for n <= kRiRows
// rows (columns i, i + nx, ..., y indices iy, iy + 1, ...), end().
template <typename B, typename R, typename E>
__device__ __forceinline__ void ri_chunk(const RiParams &p, int b, B &&begin, R &&rows, E &&end)
{
    const long nxy = (long)p.nx * p.ny, chunk = (nxy + p.nb - 1) / p.nb;
    const long i0 = b * chunk, i1 = i0 + chunk < nxy ? i0 + chunk : nxy;
    if (i0 >= i1) return;
    const int nx = p.nx, ix0 = (int)(i0 % nx), iy0 = (int)(i0 / nx), nc = i1 - i0 < nx ? (int)(i1 - i0) : nx;
    const int nr = (int)((i1 - i0 + nx - 1) / nx), per = (nr + p.rg - 1) / p.rg;
    for (int task = threadIdx.x; task < nc * p.rg; task += kRiThreads) {
        const int g = task / nc, c = task - g * nc, r0 = g * per;
        int r1 = r0 + per < nr ? r0 + per : nr;
        // the last row may end before this column
        if (r1 == nr && i0 + (long)(nr - 1) * nx + c >= i1) --r1;
        if (r0 >= r1) continue;
        const int t = ix0 + c, wrap = t >= nx;
        begin(wrap ? t - nx : t);
        long i = i0 + (long)r0 * nx + c;
        int iy = iy0 + r0 + wrap;
        for (int r = r0; r < r1; r += kRiRows, i += (long)kRiRows * nx, iy += kRiRows)
            rows(i, iy, r1 - r < kRiRows ? r1 - r : kRiRows);
        end();
    }
}

// s0 = sum m |u|, s1 = sum m |u| x, s2 = sum m |u| y over chunk b of level k
// (m = m_x m_y, the level's 2D quadrature weight up to the level's factor).
// Bound: the three fields it reads (512 x 512 x 81 nodes: 93 us, 5.5 TB/s; 122 with
// an index divided for every node).
__global__ void __launch_bounds__(kRiThreads) ri_centroid_partial(RiParams p, const double *__restrict__ q,
                                                                   double *__restrict__ part)
{
    __shared__ double red[kRiThreads / 64];
    const int b = blockIdx.x, k = blockIdx.y;
    const long nxy = (long)p.nx * p.ny;
    const double *u = q + p.U + k * nxy, *v = q + 2 * p.U + k * nxy, *w = q + 3 * p.U + k * nxy;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, mx = 0.0, x = 0.0;
    ri_chunk(
        p, b,
        [&](int ix) {
            mx = p.mx[ix];
            x = p.x[ix];
        },
        [&](long i, int iy, int n) {
            double uu[kRiRows], vv[kRiRows], ww[kRiRows], my[kRiRows], y[kRiRows];
#pragma unroll
            for (int r = 0; r < kRiRows; ++r) {
                const int rr = r < n ? r : 0;
                const long j = i + (long)rr * p.nx;
                uu[r] = u[j];
                vv[r] = v[j];
                ww[r] = w[j];
                my[r] = p.my[iy + rr];
                y[r] = p.y[iy + rr];
            }
#pragma unroll
            for (int r = 0; r < kRiRows; ++r) {
                if (r >= n) continue;
                const double sp = sqrt(uu[r] * uu[r] + vv[r] * vv[r] + ww[r] * ww[r]) * (mx * my[r]);
                s0 += sp;
                s1 += sp * x;
                s2 += sp * y[r];
            }
        },
        [] {});
    s0 = ri_block_sum(s0, red);
    s1 = ri_block_sum(s1, red);
    s2 = ri_block_sum(s2, red);
    if (threadIdx.x == 0) {
        double *o = part + ((long)k * p.nb + b) * 3;
        o[0] = s0;
        o[1] = s1;
        o[2] = s2;
    }
}

// centre of level k = blockIdx.x from its nb partials (a level at rest: the
// domain midpoint)
__global__ void __launch_bounds__(kRiThreads) ri_centroid_final(RiParams p, const double *__restrict__ part,
                                                                 double *__restrict__ center)
{
    __shared__ double red[kRiThreads / 64];
    const int k = blockIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < p.nb; b += kRiThreads)
        for (int c = 0; c < 3; ++c) s[c] += part[((long)k * p.nb + b) * 3 + c];
    for (int c = 0; c < 3; ++c) s[c] = ri_block_sum(s[c], red);
    if (threadIdx.x == 0) {
        center[k] = s[0] > 0.0 ? s[1] / s[0] : p.xmid;
        center[p.nz + k] = s[0] > 0.0 ? s[2] / s[0] : p.ymid;
    }
}

// Strip of squared radius r2: the j with (j eps)^2 < r2 < ((j+1) eps)^2,
// edges and r2 rounded exactly as written (no fused multiply-add), or -1.
__device__ __forceinline__ double ri_edge2(int j, double eps)
{
    const double b = __dmul_rn((double)j, eps);
    return __dmul_rn(b, b);
}

// (s = sqrt(r2) and ie = 1 / eps give the first guess, the edges decide)
__device__ __forceinline__ int ri_strip(double r2, double s, double ie, double eps, int ns)
{
    if (!(r2 > 0.0) || !(r2 < ri_edge2(ns, eps))) return -1;
    const double g = s * ie;
    int j = g < (double)ns ? (int)g : ns - 1;
    if (j > ns - 1) j = ns - 1;
    while (j > 0 && !(ri_edge2(j, eps) < r2)) --j;
    while (j < ns - 1 && !(r2 < ri_edge2(j + 1, eps))) ++j;
    return (ri_edge2(j, eps) < r2 && r2 < ri_edge2(j + 1, eps)) ? j : -1;
}

// s = sqrt(r2) and y = 1 / s for the quotients by it: the hardware's first value of
// 1 / sqrt, one step of third order, and a residual correction of s; outside the
// middle of the exponent range by sqrt and a division
__device__ __forceinline__ void ri_root(double r2, double &s, double &y)
{
    if (!(r2 > 1e-290 && r2 < 1e290)) {
        s = sqrt(r2);
        y = 1.0 / s;
        return;
    }
    y = __builtin_amdgcn_rsq(r2);
    const double e = __builtin_fma(-(r2 * y), y, 1.0);
    y = __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
    s = r2 * y;
    s = __builtin_fma(__builtin_fma(-s, s, r2), 0.5 * y, s);
}

// c / s (y as above), corrected by its residual; an infinite c stays infinite
__device__ __forceinline__ double ri_quotient(double c, double s, double y)
{
    const double q = c * y;
    return isinf(q) ? q : __builtin_fma(__builtin_fma(-q, s, c), y, q);
}

// strip sums and counts of chunk b of level k, and its maximum horizontal
// speed.  The levels go from the last to the first: the centroid pass leaves the
// last ones in the Infinity Cache (10 us of a call).  Bound: FP64 arithmetic and
// the LDS additions.  512 x 512 x 81 nodes, 50 strips: 111 us (152 with a division and
// a root per node, divided indices and an LDS addition per node).
__global__ void __launch_bounds__(kRiThreads) ri_strip_partial(RiParams p, const double *__restrict__ q,
                                                                const double *__restrict__ center,
                                                                double *__restrict__ ssum, int *__restrict__ scnt,
                                                                double *__restrict__ umax)
{
    extern __shared__ double hist[];                 // [ns] sums, then [ns] counts
    __shared__ double red[kRiThreads / 64];
    int *hcnt = reinterpret_cast<int *>(hist + p.nstrips);
    const int b = blockIdx.x, k = p.nz - 1 - blockIdx.y, ns = p.nstrips;
    for (int j = threadIdx.x; j < ns; j += kRiThreads) {
        hist[j] = 0.0;
        hcnt[j] = 0;
    }
    __syncthreads();
    const long nxy = (long)p.nx * p.ny;
    const double *u = q + p.U + k * nxy, *v = q + 2 * p.U + k * nxy;
    const double xc = center[k], yc = center[p.nz + k], ie = 1.0 / p.eps;
    double um = 0.0, dx = 0.0, sum = 0.0;
    int cur = -1, cnt = 0;
    auto flush = [&]() {
        if (cur >= 0) {
            atomicAdd(&hist[cur], sum);
            atomicAdd(&hcnt[cur], cnt);
        }
    };
    ri_chunk(
        p, b,
        [&](int ix) { dx = __dsub_rn(p.x[ix], xc); },
        [&](long i, int iy, int n) {
            double uu[kRiRows], vv[kRiRows], y[kRiRows];
#pragma unroll
            for (int r = 0; r < kRiRows; ++r) {
                const int rr = r < n ? r : 0;
                const long j = i + (long)rr * p.nx;
                uu[r] = u[j];
                vv[r] = v[j];
                y[r] = p.y[iy + rr];
            }
#pragma unroll
            for (int r = 0; r < kRiRows; ++r) {
                if (r >= n) continue;
                const double ui = uu[r], vi = vv[r];
                um = fmax(um, ui * ui + vi * vi);   // the root of the largest at the end
                const double dy = __dsub_rn(y[r], yc);
                const double r2 = __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
                double s, y1;
                ri_root(r2, s, y1);
                const int j = ri_strip(r2, s, ie, p.eps, ns);
                if (j != cur) {
                    flush();
                    cur = j;
                    cnt = 0;
                    sum = 0.0;
                }
                if (j >= 0) {
                    // |u_h . e_theta|: the horizontal velocity less its radial part
                    sum += ri_quotient(fabs(vi * dx - ui * dy), s, y1);
                    ++cnt;
                }
            }
        },
        [&] {
            flush();
            cur = -1;
        });
    um = ri_block_max(um, red);   // ends with a barrier: the histogram is complete
    const long base = ((long)k * p.nb + b) * ns;
    for (int j = threadIdx.x; j < ns; j += kRiThreads) {
        ssum[base + j] = hist[j];
        scnt[base + j] = hcnt[j];
    }
    if (threadIdx.x == 0) umax[(long)k * p.nb + b] = sqrt(um);
}

// the largest mean of (value, strip) pairs, the first strip of equals (-1: none)
__device__ __forceinline__ void ri_better(double &v, long &at, double ov, long oat)
{
    if (oat >= 0 && (at < 0 || ov > v || (ov == v && oat < at))) {
        v = ov;
        at = oat;
    }
}

// over the workgroup; every thread gets the result
__device__ __forceinline__ void ri_block_best(double &v, long &at, double *rv, long *ra)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ri_better(v, at, __shfl_xor(v, o), __shfl_xor(at, o));
    if (threadIdx.x % 64 == 0) {
        rv[threadIdx.x / 64] = v;
        ra[threadIdx.x / 64] = at;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kRiThreads / 64; ++w) ri_better(v, at, rv[w], ra[w]);
}

// strip means of level k = blockIdx.x from its nb partials, the largest of
// them and the largest speed of the level into lev[3 k ..] (value, strip or -1,
// speed).  The partials of a strip are summed in parts by threads of their own
// (the parts then in order): 512 x 512 x 81 nodes, 50 strips: 13 us and 5 for the
// last kernel (27 and 18 with one thread per strip and one workgroup for the maxima).
__global__ void __launch_bounds__(kRiThreads) ri_strip_final(RiParams p, const double *__restrict__ ssum,
                                                              const int *__restrict__ scnt,
                                                              const double *__restrict__ umax,
                                                              double *__restrict__ ubar, int *__restrict__ count,
                                                              double *__restrict__ lev)
{
    __shared__ double ps[kRiThreads], rv[kRiThreads / 64];
    __shared__ int pc[kRiThreads];
    __shared__ long ra[kRiThreads / 64];
    const int k = blockIdx.x, ns = p.nstrips, t = threadIdx.x;
    const int parts = p.parts, w = ns < kRiThreads ? ns : kRiThreads;
    const int part = t / w, per = (p.nb + parts - 1) / parts;
    double best = -1.0;
    long at = -1;
    for (int j0 = 0; j0 < ns; j0 += w) {
        const int j = j0 + t % w;
        double s = 0.0;
        int c = 0;
        if (part < parts && j < ns) {
            const int b1 = (part + 1) * per < p.nb ? (part + 1) * per : p.nb;
#pragma unroll 4
            for (int b = part * per; b < b1; ++b) {
                s += ssum[((long)k * p.nb + b) * ns + j];
                c += scnt[((long)k * p.nb + b) * ns + j];
            }
        }
        ps[t] = s;
        pc[t] = c;
        __syncthreads();
        if (part == 0 && j < ns) {
            for (int o = 1; o < parts; ++o) {
                s += ps[o * w + t];
                c += pc[o * w + t];
            }
            const double m = c > 0 ? s / c : 0.0;
            ubar[(long)k * ns + j] = m;
            count[(long)k * ns + j] = c;
            if (c > 0 && m > best) {   // ascending strips: the first of equals stays
                best = m;
                at = j;
            }
        }
        __syncthreads();
    }
    double um = 0.0;
    for (int b = t; b < p.nb; b += kRiThreads) um = fmax(um, umax[(long)k * p.nb + b]);
    ri_block_best(best, at, rv, ra);
    um = ri_block_max(um, ps);
    if (t == 0) {
        lev[3 * k] = best;
        lev[3 * k + 1] = (double)at;
        lev[3 * k + 2] = um;
    }
}

// result = {u_RI, radius of its strip centre, height of its level, max
// horizontal speed}; the largest mean of a populated strip, the first in
// (level, strip) order on ties; {0, -1, -1, .} when no strip is populated
__global__ void __launch_bounds__(kRiThreads) ri_max_final(RiParams p, const double *__restrict__ lev,
                                                            const double *__restrict__ z, double *__restrict__ result)
{
    __shared__ double rv[kRiThreads / 64], red[kRiThreads / 64];
    __shared__ long ra[kRiThreads / 64];
    double best = -1.0, um = 0.0;
    long at = -1;
    for (int k = threadIdx.x; k < p.nz; k += kRiThreads) {
        const double j = lev[3 * k + 1];
        ri_better(best, at, lev[3 * k], j >= 0.0 ? (long)k * p.nstrips + (long)j : -1);
        um = fmax(um, lev[3 * k + 2]);
    }
    ri_block_best(best, at, rv, ra);
    um = ri_block_max(um, red);
    if (threadIdx.x == 0) {
        result[0] = at >= 0 ? best : 0.0;
        result[1] = at >= 0 ? ((double)(at % p.nstrips) + 0.5) * p.eps : -1.0;
        result[2] = at >= 0 ? z[at / p.nstrips] : -1.0;
        result[3] = um;
    }
}

size_t ri_lds_bytes(int nstrips) { return (size_t)nstrips * (sizeof(double) + sizeof(int)); }

hipError_t launch_ri(const RiParams &p0, const double *q, bool center_given, double *center, double *ubar,
                     int *count, double *result, const double *z, const RiWork &w, hipStream_t s)
{
    RiParams p = p0;
    p.rg = ri_row_groups(p.nx, p.ny, p.nb);
    // parts of a strip's sum: the threads there are, and no more than the additions that are
    // left to one thread after them
    p.parts = 1;
    while (p.parts * p.parts < p.nb && (p.parts + 1) * p.nstrips <= kRiThreads) ++p.parts;
    const dim3 grid(p.nb, p.nz), blk(kRiThreads);
    if (!center_given) {
        hipLaunchKernelGGL(ri_centroid_partial, grid, blk, 0, s, p, q, w.cpart);
        hipLaunchKernelGGL(ri_centroid_final, dim3(p.nz), blk, 0, s, p, w.cpart, center);
    }
    hipLaunchKernelGGL(ri_strip_partial, grid, blk, ri_lds_bytes(p.nstrips), s, p, q, (const double *)center,
                       w.ssum, w.scnt, w.umax);
    // the levels' results take the place of the centroid partials (3 n_z of 3 n_z nb)
    hipLaunchKernelGGL(ri_strip_final, dim3(p.nz), blk, 0, s, p, w.ssum, w.scnt, w.umax, ubar, count, w.cpart);
    hipLaunchKernelGGL(ri_max_final, dim3(1), blk, 0, s, p, (const double *)w.cpart, z, result);
    return hipGetLastError();
}

}  // namespace nh
