// gfx950 kernels and the host-driven Krylov loop of the 3D-IMEX split
// (paper, Sec. 2.3: IMEX with the linear fast-wave operator treated
// implicitly, ARK2, matrix-free GMRES).  Here the linear operator is taken
// over all three directions:
//   (L)_rho'   = - rho0 (d/dx u + d/dy v) - d/dz (rho0 w)
//   (L)_u      = - (1/rho0) dp'_L/dx,   (L)_v = - (1/rho0) dp'_L/dy
//   (L)_w      = - (1/rho0) dp'_L/dz - g rho'/rho0 - tau(z) w
//   (L)_theta' = - w dtheta0/dz,        p'_L = gamma p0 (rho'/rho0 + theta'/theta0),
// the vertical terms from the column-walking L_v kernel, the horizontal ones
// from the DSS'd x/y derivative stencils of the explicit path (a tiled pass
// with the x/y planes staged in LDS), the damping
// of w in the absorbing layer implicit (the Klemp form of an upper sponge).
// Each stage system (I - a L) x = b is one global system in 5U unknowns,
// solved by restarted GMRES with classical Gram-Schmidt (a second pass when
// the kept norm falls below 1e-2 of the vector's), its dot products reduced
// in a fixed order and its small Hessenberg problem solved on the device;
// optionally right-preconditioned by the column systems of the 1D split,
// solved directly (the preconditioned vectors are kept, as flexible GMRES does).
#include "nh_internal.h"
#include "nh_lanes.h"

#include <cmath>
#include <vector>

namespace nh {

// out[f] = a x[f] + c (L x)[f] at every node, all of L in one walk (out may
// not alias x); RES: out = b - that, and
// part[workgroup] = the sum of its squares.  Walls: u rows zero at x walls, v rows at y walls, w rows at
// the bottom and top.  A workgroup of 64 x 8 lattice columns walks a chunk
// of kz levels.  Per level it stages the planes of u, v and p'_L of its
// tile plus an N-wide x/y halo in LDS (two buffers, one barrier per level)
// for the x and y taps; each thread stages its own node, which it needs
// itself, and up to two of the halo.  The vertical part (L_v) comes from a
// (2N+1)-level window of rho0 w and p'_L of the thread's own column in
// registers, filled with the N levels below the chunk and the N levels above
// each level as the walk goes (taps outside the column see zero inputs), as in
// the column-walking L_v kernel.  The loads of a level, the window's lead level
// included, are issued one level ahead.  Bound: the LDS taps and the latency of a
// level (2 us with one workgroup on a CU), not memory: what counts is that two
// workgroups share a CU, so registers are held to 128 for N <= 4 (the y stencil
// row, one per wave, is in scalar registers; node offsets are 32 bits on uniform
// level bases), and that the chunks spread evenly over the CUs (l3_levels).
// 256 x 256 x 41 nodes, N = 4: 55 us (85 before), 41 at the rate of a copy; the
// residual form 96 us, where L and a combination with norms took 55 + 62.
constexpr int kL3TX = 64, kL3TY = 8;

// (lev and gz are h.lev and h.hv.gz passed again as restrict pointers so
// that their per-level values are read with scalar loads)
template <int N, bool RES>
__global__ void __launch_bounds__(kL3TX * kL3TY, N <= 4 ? 4 : 2) l3_tile_kernel(L3Params h, const double *__restrict__ x,
                                                                double *out, double a, double c,
                                                                const double *__restrict__ lev,
                                                                const double *__restrict__ gz, int kz,
                                                                const int *gate,
                                                                const double *__restrict__ b,
                                                                double *__restrict__ part)
{
    if (gate && *gate == 0) return;
    double norm2 = 0.0;
    constexpr int NC = 2 * N + 1, PX = kL3TX + 2 * N, PY = kL3TY + 2 * N, PS = PX * PY;
    constexpr int NT = kL3TX * kL3TY, NH = (PS - NT + NT - 1) / NT;   // NH: halo nodes per thread
    __shared__ double tile[2][3][PS];   // u, v, p'_L
    const long nxy = (long)h.nx * h.ny;
    const int nz = h.nz;
    const long U = nxy * nz;
    const int ntx = (h.nx + kL3TX - 1) / kL3TX, nty = (h.ny + kL3TY - 1) / kL3TY;
    const int t = xcd_block(blockIdx.x, gridDim.x);
    const int tt = t % (ntx * nty), kc = t / (ntx * nty);
    const int kb = kc * kz, ke = kb + kz < nz ? kb + kz : nz;
    const int tx = threadIdx.x % kL3TX, ty = __builtin_amdgcn_readfirstlane(threadIdx.x / kL3TX);
    const int x0 = (tt % ntx) * kL3TX, y0 = (tt / ntx) * kL3TY;
    const int ix = x0 + tx, iy = y0 + ty;
    const bool own = ix < h.nx && iy < h.ny;
    const unsigned col = own ? ix + iy * h.nx : 0;
    const double gamma = h.gamma, grav = h.hv.g;
    double cx[NC], cy[NC];
#pragma unroll
    for (int o = 0; o < NC; ++o) {
        cx[o] = h.gx[(long)(ix < h.nx ? ix : 0) * NC + o];
        cy[o] = h.gy[(long)(iy < h.ny ? iy : 0) * NC + o];   // one row of the lattice per wave
    }
    // the halo nodes: N rows below and above the tile, then N columns on each side
    unsigned sc[NH];
    int si[NH];   // place in the tile, -1: none
    bool sv[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        const int e = threadIdx.x + i * NT, f = e - 2 * N * PX;
        const int r = e / PX, g = f % (2 * N);
        const int px = f < 0 ? e % PX : g < N ? g : g + kL3TX, py = f < 0 ? (r < N ? r : r + kL3TY) : N + f / (2 * N);
        int jx = x0 - N + px, jy = y0 - N + py;
        bool ok = e < PS - NT;
        si[i] = ok ? py * PX + px : -1;
        if (jx < 0 || jx >= h.nx) {
            ok = ok && h.perx;
            jx = ((jx % h.nx) + h.nx) % h.nx;
        }
        if (jy < 0 || jy >= h.ny) {
            ok = ok && h.pery;
            jy = ((jy % h.ny) + h.ny) % h.ny;
        }
        sv[i] = ok;
        sc[i] = ok ? jx + jy * h.nx : 0;
    }
    // the thread's own node: beyond the lattice (a ragged tile) it is a halo node of its neighbours
    const bool inx = ix < h.nx || h.perx, iny = iy < h.ny || h.pery, okc = inx && iny;
    const unsigned cs = okc ? ix % h.nx + (iy % h.ny) * h.nx : 0;
    const int jo = (ty + N) * PX + tx + N;
    auto level = [&](int k) -> long { return (long)(k < ke ? k : ke - 1) * nxy; };
    // rho0 w and p'_L of the own column at level kk (zero outside the column)
    auto vert = [&](int kk, double r, double w, double th, double &va, double &vb) {
        const double *L = lev + (long)(kk < 0 ? 0 : kk < nz ? kk : nz - 1) * kLevW;
        const bool in = kk >= 0 && kk < nz;
        va = in ? L[0] * w : 0.0;
        vb = in ? gamma * L[2] * (r * L[7] + th * L[8]) : 0.0;
    };
    // the vertical window: slots o = 0 .. 2N hold levels k - N + o
    double ta[NC], tb[NC];
#pragma unroll
    for (int o = 0; o < 2 * N; ++o) {
        const int kk = kb - N + o;
        const long L = (long)(kk < 0 ? 0 : kk < nz ? kk : nz - 1) * nxy;
        vert(kk, (x + L)[col], (x + 3 * U + L)[col], (x + 4 * U + L)[col], ta[o], tb[o]);
    }
    // the next level's values: rho', u, v, theta' of the halo nodes; all fields of the
    // thread's node (rho', u, v, w, theta'); rho', w, theta' of its column at the
    // window's lead level (level + N)
    double sr[NH], su[NH], sv2[NH], st[NH], ox[5], oz[3];
    auto load = [&](int k) {
        const double *xl = x + level(k);
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            sr[i] = xl[sc[i]];
            su[i] = (xl + U)[sc[i]];
            sv2[i] = (xl + 2 * U)[sc[i]];
            st[i] = (xl + 4 * U)[sc[i]];
        }
#pragma unroll
        for (int f = 0; f < 5; ++f) ox[f] = (xl + f * U)[cs];
        const double *xz = x + (long)(k + N < nz ? k + N : nz - 1) * nxy;
        oz[0] = xz[col];
        oz[1] = (xz + 3 * U)[col];
        oz[2] = (xz + 4 * U)[col];
    };
    // (written into the loop itself, a level spills registers: 62 us for 57 at 256 x 256 x 41)
    auto step = [&](int k) {
        const double *Lv = lev + (long)k * kLevW;
        const double rho0 = Lv[0], p0 = Lv[2], dth0 = Lv[3], tau = Lv[4], irho0 = Lv[7], ith0 = Lv[8];
        const double gp = gamma * p0;
        double(*T)[PS] = tile[(k - kb) & 1];
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            if (si[i] >= 0) {
                T[0][si[i]] = sv[i] ? su[i] : 0.0;
                T[1][si[i]] = sv[i] ? sv2[i] : 0.0;
                T[2][si[i]] = sv[i] ? gp * (sr[i] * irho0 + st[i] * ith0) : 0.0;
            }
        }
        const double xr = ox[0], xu = ox[1], xv = ox[2], xw = ox[3], xt = ox[4];
        T[0][jo] = okc ? xu : 0.0;
        T[1][jo] = okc ? xv : 0.0;
        T[2][jo] = okc ? gp * (xr * irho0 + xt * ith0) : 0.0;
        vert(k + N, oz[0], oz[1], oz[2], ta[2 * N], tb[2 * N]);
        load(k + 1);
        // vertical part at level k
        const double *G = gz + (long)k * NC;
        double d_rw = 0.0, d_pl = 0.0;
#pragma unroll
        for (int o = 0; o < NC; ++o) {
            d_rw += G[o] * ta[o];
            d_pl += G[o] * tb[o];
        }
#pragma unroll
        for (int o = 0; o < 2 * N; ++o) {
            ta[o] = ta[o + 1];
            tb[o] = tb[o + 1];
        }
        __syncthreads();
        double dux = 0.0, dpx = 0.0, dvy = 0.0, dpy = 0.0;
#pragma unroll
        for (int o = 0; o < NC; ++o) {
            const int jx = (ty + N) * PX + tx + o, jy = (ty + o) * PX + tx + N;
            dux += cx[o] * T[0][jx];
            dpx += cx[o] * T[2][jx];
            dvy += cy[o] * T[1][jy];
            dpy += cy[o] * T[2][jy];
        }
        double Lr = -d_rw - rho0 * (dux + dvy);
        double Lu = -irho0 * dpx, Lvv = -irho0 * dpy;
        double Lw = -d_pl * irho0 - grav * xr * irho0 - tau * xw;
        const double Lt = -xw * dth0;
        if (!h.perx && (ix == 0 || ix == h.nx - 1)) Lu = 0.0;
        if (!h.pery && (iy == 0 || iy == h.ny - 1)) Lvv = 0.0;
        if (k == 0 || k == nz - 1) Lw = 0.0;
        if (own) {
            double *ol = out + (long)k * nxy;
            if constexpr (RES) {
                const double v[5] = {a * xr + c * Lr, a * xu + c * Lu, a * xv + c * Lvv, a * xw + c * Lw,
                                     a * xt + c * Lt};
                const double *bl = b + (long)k * nxy;
#pragma unroll
                for (int f = 0; f < 5; ++f) {
                    const double r = (bl + f * U)[col] - v[f];
                    norm2 += r * r;
                    (ol + f * U)[col] = r;
                }
            } else {
                ol[col] = a * xr + c * Lr;
                (ol + U)[col] = a * xu + c * Lu;
                (ol + 2 * U)[col] = a * xv + c * Lvv;
                (ol + 3 * U)[col] = a * xw + c * Lw;
                (ol + 4 * U)[col] = a * xt + c * Lt;
            }
        }
    };
    load(kb);
    for (int k = kb; k < ke; ++k) step(k);
    if constexpr (RES) {
        __shared__ double red[NT / 64];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) norm2 += __shfl_xor(norm2, o);
        if (tx == 0) red[ty] = norm2;
        __syncthreads();
        if (threadIdx.x == 0) {
            double r = 0.0;
            for (int w = 0; w < NT / 64; ++w) r += red[w];
            part[blockIdx.x] = r;
        }
    }
}

// Levels per chunk: a CU that gets r workgroups takes about (r + 0.4) times the
// levels of a chunk and 2.5 levels' worth of window fill and start (orders up to 4:
// two workgroups on a CU at a time; above, one: r times).  Measured on 256 x 256
// x 41 nodes, N = 4 (128 tiles), chunks of 41, 21, 16, 14, 11, 7, 5 levels: 96.3, 62.8, 65.5,
// 59.3, 55.1, 57.3, 69.6 us; on 384 x 384 x 65 (288 tiles), 65, 33, 22, 16, 13, 8: 326, 263,
// 248, 276, 240, 272 us; on 48 x 48 x 49 (6 tiles), 41, 16, 4: 85.8, 37.4, 14.3 us.  (Chunks
// of 16 levels in slots of two levels, one workgroup to a CU: 84.7, 330 and 36.6 us.)
static int l3_levels(int tiles, int nz, int N)
{
    double best = 1e300;
    int kz = nz;
    for (int c = 1; c <= nz; ++c) {
        const int k = (nz + c - 1) / c, r = (tiles * ((nz + k - 1) / k) + 255) / 256;
        const double t = (r + (N <= 4 ? 0.4 : 0.0)) * (k + 2.5);
        if (t < best) {
            best = t;
            kz = k;
        }
    }
    return kz;
}

int l3_max_blocks(int nx, int ny, int nz)
{
    return ((nx + kL3TX - 1) / kL3TX) * ((ny + kL3TY - 1) / kL3TY) * nz;
}

template <bool RES>
static hipError_t launch_l3_form(const L3Params &h, const double *x, double *out, double a, double c, hipStream_t s,
                                 const int *gate, const double *b, double *part, int *blocks)
{
    const int ntx = (h.nx + kL3TX - 1) / kL3TX, nty = (h.ny + kL3TY - 1) / kL3TY;
    const int kz = l3_levels(ntx * nty, h.nz, h.N), nkc = (h.nz + kz - 1) / kz;
    const dim3 grid((unsigned)(ntx * nty * nkc)), blk(kL3TX * kL3TY);
    if (blocks) *blocks = ntx * nty * nkc;
    switch (h.N) {
#define NH_L3(NN)                                                                                              \
    case NN:                                                                                                   \
        hipLaunchKernelGGL((l3_tile_kernel<NN, RES>), grid, blk, 0, s, h, x, out, a, c, h.lev, h.hv.gz, kz, gate, \
                           b, part);                                                                           \
        break;
        NH_L3(2) NH_L3(3) NH_L3(4) NH_L3(5) NH_L3(6)
#undef NH_L3
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_l3(const L3Params &h, const double *x, double *out, double a, double c, hipStream_t s,
                     const int *gate)
{
    return launch_l3_form<false>(h, x, out, a, c, s, gate, nullptr, nullptr, nullptr);
}

// ---- Krylov kernels on n-vectors.  Dot products are summed per block into
// quantity-major partials, then by one workgroup in a fixed order: the same
// result on every call.  The Hessenberg problem, the rotations and the
// convergence test live on the device (G3State), so the host queues the
// launches of a cycle ahead of their results; launches past the end of the
// process see their gate flag at 0 and return at once.
constexpr int kKryBlocks = 1024, kKryThreads = 256, kKryMaxV = 34, kKryCtl = 1024;

__device__ __forceinline__ double kry_wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// part[j][b] = sum over block b's elements of V_j . w (j < NV), and
// part[NV][b] = w . w.  All loads of an iteration are unconditional (the
// index of a lane past the end is clamped and its weight zeroed after the
// loads), so they are in flight together; for short bases each lane takes
// UF elements a grid stride apart, so that every CU still has enough bytes
// in flight to run at memory speed.
template <int NV>
__global__ void __launch_bounds__(kKryThreads) kry_dots_kernel(const double *__restrict__ V, long stride,
                                                               const double *__restrict__ w, long n,
                                                               double *__restrict__ part, const int *gate)
{
    constexpr int UF = NV <= 1 ? 4 : NV <= 3 ? 2 : 1;
    if (gate && *gate == 0) return;
    __shared__ double red[kKryThreads / 64][NV + 1];
    double acc[NV + 1];
#pragma unroll
    for (int j = 0; j <= NV; ++j) acc[j] = 0.0;
    const long S = (long)gridDim.x * kKryThreads;
    for (long i0 = blockIdx.x * (long)kKryThreads + threadIdx.x; i0 < n; i0 += S * UF) {
        long ii[UF];
        double wi[UF], vv[NV > 0 ? NV : 1][UF];
#pragma unroll
        for (int u = 0; u < UF; ++u) ii[u] = i0 + u * S < n ? i0 + u * S : n - 1;
#pragma unroll
        for (int u = 0; u < UF; ++u) wi[u] = w[ii[u]];
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int u = 0; u < UF; ++u) vv[j][u] = V[j * stride + ii[u]];
#pragma unroll
        for (int u = 1; u < UF; ++u)
            if (i0 + u * S >= n) wi[u] = 0.0;
#pragma unroll
        for (int u = 0; u < UF; ++u) {
            acc[NV] += wi[u] * wi[u];
#pragma unroll
            for (int j = 0; j < NV; ++j) acc[j] += vv[j][u] * wi[u];
        }
    }
    const int wv = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
    for (int j = 0; j <= NV; ++j) {
        const double s = kry_wave_sum(acc[j]);
        if (lane == 0) red[wv][j] = s;
    }
    __syncthreads();
    for (int j = threadIdx.x; j <= NV; j += kKryThreads) {
        double s = 0.0;
        for (int q = 0; q < kKryThreads / 64; ++q) s += red[q][j];
        part[(long)j * kKryBlocks + blockIdx.x] = s;
    }
}

template <int NV>
static void launch_dots(int nv, const double *V, long n, const double *x, double *part, const int *gate,
                        hipStream_t s)
{
    if constexpr (NV <= kG3MaxRestart) {
        if (nv == NV)
            hipLaunchKernelGGL(kry_dots_kernel<NV>, dim3(kKryBlocks), dim3(kKryThreads), 0, s, V, n, x, n, part,
                               gate);
        else
            launch_dots<NV + 1>(nv, V, n, x, part, gate, s);
    }
}

// (Each thread takes two elements 2 KB apart: 67 us on average over a 3D-IMEX step's
// launches, 71 with one.)
// y = s (w - sum_j c_j V_j) for j < nv, nv = *nvp when given, s = *sc when
// given (else 1), coefficients c in device memory.  y may alias w.
__global__ void __launch_bounds__(kKryThreads) kry_axpy_kernel(const double *__restrict__ V, long stride, int nv,
                                                               const int *nvp, const double *cf, const double *w,
                                                               double *y, long n, const double *sc, const int *gate)
{
    if (gate && *gate == 0) return;
    const int nvv = nvp ? *nvp : nv;
    const double s = sc ? *sc : 1.0;
    constexpr int UF = 2;
    for (long i0 = blockIdx.x * (long)(kKryThreads * UF) + threadIdx.x; i0 < n;
         i0 += (long)gridDim.x * (kKryThreads * UF)) {
        const bool two = i0 + kKryThreads < n;
        const long i1 = two ? i0 + kKryThreads : i0;
        double v0 = w[i0], v1 = w[i1];
#pragma unroll 4
        for (int j = 0; j < nvv; ++j) {
            v0 -= cf[j] * V[j * stride + i0];
            v1 -= cf[j] * V[j * stride + i1];
        }
        y[i0] = s * v0;
        if (two) y[i1] = s * v1;
    }
}

// The nq quantities of the block partials summed into out (LDS): wave v
// sums quantities v, v + 16, ..., each lane a fixed strided subset of the
// blocks, then a fixed butterfly.  Ends with a barrier.
__device__ void kry_reduce(const double *__restrict__ part, int nq, double *out)
{
    const int wv = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int q = wv; q < nq; q += kKryCtl / 64) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < kKryBlocks / 64; ++b) s += part[(long)q * kKryBlocks + b * 64 + lane];
        s = kry_wave_sum(s);
        if (lane == 0) out[q] = s;
    }
    __syncthreads();
}

__device__ void g3_publish(const G3State *st, G3Status *hs)
{
    volatile G3Status *v = hs;
    v->go = st->go;
    v->open = st->open;
    v->iters = st->iters;
    v->relres = st->relres;
    __threadfence_system();
}

// Start of a solve: ||b|| from the partials of b . b
__global__ void __launch_bounds__(kKryCtl) g3_begin_kernel(G3State *st, const double *__restrict__ part,
                                                           G3Status *hs)
{
    __shared__ double red[1];
    kry_reduce(part, 1, red);
    if (threadIdx.x != 0) return;
    const double bn = sqrt(red[0]);
    st->bn = bn;
    st->bzero = bn == 0.0;
    st->open = bn > 0.0;
    st->go = 0;
    st->pass2 = 0;
    st->ncols = 0;
    st->iters = 0;
    st->relres = 0.0;
    st->zero = 0.0;
    g3_publish(st, hs);
}

// Start of a cycle: beta = ||r|| from the nb partials of the residual; the solve
// ends when beta <= rtol ||b||, else (unless this is the final check) the
// Arnoldi process starts from V_0 = r / beta.  With a preconditioner, the only
// other reader of V_0, V_0 holds r and its users scale it by v0s = 1 / beta, which
// saves a pass over it.
__global__ void __launch_bounds__(kKryCtl) g3_cycle_kernel(G3State *st, const double *__restrict__ part, int nb,
                                                           double rtol, int final, int precond, G3Status *hs)
{
    if (st->open == 0) return;
    __shared__ double red[kKryCtl / 64];
    double r2 = 0.0;
    for (int i = threadIdx.x; i < nb; i += kKryCtl) r2 += part[i];
    r2 = kry_wave_sum(r2);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = r2;
    __syncthreads();
    if (threadIdx.x != 0) return;
    r2 = 0.0;
    for (int w = 0; w < kKryCtl / 64; ++w) r2 += red[w];
    const double beta = sqrt(r2), bn = st->bn;
    st->relres = beta / bn;
    st->ncols = 0;
    st->pass2 = 0;
    if (beta <= rtol * bn) {
        st->open = 0;
        st->go = 0;
    } else {
        st->go = final ? 0 : 1;
        st->scale = 1.0 / beta;
        st->v0s = precond ? st->scale : 1.0;
        st->gv[0] = beta;
        for (int i = 1; i <= kG3MaxRestart; ++i) st->gv[i] = 0.0;
    }
    g3_publish(st, hs);
}

// Column j of the Hessenberg matrix from the partials of V_i . w (i <= j) and
// w . w (pass 1) or of the second pass.  The norm of the kept part is
// ||w||^2 - sum h_i^2 when that keeps at least 1e-4 of ||w||^2 (the vector
// is then written normalised by the combination that orthogonalises it);
// otherwise a second pass orthogonalises the kept part again and its norm
// comes from that pass.  Then the earlier rotations, a new one, the rotated
// residual and the convergence test.
__global__ void __launch_bounds__(kKryCtl) g3_column_kernel(G3State *st, const double *__restrict__ part, int j,
                                                            int m, double rtol, int pass, G3Status *hs)
{
    if (pass == 1 ? st->go == 0 : st->pass2 == 0) return;
    __shared__ double red[kKryMaxV + 1];
    kry_reduce(part, j + 2, red);
    if (threadIdx.x != 0) return;
    red[0] *= st->v0s;
    double h2 = 0.0;
    for (int i = 0; i <= j; ++i) h2 += red[i] * red[i];
    const double w2 = red[j + 1];
    double k2 = w2 - h2;
    if (pass == 1) {
        for (int i = 0; i <= j; ++i) st->coef[i] = i == 0 ? red[0] * st->v0s : red[i];
        if (!(k2 >= 1e-4 * w2)) {   // second pass
            for (int i = 0; i <= j; ++i) st->hc[i] = red[i];
            st->pass2 = 1;
            st->scale = 1.0;
            return;
        }
        for (int i = 0; i <= j; ++i) st->hc[i] = red[i];
        st->pass2 = 0;
    } else {
        for (int i = 0; i <= j; ++i) {
            st->coef[i] = i == 0 ? red[0] * st->v0s : red[i];
            st->hc[i] += red[i];
        }
    }
    const double hn = k2 > 0.0 ? sqrt(k2) : 0.0;
    st->scale = hn > 0.0 ? 1.0 / hn : 0.0;
    double *H = st->H;
    constexpr int R = kG3MaxRestart;
    for (int i = 0; i <= j; ++i) H[i * R + j] = st->hc[i];
    H[(j + 1) * R + j] = hn;
    for (int i = 0; i < j; ++i) {
        const double a0 = H[i * R + j], a1 = H[(i + 1) * R + j];
        H[i * R + j] = st->cs[i] * a0 + st->sn[i] * a1;
        H[(i + 1) * R + j] = -st->sn[i] * a0 + st->cs[i] * a1;
    }
    const double a0 = H[j * R + j], a1 = H[(j + 1) * R + j];
    const double rr = hypot(a0, a1);
    st->cs[j] = rr > 0.0 ? a0 / rr : 1.0;
    st->sn[j] = rr > 0.0 ? a1 / rr : 0.0;
    H[j * R + j] = rr;
    H[(j + 1) * R + j] = 0.0;
    st->gv[j + 1] = -st->sn[j] * st->gv[j];
    st->gv[j] = st->cs[j] * st->gv[j];
    st->iters += 1;
    st->ncols = j + 1;
    // estimate met (the next cycle checks the true residual), breakdown or
    // the restart length reached
    if (fabs(st->gv[j + 1]) <= rtol * st->bn || hn == 0.0 || j + 1 == m) {
        st->go = 0;
        st->pass2 = 0;
    }
    g3_publish(st, hs);
}

// End of a cycle: H y = g over the cycle's columns (upper triangular), and
// the coefficients -y of the update x += Z y (Z = V unpreconditioned)
__global__ void __launch_bounds__(64) g3_end_kernel(G3State *st)
{
    const int nc = st->ncols;
    if (nc == 0 || threadIdx.x != 0) return;
    constexpr int R = kG3MaxRestart;
    double y[kG3MaxRestart];
    for (int i = nc - 1; i >= 0; --i) {
        double v = st->gv[i];
        for (int l = i + 1; l < nc; ++l) v -= st->H[i * R + l] * y[l];
        y[i] = v / st->H[i * R + i];
    }
    for (int i = 0; i < nc; ++i) st->coef[i] = -y[i];
}

namespace {

struct Kry {
    const G3Work &w;
    hipStream_t s;
    long n;

    void dots(const double *V, int nv, const double *x, const int *gate)
    {
        launch_dots<0>(nv, V, n, x, w.part, gate, s);
    }
    // y = sc (x - sum_j cf_j V_j)
    void axpy(const double *V, int nv, const int *nvp, const double *cf, const double *x, double *y,
              const double *sc, const int *gate)
    {
        hipLaunchKernelGGL(kry_axpy_kernel, dim3(kKryBlocks), dim3(kKryThreads), 0, s, V, n, nv, nvp, cf, x, y, n, sc,
                           gate);
    }
};

}  // namespace

// ---- column preconditioner z = (I - alpha L_v)^-1 v, solved directly.  The
// reference state depends on z alone, so every column has the same matrix, and
// with rho' and theta' eliminated
//   M w = b_w - alpha (1/rho0) (D p_b + g b_rho),   p_b = gamma p0 (b_rho/rho0 + b_theta/theta0),
//   rho' = b_rho - alpha D (rho0 w),   theta' = b_theta - alpha theta0' w
// (D: the DSS'd vertical derivative; identity rows of M and unchanged w at the
// walls).  pc_setup_kernel forms M from three stencil rows, inverts it (n_z <= 130,
// one workgroup) and stores M^-1 and D as operands of v_mfma_f64_16x16x4_f64, once
// per solve.  pc_apply_kernel then is three small products per column, on the
// matrix cores: a workgroup has 16 columns and a wave per 16-level tile of them; a
// lane has column lane % 16 and of block s of four levels the level 4 s + lane / 16.
// That is the B operand of k step s (k = lane / 16) and also the layout of the result
// (row 4 i + lane / 16 in register i), so what the waves hand each other through LDS
// is read and written without conflicts; a wave loads its operands of M^-1 ahead of
// everything else.
// Bound: the pass over memory, 5 fields read and 5 written (41 us for the 65536
// columns of 41 levels of a 64 x 64 x 10, N = 4 mesh at the 5.15 TB/s of a copy;
// 7 us of products): 47 us, where the column GMRES(10) to 1e-6 took 198.  With all
// tiles of 16 columns in one wave, its registers full and every operand waited for:
// 48 us there, and on 61, 77 and 129 levels of 36864 columns 75, 191 and 483 us
// instead of 47, 71 and 138; of 256 columns 20, 33 and 76 instead of 7, 8 and 13.
constexpr int kPcMaxTiles = 9;   // 16-level tiles: n_z <= 130 (and 144)

__host__ __device__ constexpr int pc_halo(int N) { return (N + 3) / 4; }   // blocks of four levels beside a tile's own
__host__ __device__ constexpr int pc_band(int HB) { return 4 + 2 * HB; }

// packed operands: [T][4 NT][64] of M^-1, then [T][pc_band][64] of D
static size_t pc_doubles(int nz, int N)
{
    const size_t NT = (nz + 15) / 16;
    return 64 * NT * (4 * NT + pc_band(pc_halo(N)));
}

size_t g3_precond_bytes(int nz, int N) { return nz <= 16 * kPcMaxTiles ? sizeof(double) * pc_doubles(nz, N) : 0; }

constexpr int kPcThreads = 512;
constexpr int kPcPanel = 8;   // columns per panel (16: 37 for 34 us at 41 levels, alike from 113 on, spills at 129)

// lane l's value, l uniform
__device__ __forceinline__ double lane_of(double v, int l)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return join_d((unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l),
                  (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l));
}

// every lane <- the largest of the wave
__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, lane_move<kSwapPair>(v));
    v = fmax(v, lane_move<kSwapTwo>(v));
    v = fmax(v, lane_move<kHalfMirror>(v));
    v = fmax(v, lane_move<kRowMirror>(v));
    double a = v, b = v;
    swap16(a, b);
    a = b = fmax(a, b);
    swap32(a, b);
    return fmax(a, b);
}

// M from the level table and the stencil rows (staged in LDS), then Gauss-Jordan in
// place with partial pivoting, kPcPanel columns at a time.  The matrix stays in
// registers as 16 x 16 tiles in the layout of an MFMA result, tile w + 8 m in wave w.
// Per panel: its columns go through LDS to wave 0, which eliminates them in its own
// registers (a lane has rows lane + 64 s; no barrier in the steps); then every other
// element a_ij (0 in a pivot row) gains sum_m panel_im a_{p_m j}, two MFMAs a tile.  No rows
// are exchanged: at the end row p_k stands for x_k and column k for right-hand side
// p_k, and the operands are written accordingly.  Once per step (its solves share
// alpha).  Bound: the chain of pivots, about 1 us each.  41, 77, 125 and 129 levels: 34, 72,
// 144 and 191 us; the matrix in the LDS and a barrier after every search, row and
// update: 83 us at 41 levels, about 1150 at 129.
template <int NT>
__global__ void __launch_bounds__(kPcThreads) pc_setup_kernel(HeviParams h, double alpha, double *__restrict__ pack)
{
    typedef double double4v __attribute__((ext_vector_type(4)));
    constexpr int R = 16 * NT, PW = kPcPanel, W = kPcThreads / 64, MT = (NT * NT + W - 1) / W, NS = (R + 63) / 64;
    extern __shared__ double lds[];
    __shared__ double panel[R][PW + 1], prow[PW][R + 1];
    __shared__ int pv[R], kof[R], slot[R];   // p_k, its inverse, a row's place among the panel's pivots (-1: none)
    const int n = h.nz, N = h.N, NC = 2 * N + 1, t = threadIdx.x, lane = t % 64, q = lane / 16, l16 = lane % 16;
    const int wave = __builtin_amdgcn_readfirstlane(t / 64);
    double *L0 = lds, *Lp = L0 + n, *L3 = Lp + n, *L7 = L3 + n, *L8 = L7 + n, *G = L8 + n;
    for (int k = t; k < n; k += kPcThreads) {
        const double *L = h.lev + (long)k * kLevW;
        L0[k] = L[0];
        Lp[k] = h.gamma * L[2];
        L3[k] = L[3];
        L7[k] = L[7];
        L8[k] = L[8];
    }
    for (int e = t; e < n * NC; e += kPcThreads) G[e] = h.gz[e];
    __syncthreads();
    auto D = [&](int r, int c) { return c - r >= -N && c - r <= N ? G[r * NC + c - r + N] : 0.0; };
    auto element = [&](int i, int j) {
        double m = i == j && i < n ? 1.0 : 0.0;
        if (i > 0 && i < n - 1 && j < n) {
            // column j: rho'_k = -alpha D_kj rho0_j, theta'_j = -alpha theta0'_j
            const double cj = -alpha * L0[j];
            const int lo = i > j ? i - N : j - N, hi = i < j ? i + N : j + N;
            double dp = 0.0;
            for (int k = lo > 0 ? lo : 0; k <= hi && k < n; ++k) {
                double pk = cj * D(k, j) * L7[k];
                if (k == j) pk -= alpha * L3[j] * L8[k];
                dp += D(i, k) * Lp[k] * pk;
            }
            m += alpha * L7[i] * (dp + h.g * cj * D(i, j));
        }
        return m;
    };
    // value i of tile (I, J): row 16 I + 4 i + lane / 16, column 16 J + lane % 16
    double4v A[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int id = wave + W * m, I = id / NT, J = id % NT;
#pragma unroll
        for (int i = 0; i < 4; ++i) A[m][i] = id < NT * NT ? element(16 * I + 4 * i + q, 16 * J + l16) : 0.0;
    }
    unsigned taken = 0;   // wave 0, bit s: row lane + 64 s has been a pivot row
    for (int c0 = 0; c0 < n; c0 += PW) {
        const int nk = n - c0 < PW ? n - c0 : PW;
        const bool mine = l16 / PW == c0 % 16 / PW;   // the lane's column in the panel's tiles is one of the panel
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int id = wave + W * m, I = id / NT;
            if (id < NT * NT && id % NT == c0 / 16 && mine)
#pragma unroll
                for (int i = 0; i < 4; ++i) panel[16 * I + 4 * i + q][l16 % PW] = A[m][i];
        }
        for (int i = t; i < R; i += kPcThreads) slot[i] = -1;
        for (int e = t; e < PW * R; e += kPcThreads) prow[e / R][e % R] = 0.0;
        __syncthreads();
        if (wave == 0) {
            double X[NS][PW];
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int c = 0; c < PW; ++c) X[s][c] = lane + 64 * s < R ? panel[lane + 64 * s][c] : 0.0;
            static_for<PW>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                if (j < nk) {
                    // a NaN counts less than any number and more than a row taken
                    double v[NS], iv[NS], m = -1.0;
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const double x = fabs(X[s][j]);
                        v[s] = lane + 64 * s < n && !(taken >> s & 1) ? (x >= 0.0 ? x : -0.5) : -1.0;
                        iv[s] = 1.0 / X[s][j];
                        m = fmax(m, v[s]);
                    }
                    m = wave_max(m);
                    int sp = -1, lp = 0;
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const unsigned long long w = __ballot(v[s] == m);
                        if (sp < 0 && w) {
                            sp = s;
                            lp = __builtin_ctzll(w);
                        }
                    }
                    // the pivot row, scaled
                    double r[PW];
                    static_for<NS>([&](auto sc) __attribute__((always_inline)) {
                        constexpr int s = decltype(sc)::value;
                        if (sp == s) {
                            const double ip = lane_of(iv[s], lp);
#pragma unroll
                            for (int c = 0; c < PW; ++c) r[c] = c == j ? ip : lane_of(X[s][c], lp) * ip;
                        }
                    });
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const double f = X[s][j];
#pragma unroll
                        for (int c = 0; c < PW; ++c) X[s][c] = (c == j ? 0.0 : X[s][c]) - f * r[c];
                    }
                    static_for<NS>([&](auto sc) __attribute__((always_inline)) {
                        constexpr int s = decltype(sc)::value;
                        if (sp == s && lane == lp) {
#pragma unroll
                            for (int c = 0; c < PW; ++c) X[s][c] = r[c];
                            taken |= 1u << s;
                            slot[64 * s + lp] = j;
                            pv[c0 + j] = 64 * s + lp;
                            kof[64 * s + lp] = c0 + j;
                        }
                    });
                }
            });
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int c = 0; c < PW; ++c)
                    if (lane + 64 * s < R) panel[lane + 64 * s][c] = X[s][c];
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int id = wave + W * m, I = id / NT, J = id % NT;
            if (id < NT * NT)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int p = slot[16 * I + 4 * i + q];
                    if (p >= 0) {
                        prow[p][16 * J + l16] = A[m][i];
                        A[m][i] = 0.0;
                    }
                }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int id = wave + W * m, I = id / NT, J = id % NT;
            if (id < NT * NT) {
#pragma unroll
                for (int k = 0; k < PW; k += 4)
                    A[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(panel[16 * I + l16][k + q], prow[k + q][16 * J + l16], A[m],
                                                                0, 0, 0);
                if (J == c0 / 16 && mine)
#pragma unroll
                    for (int i = 0; i < 4; ++i) A[m][i] = panel[16 * I + 4 * i + q][l16 % PW];
            }
        }
        __syncthreads();
    }
    constexpr int S = 4 * NT;
    const int HB = pc_halo(N), NBD = pc_band(HB);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int id = wave + W * m;
        if (id < NT * NT)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * (id / NT) + 4 * i + q, c = 16 * (id % NT) + l16;
                const bool in = r < n && c < n;
                const int x = in ? kof[r] : r, k = in ? pv[c] : c;
                pack[((long)(x / 16) * S + k / 4) * 64 + k % 4 * 16 + x % 16] = in ? A[m][i] : 0.0;
            }
    }
    double *pd = pack + (long)NT * S * 64;
    for (int e = t; e < NT * NBD * 64; e += kPcThreads) {
        const int l = e % 64, b = e / 64 % NBD, T = e / (64 * NBD);
        const int i = 16 * T + l % 16, k = 4 * (4 * T - HB + b) + l / 16;
        pd[e] = i < n && k >= 0 && k < n && k - i >= -N && k - i <= N ? G[i * NC + k - i + N] : 0.0;
    }
}

template <int NT, int HB>
__global__ void __launch_bounds__(64 * NT) pc_apply_kernel(HeviParams h, double alpha,
                                                                const double *__restrict__ v, double *__restrict__ z,
                                                                const double *__restrict__ pack,
                                                                const double *__restrict__ lev, const int *gate,
                                                                const double *scale)
{
    if (gate && *gate == 0) return;
    typedef double double4v __attribute__((ext_vector_type(4)));
    constexpr int S = 4 * NT, NB = pc_band(HB);
    __shared__ double su[S][64], sw[S][64];
    const double sc = scale ? *scale : 1.0;
    const int lane = threadIdx.x % 64, T = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), q = lane / 16;
    const long nxy = (long)h.nx * h.ny, U = nxy * h.nz, c = blockIdx.x * 16L + lane % 16;
    const bool own = c < nxy;
    const double *x = v + (own ? c : nxy - 1);
    double *y = z + c;
    const int nz = h.nz;
    const double *pm = pack + (long)T * S * 64 + lane, *pd = pack + ((long)NT * S + T * NB) * 64 + lane;
    double om[S], od[NB], br[4], bw[4], bt[4], bu[4], bv[4], L0[4], L3[4], L7[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * (4 * T + i) + q;
        const long o = (long)(k < nz ? k : nz - 1) * nxy;
        br[i] = sc * x[o];
        bu[i] = sc * x[U + o];
        bv[i] = sc * x[2 * U + o];
        bw[i] = sc * x[3 * U + o];
        bt[i] = sc * x[4 * U + o];
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) od[b] = pd[b * 64];
#pragma unroll
    for (int s = 0; s < S; ++s) om[s] = pm[s * 64];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * (4 * T + i) + q;
        const bool in = k < nz;
        const double *L = lev + (long)(in ? k : nz - 1) * kLevW;
        L0[i] = L[0];
        L3[i] = L[3];
        L7[i] = L[7];
        su[4 * T + i][lane] = in ? h.gamma * L[2] * (br[i] * L[7] + bt[i] * L[8]) : 0.0;
        if (own && in) {
            const long o = (long)k * nxy;
            y[U + o] = bu[i];
            y[2 * U + o] = bv[i];
        }
    }
    // D u over the levels of the tile
    auto deriv = [&]() __attribute__((always_inline)) {
        double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int s = 4 * T - HB + b;
            if (s >= 0 && s < S) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(od[b], su[s][lane], acc, 0, 0, 0);
        }
        return acc;
    };
    __syncthreads();
    {
        const double4v acc = deriv();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 4 * (4 * T + i) + q;
            const double r = k > 0 && k < nz - 1 ? bw[i] - alpha * L7[i] * (acc[i] + h.g * br[i]) : bw[i];
            sw[4 * T + i][lane] = k < nz ? r : 0.0;
        }
    }
    __syncthreads();
    {
        double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < S; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(om[s], sw[s][lane], acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 4 * (4 * T + i) + q;
            su[4 * T + i][lane] = k < nz ? L0[i] * acc[i] : 0.0;
            if (own && k < nz) {
                const long o = (long)k * nxy;
                y[3 * U + o] = acc[i];
                y[4 * U + o] = bt[i] - alpha * L3[i] * acc[i];
            }
        }
    }
    __syncthreads();
    const double4v acc = deriv();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * (4 * T + i) + q;
        if (own && k < nz) y[(long)k * nxy] = br[i] - alpha * acc[i];
    }
}

template <int NT>
static hipError_t launch_pc_setup(int nt, const L3Params &h, double alpha, double *pack, hipStream_t s)
{
    if constexpr (NT > kPcMaxTiles) {
        return hipErrorInvalidValue;
    } else {
        if (nt != NT) return launch_pc_setup<NT + 1>(nt, h, alpha, pack, s);
        const size_t lds = sizeof(double) * (size_t)h.nz * (5 + 2 * h.N + 1);
        hipLaunchKernelGGL((pc_setup_kernel<NT>), dim3(1), dim3(kPcThreads), lds, s, h.hv, alpha, pack);
        return hipGetLastError();
    }
}

template <int NT>
static hipError_t launch_pc_apply(int nt, const L3Params &h, double alpha, const double *v, double *z,
                                  const double *pack, const int *gate, const double *scale, hipStream_t s)
{
    if constexpr (NT > kPcMaxTiles) {
        return hipErrorInvalidValue;
    } else {
        if (nt != NT) return launch_pc_apply<NT + 1>(nt, h, alpha, v, z, pack, gate, scale, s);
        const dim3 grid((unsigned)(((long)h.nx * h.ny + 15) / 16)), blk(64 * NT);
        if (pc_halo(h.N) == 1)
            hipLaunchKernelGGL((pc_apply_kernel<NT, 1>), grid, blk, 0, s, h.hv, alpha, v, z, pack, h.lev, gate, scale);
        else
            hipLaunchKernelGGL((pc_apply_kernel<NT, 2>), grid, blk, 0, s, h.hv, alpha, v, z, pack, h.lev, gate, scale);
        return hipGetLastError();
    }
}

// The host queues one Arnoldi step while the previous one runs: before it
// queues step j it waits for the event after step j - 2 (the cycle start for
// j = 1) and reads the status the kernels wrote, so at most one step is
// queued past the end of the process, and that one does nothing.  One
// stream synchronisation per solve reads the result.
hipError_t gmres3d(const L3Params &h, const G3Work &w, double alpha, const double *b, const double *x0, double *x,
                   int m, int max_restarts, double rtol, bool precond, bool pc_ready, hipStream_t s, int *iters,
                   double *relres)
{
    const long n = (long)kNF * h.nx * h.ny * h.nz;
    Kry k{w, s, n};
    hipError_t e;
    G3State *st = w.state;
    double *V = w.V;   // (m + 1) vectors of n
    *iters = 0;
    *relres = 0.0;
    if (precond && !pc_ready && (e = launch_pc_setup<1>((h.nz + 15) / 16, h, alpha, w.pc, s)) != hipSuccess) return e;
    // ||b||; the first cycle starts from x0 (or b) and writes x; x = 0 when b = 0
    k.dots(V, 0, b, nullptr);
    hipLaunchKernelGGL(g3_begin_kernel, dim3(1), dim3(kKryCtl), 0, s, st, (const double *)w.part, w.status_dev);
    const double *xs = x0 ? x0 : b;
    if ((e = hipGetLastError()) != hipSuccess) return e;
    auto mark = [&](int i) { return hipEventRecord(w.ev[i & 1], s); };
    for (int cyc = 0; cyc <= max_restarts + 1; ++cyc) {
        const bool final = cyc == max_restarts + 1;
        // V_0 = r = b - (x - alpha L x) and the partials of ||r||
        int nb = 0;
        if ((e = launch_l3_form<true>(h, xs, V, 1.0, -alpha, s, &st->open, b, w.part, &nb)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(g3_cycle_kernel, dim3(1), dim3(kKryCtl), 0, s, st, (const double *)w.part, nb, rtol,
                           final ? 1 : 0, precond ? 1 : 0, w.status_dev);
        if (final) break;
        if (!precond) k.axpy(V, 0, nullptr, nullptr, V, V, &st->scale, &st->go);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = mark(0)) != hipSuccess) return e;
        bool waited = false;
        for (int j = 0; j < m; ++j) {
            if (j >= 1) {
                if ((e = hipEventSynchronize(w.ev[(j - 1) & 1])) != hipSuccess) return e;
                waited = true;
                if (w.status->go == 0) break;
            }
            double *vj = V + (long)j * n, *vn = V + (long)(j + 1) * n;
            // flexible GMRES: z_j = M^-1 v_j kept, the new direction is A z_j
            const double *zj = vj;
            if (precond) {
                double *zz = w.Z + (long)j * n;
                if ((e = launch_pc_apply<1>((h.nz + 15) / 16, h, alpha, vj, zz, w.pc, &st->go,
                                            j == 0 ? &st->v0s : nullptr, s)) != hipSuccess)
                    return e;
                zj = zz;
            }
            if ((e = launch_l3(h, zj, vn, 1.0, -alpha, s, &st->go)) != hipSuccess) return e;
            // classical Gram-Schmidt, the second pass gated on the first's verdict
            k.dots(V, j + 1, vn, &st->go);
            hipLaunchKernelGGL(g3_column_kernel, dim3(1), dim3(kKryCtl), 0, s, st, (const double *)w.part, j, m, rtol,
                               1, w.status_dev);
            k.axpy(V, j + 1, nullptr, st->coef, vn, vn, &st->scale, &st->go);
            k.dots(V, j + 1, vn, &st->pass2);
            hipLaunchKernelGGL(g3_column_kernel, dim3(1), dim3(kKryCtl), 0, s, st, (const double *)w.part, j, m, rtol,
                               2, w.status_dev);
            k.axpy(V, j + 1, nullptr, st->coef, vn, vn, &st->scale, &st->pass2);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = mark(j + 1)) != hipSuccess) return e;
        }
        if (!waited && (e = hipEventSynchronize(w.ev[0])) != hipSuccess) return e;
        // x += Z y over the cycle's columns
        hipLaunchKernelGGL(g3_end_kernel, dim3(1), dim3(64), 0, s, st);
        k.axpy(precond ? w.Z : V, 0, &st->ncols, st->coef, xs, x, nullptr, cyc == 0 ? nullptr : &st->ncols);
        xs = x;
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (w.status->open == 0) break;
    }
    k.axpy(V, 0, nullptr, nullptr, x, x, &st->zero, &st->bzero);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    *iters = w.status->iters;
    *relres = w.status->relres;
    return hipSuccess;
}

}  // namespace nh
