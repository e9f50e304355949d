// gfx950 kernels of the batched column GMRES with z-elements mapped to lanes:
// (I - alpha L_v) x = b in every lattice column (the HEVI stage systems,
// Sec. 2.3), and its Schur complement in w, for columns of at most 16
// elements and restart lengths up to 20.  The method is that of nh_hevi.hip
// (restarted GMRES(m), classical Gram-Schmidt with the re-orthogonalisation
// test of Daniel, Gragg, Kaufman and Stewart, Arnoldi on L_v itself, the
// residual test ||b - A x|| <= rtol ||b|| confirmed with the true residual);
// what differs is where a column's unknowns live.
//
// A column takes 16 or 32 lanes of the wavefront and a lane owns a z-element
// (or one of two halves of its unknowns), so that
//   * L_v is the element-local contraction with the LGL matrix D, whose
//     entries are wave-uniform (scalar registers), plus one value exchanged
//     with the element above and one with the element below (DPP moves): the
//     (2N+1)-tap rows and the LDS exchange of the one-column-per-wave form
//     are gone;
//   * dot products end in a 16- or 32-lane butterfly, and everything done
//     once per column and step (norms, convergence, the least-squares problem)
//     is done for the four (two) columns of a wave by one instruction.
// The columns of a wave restart together and a column that has converged is
// frozen; each column's Arnoldi steps and its solution are those it would
// have alone.
//
// What bounds it: VALU issue of one wave per SIMD (the basis fills the
// register file).  Measured on 147,456 columns of 16 order-4 elements
// (n_z = 65, GMRES(10) to 1e-10, 28.9 steps): 3.23 ms per solve against 7.53
// with one column per wave, 234 VALU instructions per column and step
// against 524, VALU issue in 51 % of the cycles.
#include "nh_internal.h"
#include "nh_lanes.h"

#include <float.h>
#include <math.h>

namespace nh {

namespace {

constexpr int kColElems = 16;   // elements of a column, at most

constexpr int kRowShl1 = 0x101;   // lane i <- lane i + 1, inside 16-lane rows
constexpr int kRowShr1 = 0x111;   // lane i <- lane i - 1
constexpr int kRowShr2 = 0x112;
constexpr int kRowBcast = 0x150;  // every lane of a row <- lane L (0x150 + L)
constexpr int kWaveShl1 = 0x130;  // lane i <- lane i + 1, over the wave
constexpr int kWaveShr1 = 0x138;

// Lane groups of a column: 16 lanes (a DPP row) or 32 (half the wave).
// sum, sum2: one or two sums over the group, left in every lane;
// bcast<L>: lane L of the group to every lane.
struct Row16 {
    static constexpr int LANES = 16;
    static __device__ __forceinline__ double sum(double a) { return row_sum(a); }
    static __device__ __forceinline__ void sum2(double &a, double &b)
    {
        a = row_sum(a);
        b = row_sum(b);
    }
    template <int L>
    static __device__ __forceinline__ double bcast(double v)
    {
        return lane_move<kRowBcast + L>(v);
    }
};
struct Half32 {
    static constexpr int LANES = 32;
    static __device__ __forceinline__ void sum2(double &a, double &b)
    {
        swap16(a, b);
        a = row_sum(a + b);   // rows 0, 2: sums of a; rows 1, 3: sums of b
        b = a;
        swap16(a, b);
    }
    static __device__ __forceinline__ double sum(double a)
    {
        double b = 0.0;
        sum2(a, b);
        return a;
    }
    template <int L>
    static __device__ __forceinline__ double bcast(double v)
    {
        double a = lane_move<kRowBcast + L % 16>(v), b = a;
        swap16(a, b);      // a: row 0 (2) of the broadcast in rows 0, 1 (2, 3); b: row 1 (3)
        return L < 16 ? a : b;
    }
};

// 1 / sqrt(x) for normal x > 0: the hardware estimate and two Newton steps
// (the residual in full precision), within a few units in the last place
__device__ __forceinline__ double inv_sqrt(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = y + 0.5 * y * fma(-x * y, y, 1.0);
    return y + 0.5 * y * fma(-x * y, y, 1.0);
}

// The LGL derivative matrix in scalar registers: the host makes it exactly
// antisymmetric, D[N-i][N-j] = -D[i][j], so half of its entries are kept.
template <int N>
struct DMat {
    static constexpr int NN = (N + 1) * (N + 1), H = NN / 2;
    double v[H];
    __device__ __forceinline__ explicit DMat(const double *__restrict__ D)
    {
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const unsigned long long b = (unsigned long long)__double_as_longlong(D[i]);
            v[i] = join_d((unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b),
                          (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32)));
        }
    }
    // d[l] = sum_m D[l][m] F[m], l = 0 .. N
    __device__ __forceinline__ void contract(const double (&F)[N + 1], double (&d)[N + 1]) const
    {
#pragma unroll
        for (int l = 0; l <= N; ++l) {
            double a = 0.0;
            bool first = true;
#pragma unroll
            for (int m = 0; m <= N; ++m) {
                const int i = l * (N + 1) + m;
                if (2 * i == NN - 1) continue;   // the centre entry of an even order is zero
                const double c = i < H ? v[i] : -v[NN - 1 - i];
                a = first ? c * F[m] : a + c * F[m];
                first = false;
            }
            d[l] = a;
        }
    }
};

// Column groups of a wave: XCD b mod 8 works through a contiguous range of
// groups, so that the pieces of a cache line that different waves read meet
// in one L2.
struct GroupWalk {
    int at, end, step;
    __device__ __forceinline__ GroupWalk(int ngrp)
    {
        const int x = blockIdx.x & (kXcds - 1), per = (ngrp + kXcds - 1) / kXcds;
        at = x * per + (int)(blockIdx.x / kXcds);
        end = (x + 1) * per < ngrp ? (x + 1) * per : ngrp;
        step = (int)(gridDim.x / kXcds);
    }
};

template <int S>
__device__ __forceinline__ double dot(const double (&a)[S], const double (&b)[S])
{
    double p = a[0] * b[0], q = S > 1 ? a[S > 1 ? 1 : 0] * b[S > 1 ? 1 : 0] : 0.0;
#pragma unroll
    for (int s = 2; s < S; ++s) (s & 1 ? q : p) += a[s] * b[s];
    return p + q;
}

// r = b - (x - al Op x); its norm
template <class G, class Op>
__device__ __forceinline__ double residual(const Op &op, double al, const double (&x)[Op::S], const double (*sb)[64],
                                           double (&r)[Op::S])
{
    const int lane = threadIdx.x;
    double cf[Op::NC];
    op.coefficients(cf);
    op.apply(x, cf, r);
#pragma unroll
    for (int s = 0; s < Op::S; ++s) r[s] = sb[s][lane] - (x[s] - al * r[s]);
    return sqrt(G::sum(dot(r, r)));
}

// Restarted GMRES(m), m <= M, for A = I - al Op in every lane group of the
// wave.  sx: iterate (updated), sb: right-hand side, one row of 64 lanes per
// slot; sv: basis vectors VR .. M-1 (the first VR are in registers); sH: the
// group's M (M + 1) doubles.  act: the group has a system to solve; conv and
// iters are set for it.
template <class G, class Op, int M, int VR>
__device__ __forceinline__ void gmres_lanes(const Op &op, double al, double tol, int m, int max_restarts, bool act,
                                            double (*sx)[64], const double (*sb)[64], double (*sv)[64], double *sH,
                                            bool &conv, int &iters)
{
    static_assert(M <= G::LANES, "a lane per Hessenberg column");
    constexpr int S = Op::S, ML = M > VR ? M - VR : 0;
    const int lane = threadIdx.x, ln = lane % G::LANES;
    const double ial = 1.0 / al;
    bool est = false;
    for (int rs = 0;; ++rs) {
        double V[VR][S], cur[S], w[S];
#pragma unroll
        for (int s = 0; s < S; ++s) w[s] = sx[s][lane];
        const double rn = residual<G>(op, al, w, sb, cur);
        // a system stops with its true residual; after the last cycle only
        // where the residual estimate had said so too
        if (act && rn <= tol && (rs <= max_restarts || est)) {
            conv = true;
            act = false;
        }
        if (rs > max_restarts || !__any(act)) break;
        {
            const double inv = rn > 0.0 ? 1.0 / rn : 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                cur[s] *= inv;
                V[0][s] = cur[s];
            }
            static_for<VR - 1>([&](auto ic) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < S; ++s) V[decltype(ic)::value + 1][s] = 0.0;
            });
        }
        // Residual estimate without rotations: the left null vector p of the
        // (j+2) x (j+1) Hessenberg matrix of A, p_0 = 1 and
        // p_{j+1} = -sum_i p_i h_ij / h_{j+1,j}; the least-squares residual is
        // parallel to it, of norm rn / |p|.
        double p[M + 1], pp = 1.0;
        p[0] = 1.0;
        static_for<M>([&](auto ic) __attribute__((always_inline)) { p[decltype(ic)::value + 1] = 0.0; });
        int jn = 0, j = 0;
        bool run = act;
        est = false;
        const double rt = rn / tol, rt2 = rt * rt;
        {
            double cf[Op::NC];
            op.coefficients(cf);
            op.apply(cur, cf, w);
        }
        // One step's code for every j (unrolled steps spilled): register
        // vectors beyond V_j are zero, and pairs of them past j are skipped.
        // w = Op V_j on entry; the next step's product is formed before the
        // convergence test, beside the scalar work of this one.
        for (; j < m && __any(run); ++j) {
            // Gram-Schmidt: all dot products, then one update, the norm from
            // Pythagoras
            double hc[VR], hl[ML ? ML : 1];
            double w2 = dot(w, w);
            static_for<(VR + 1) / 2>([&](auto qc) __attribute__((always_inline)) {
                constexpr int i = 2 * decltype(qc)::value;
                hc[i] = 0.0;
                if constexpr (i + 1 < VR) hc[i + 1] = 0.0;
                if (i <= j) {
                    hc[i] = dot(w, V[i]);
                    if constexpr (i + 1 < VR) hc[i + 1] = dot(w, V[i + 1]);
                }
            });
            w2 = G::sum(w2);
            static_for<(VR + 1) / 2>([&](auto qc) __attribute__((always_inline)) {
                constexpr int i = 2 * decltype(qc)::value;
                if (i <= j) {
                    if constexpr (i + 1 < VR) G::sum2(hc[i], hc[i + 1]);
                    else hc[i] = G::sum(hc[i]);
                }
            });
            double p2 = 0.0;
            if constexpr (ML > 0)
                static_for<ML>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    hl[i] = 0.0;
                    if (VR + i <= j) {
                        double v[S];
#pragma unroll
                        for (int s = 0; s < S; ++s) v[s] = sv[i * S + s][lane];
                        hl[i] = G::sum(dot(w, v));
                        p2 += hl[i] * hl[i];
                    }
                });
            static_for<(VR + 1) / 2>([&](auto qc) __attribute__((always_inline)) {
                constexpr int i = 2 * decltype(qc)::value;
                if (i <= j) {
                    p2 += hc[i] * hc[i];
#pragma unroll
                    for (int s = 0; s < S; ++s) w[s] -= hc[i] * V[i][s];
                    if constexpr (i + 1 < VR) {
                        p2 += hc[i + 1] * hc[i + 1];
#pragma unroll
                        for (int s = 0; s < S; ++s) w[s] -= hc[i + 1] * V[i + 1][s];
                    }
                }
            });
            if constexpr (ML > 0)
                static_for<ML>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    if (VR + i <= j)
#pragma unroll
                        for (int s = 0; s < S; ++s) w[s] -= hl[i] * sv[i * S + s][lane];
                });
            double nn2 = w2 - p2;
            const bool again = nn2 < 1e-4 * w2;
            if (__any(again && run)) {
                // the projection kept less than 1 % of |w| (about 45 % of the
                // steps of an acoustic column): a second pass, two vectors at
                // a time against the updated w, and the norm taken directly
                static_for<(VR + 1) / 2>([&](auto qc) __attribute__((always_inline)) {
                    constexpr int i = 2 * decltype(qc)::value, i1 = i + 1 < VR ? i + 1 : i;
                    if (i <= j) {
                        double q0 = dot(w, V[i]), q1 = i1 > i ? dot(w, V[i1]) : 0.0;
                        G::sum2(q0, q1);
                        q0 = again ? q0 : 0.0;
                        q1 = again && i1 > i ? q1 : 0.0;
                        hc[i] += q0;
                        if (i1 > i) hc[i1] += q1;
#pragma unroll
                        for (int s = 0; s < S; ++s) w[s] = w[s] - q0 * V[i][s] - q1 * V[i1][s];
                    }
                });
                if constexpr (ML > 0)
                    static_for<ML>([&](auto ic) __attribute__((always_inline)) {
                        constexpr int i = decltype(ic)::value;
                        if (VR + i <= j) {
                            double v[S];
#pragma unroll
                            for (int s = 0; s < S; ++s) v[s] = sv[i * S + s][lane];
                            const double q0 = G::sum(dot(w, v)), q = again ? q0 : 0.0;
                            hl[i] += q;
#pragma unroll
                            for (int s = 0; s < S; ++s) w[s] -= q * v[s];
                        }
                    });
                const double t2 = G::sum(dot(w, w));
                nn2 = again ? t2 : nn2;
            }
            double cf[Op::NC];
            op.coefficients(cf);
            const bool brk = !(nn2 > 0.0);   // breakdown (or NaN): the vector is left unscaled
            const double inv = brk ? 1.0 : inv_sqrt(nn2), nn = brk ? 0.0 : nn2 * inv;
#pragma unroll
            for (int s = 0; s < S; ++s) cur[s] = w[s] * inv;
            static_for<VR - 1>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value + 1;
                if (j + 1 == i) {
#pragma unroll
                    for (int s = 0; s < S; ++s) V[i][s] = cur[s];
                    // ends each branch differently: merged, the stores would
                    // index V at run time and move it to scratch
                    asm volatile("; basis vector %0" ::"n"(i));
                }
            });
            if constexpr (ML > 0)
                if (j + 1 >= VR && j + 1 < M)
#pragma unroll
                    for (int s = 0; s < S; ++s) sv[(j + 1 - VR) * S + s][lane] = cur[s];
            op.apply(cur, cf, w);
            // column j of the Hessenberg matrix of Op to LDS; the new
            // component of p (h_ij = delta_ij - al times it)
            double A = 0.0, pl = p[0];
            static_for<M>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                A += p[i] * (i < VR ? hc[i < VR ? i : 0] : hl[i < VR ? 0 : i - VR]);
                if constexpr (i > 0) pl = i <= j ? p[i] : pl;
            });
            if (ln == 0) {
                static_for<M>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    sH[j * (M + 1) + i] = i < VR ? hc[i < VR ? i : 0] : hl[i < VR ? 0 : i - VR];
                });
                sH[j * (M + 1) + j + 1] = nn;
            }
            const double pj = (pl - al * A) * (inv * ial);
            static_for<M>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value + 1;
                p[i] = i == j + 1 ? pj : p[i];
            });
            pp += pj * pj;
            if (run) {
                ++iters;
                jn = j + 1;
                est = (Op::NAN_ENDS ? brk : nn2 <= 0.0) || rt2 <= pp;
                run = !est;
            }
        }
        wave_sync();
        // Least squares: lane k of a group takes column k of the Hessenberg
        // matrix of A and the rotations run over all columns at once
        // (rotation i from column i, broadcast over the group); a system that
        // stopped at jn takes its first jn columns.  The long form leaves out
        // what lies past the last step any column of the wave took: 20 columns
        // cost more than the steps of a short column do (10 do not, measured).
        constexpr bool kAll = M <= kGmresRegM;
        double y[M];
        {
            double q[M + 1], gv[M + 1], idiag = 1.0;
            static_for<M + 1>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                const bool in = ln < jn && i <= ln + 1;
                const double v = sH[in ? ln * (M + 1) + i : 0];
                q[i] = in ? (i == ln ? 1.0 : 0.0) - al * v : 0.0;
            });
            gv[0] = rn;
            static_for<M>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                if (kAll || i < j) {
                    const double a = G::template bcast<i>(q[i]), b = G::template bcast<i>(q[i + 1]);
                    const double d2 = a * a + b * b;
                    const double id = d2 > 0.0 ? inv_sqrt(d2) : 0.0;
                    const double c = d2 > 0.0 ? a * id : 1.0, sn = b * id;
                    if (ln == i && i < jn) idiag = id;
                    const double u = q[i], v = q[i + 1];
                    q[i] = c * u + sn * v;
                    q[i + 1] = c * v - sn * u;
                    gv[i + 1] = -sn * gv[i];
                    gv[i] = c * gv[i];
                }
            });
            static_for<M>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = M - 1 - decltype(ic)::value;
                y[i] = 0.0;
                if (kAll || i < j) {
                    const double yi = i < jn ? gv[i] * G::template bcast<i>(idiag) : 0.0;
                    y[i] = yi;
                    static_for<i>([&](auto kc) __attribute__((always_inline)) {
                        constexpr int k = decltype(kc)::value;
                        gv[k] -= yi * G::template bcast<i>(q[k]);
                    });
                }
            });
        }
#pragma unroll
        for (int s = 0; s < S; ++s) cur[s] = sx[s][lane];
        static_for<M>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            if (i < j) {
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    if constexpr (i < VR) cur[s] += y[i] * V[i][s];
                    else cur[s] += y[i] * sv[(i < VR ? 0 : i - VR) * S + s][lane];
                }
            }
        });
        if (jn > 0)
#pragma unroll
            for (int s = 0; s < S; ++s) sx[s][lane] = cur[s];
        wave_sync();   // sH is rewritten by the next cycle
    }
}

// ---------------------------------------------------------------- one element per lane
// Level coefficients of a lane's element, one LDS row of 16 lanes each.  The
// top level nz - 1 belongs to lane nelz (level 0) when there is such a lane,
// else (FULL: 16 elements) to the extra coefficients of lane 15.
template <int N>
struct Cf {
    static constexpr int RHO = 0;          // rho0 of level l
    static constexpr int PR = N;           // gamma p0 / rho0
    static constexpr int PT = 2 * N;       // gamma p0 / theta0
    static constexpr int IW = 3 * N;       // 1 / rho0, 0 on the walls (their w row is zero)
    static constexpr int DT = 4 * N;       // d theta0 / dz
    static constexpr int H2 = 5 * N;       // 2 / h
    static constexpr int WB = H2 + 1;      // w_hi 2 / h of the bottom level
    static constexpr int WT = H2 + 2;      // w_lo 2 / h of the element's top level
    static constexpr int T_RHO = H2 + 3;   // FULL, lane 15 (T_DT: lane tdl) only: the top level's
    static constexpr int T_PR = H2 + 4;
    static constexpr int T_PT = H2 + 5;
    static constexpr int T_DT = H2 + 6;
    static constexpr int COUNT = H2 + 7;
};

template <int N, bool FULL>
__device__ __forceinline__ void fill_coefficients(const HeviParams &h, double (*sc)[kColElems], int tdl)
{
    using C = Cf<N>;
    const int lane = threadIdx.x, nz = h.nz, nelz = (nz - 1) / N;
    for (int i = lane; i < C::COUNT * kColElems; i += 64) {
        const int c = i / kColElems, e = i % kColElems;
        const bool elem = e < nelz;
        double v = 0.0;
        if (c < C::H2) {
            const int k = e * N + c % N;
            if (elem || (e == nelz && c % N == 0)) {
                const double *L = h.lev + (long)k * kLevW;
                switch (c / N) {
                case 0: v = L[0]; break;
                case 1: v = h.gamma * L[2] * L[7]; break;
                case 2: v = h.gamma * L[2] * L[8]; break;
                case 3: v = (k == 0 || k == nz - 1) ? 0.0 : L[7]; break;
                default: v = L[3]; break;
                }
            }
        } else if (c < C::T_RHO) {
            if (elem) {
                if (c == C::H2) v = h.hz2[e];
                if (c == C::WB) v = h.hz2[e] * h.lev[(long)(e * N) * kLevW + 6];
                if (c == C::WT) v = h.hz2[e] * h.lev[(long)(e * N + N) * kLevW + 5];
            }
        } else if (FULL) {
            const double *T = h.lev + (long)(nz - 1) * kLevW;
            if (c == C::T_RHO && e == kColElems - 1) v = T[0];
            if (c == C::T_PR && e == kColElems - 1) v = h.gamma * T[2] * T[7];
            if (c == C::T_PT && e == kColElems - 1) v = h.gamma * T[2] * T[8];
            if (c == C::T_DT && e == tdl) v = T[3];
        }
        sc[c][e] = v;
    }
}

// L_v on (rho', w, theta').  Slots of a lane: 0 .. N-1 rho', N .. 2N-1 w,
// 2N .. 3N-1 theta' of its element's levels; with 16 elements (FULL) one more
// slot holds the top level, theta' in lane 13, w in lane 14, rho' in lane 15.
template <int N, bool FULL>
struct ElemOp {
    using C = Cf<N>;
    static constexpr int S = 3 * N + (FULL ? 1 : 0), NC = C::COUNT, TDL = kColElems - 3;
    static constexpr bool NAN_ENDS = false;   // a NaN ends a cycle of GMRES
    const double (*sc)[kColElems];
    DMat<N> D;
    double grav;
    int e;
    __device__ __forceinline__ void coefficients(double (&c)[NC]) const
    {
        int l = e;   // laundered: read anew each time rather than kept in registers
        asm volatile("" : "+v"(l));
#pragma unroll
        for (int i = 0; i < (FULL ? C::COUNT : C::T_RHO); ++i) c[i] = sc[i][l];
    }
    __device__ __forceinline__ void apply(const double (&x)[S], const double (&c)[NC], double (&y)[S]) const
    {
        double F[N + 1], P[N + 1], dF[N + 1], dP[N + 1];
#pragma unroll
        for (int l = 0; l < N; ++l) {
            F[l] = c[C::RHO + l] * x[N + l];
            P[l] = c[C::PR + l] * x[l] + c[C::PT + l] * x[2 * N + l];
        }
        F[N] = lane_move<kRowShl1>(F[0]);
        P[N] = lane_move<kRowShl1>(P[0]);
        if constexpr (FULL) {
            F[N] += c[C::T_RHO] * lane_move<kRowShr1>(x[3 * N]);
            P[N] += c[C::T_PR] * x[3 * N] + c[C::T_PT] * lane_move<kRowShr2>(x[3 * N]);
        }
        D.contract(F, dF);
        D.contract(P, dP);
        const double tF = c[C::WT] * dF[N], tP = c[C::WT] * dP[N];
        dF[0] = c[C::WB] * dF[0] + lane_move<kRowShr1>(tF);
        dP[0] = c[C::WB] * dP[0] + lane_move<kRowShr1>(tP);
#pragma unroll
        for (int l = 1; l < N; ++l) {
            dF[l] *= c[C::H2];
            dP[l] *= c[C::H2];
        }
#pragma unroll
        for (int l = 0; l < N; ++l) {
            y[l] = -dF[l];
            y[N + l] = -c[C::IW + l] * (dP[l] + grav * x[l]);
            y[2 * N + l] = -c[C::DT + l] * x[N + l];
        }
        if constexpr (FULL) {
            // rho' row of the top level in lane 15, theta' row in lane 13
            // (T_DT is kept there), w row zero
            const double yt = c[C::T_DT] * lane_move<kRowShl1>(x[3 * N]);
            y[3 * N] = e == kColElems - 1 ? -tF : -yt;
        }
    }
};

// The Schur complement's operator M w = L_w(L_rw w, L_tw w) on the interior w
// (nh_hevi.hip): slots 0 .. N-1 the w of the lane's levels, zero on the walls.
template <int N, bool FULL>
struct SchurOp {
    using C = Cf<N>;
    static constexpr int S = N, NC = C::COUNT, TDL = kColElems - 1;
    static constexpr bool NAN_ENDS = true;
    const double (*sc)[kColElems];
    DMat<N> D;
    double grav;
    int e;
    __device__ __forceinline__ void coefficients(double (&c)[NC]) const
    {
        int l = e;   // laundered: read anew each time rather than kept in registers
        asm volatile("" : "+v"(l));
#pragma unroll
        for (int i = 0; i < (FULL ? C::COUNT : C::T_RHO); ++i) c[i] = sc[i][l];
    }
    __device__ __forceinline__ void derivative(const double (&F)[N + 1], const double (&c)[NC], double (&d)[N + 1]) const
    {
        // d[N]: the element's weighted share at its top level
        D.contract(F, d);
        d[N] *= c[C::WT];
        d[0] = c[C::WB] * d[0] + lane_move<kRowShr1>(d[N]);
#pragma unroll
        for (int l = 1; l < N; ++l) d[l] *= c[C::H2];
    }
    // r = rb + a L_rw w, t = tb + a L_tw w on every level (index N: the top
    // level, FULL, lane 15), y = L_w(r, t)
    __device__ __forceinline__ void chain(double a, const double (&w)[N + 1], const double (&rb)[N + 1],
                                          const double (&tb)[N + 1], const double (&c)[NC], double (&r)[N + 1],
                                          double (&t)[N + 1], double (&y)[N]) const
    {
        double F[N + 1], P[N + 1], d[N + 1];
#pragma unroll
        for (int l = 0; l < N; ++l) F[l] = c[C::RHO + l] * w[l];
        F[N] = lane_move<kRowShl1>(F[0]);
        if constexpr (FULL) F[N] += c[C::T_RHO] * w[N];
        derivative(F, c, d);
#pragma unroll
        for (int l = 0; l < N; ++l) {
            r[l] = rb[l] - a * d[l];
            t[l] = tb[l] - a * c[C::DT + l] * w[l];
            P[l] = c[C::PR + l] * r[l] + c[C::PT + l] * t[l];
        }
        P[N] = lane_move<kRowShl1>(P[0]);
        if constexpr (FULL) {
            r[N] = rb[N] - a * d[N];
            t[N] = tb[N] - a * c[C::T_DT] * w[N];
            P[N] += c[C::T_PR] * r[N] + c[C::T_PT] * t[N];
        }
        derivative(P, c, d);
#pragma unroll
        for (int l = 0; l < N; ++l) y[l] = -c[C::IW + l] * (d[l] + grav * r[l]);
    }
    __device__ __forceinline__ void apply(const double (&x)[S], const double (&c)[NC], double (&y)[S]) const
    {
        const double zero[N + 1] = {};
        double w[N + 1], r[N + 1], t[N + 1];
#pragma unroll
        for (int l = 0; l < N; ++l) w[l] = x[l];
        w[N] = 0.0;
        chain(1.0, w, zero, zero, c, r, t, y);
    }
};

// u and v rows of (I - alpha L_v) are the identity: lane e copies its levels
template <int N, bool FULL>
__device__ __forceinline__ void copy_uv(const GmresArgs &g, int nz, long nxy, long col, bool have, int e)
{
    const long U = nxy * nz;
    double c[2 * N + 2];
#pragma unroll
    for (int l = 0; l <= N; ++l) {
        const int k = e * N + l;
        const long I = (have ? col : 0) + (long)(k < nz ? k : nz - 1) * nxy;
        c[2 * l] = g.b[U + I];
        c[2 * l + 1] = g.b[2 * U + I];
    }
#pragma unroll
    for (int l = 0; l <= N; ++l) {
        const int k = e * N + l;
        if (have && k < nz && (l < N || (FULL && k == nz - 1))) {
            const long I = col + (long)k * nxy;
            g.x[U + I] = c[2 * l];
            g.x[2 * U + I] = c[2 * l + 1];
        }
    }
}

// Full form, four columns per wave, restart lengths up to M.
template <int N, bool FULL, int M, int VR>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1)))
gmres_elem_kernel(const HeviParams h, const GmresArgs g, const int ngrp)
{
    using Op = ElemOp<N, FULL>;
    constexpr int S = Op::S, ML = M > VR ? M - VR : 0;
    __shared__ double sc[Op::NC][kColElems];
    __shared__ double sx[S][64], sb[S][64];
    __shared__ double sv[ML ? ML * S : 1][64];
    __shared__ double sH[4][M * (M + 1)];
    const int lane = threadIdx.x, e = lane % 16, row = lane / 16;
    const int nz = h.nz;
    fill_coefficients<N, FULL>(h, sc, Op::TDL);
    __syncthreads();
    const Op op{sc, DMat<N>(h.cst + kCstD), h.g, e};
    const long nxy = (long)h.nx * h.ny, U = nxy * nz;
    for (GroupWalk walk(ngrp); walk.at < walk.end; walk.at += walk.step) {
        const long col = (long)walk.at * 4 + row;
        const bool have = col < nxy;
        // the lane's element, laundered, so that node offsets are not hoisted
        // out of the loop and held in registers through the solve
        int el = e;
        asm volatile("" : "+v"(el));
        // node of slot s: offset in b and x ([5][U], fields rho', w, theta' are
        // 0, 3, 4) and in x0 ([3][U]), clamped into the lattice; slots without
        // a node hold 0.  Loads are unconditional: a load under a branch is
        // waited for where the branch joins.
        auto node = [&](int s, long &o5, long &o3) {
            int f, k;
            bool ok;
            if (FULL && s == 3 * N) {
                f = kColElems - 1 - el;
                ok = f < 3;
                f = ok ? f : 0;
                k = nz - 1;
            } else {
                f = s / N;
                k = el * N + s % N;
                ok = k < nz;
                k = ok ? k : nz - 1;
            }
            const long o = (long)k * nxy + (have ? col : 0);
            o5 = (f == 0 ? 0 : (f + 2) * U) + o;
            o3 = f * U + o;
            return ok && have;
        };
        double b2 = 0.0;
        {
            const double *x0 = g.x0 ? g.x0 : g.b;
            double bb[S], xx[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                long o5, o3;
                const bool ok = node(s, o5, o3);
                const double vb = g.b[o5], vx = x0[g.x0 ? o3 : o5];
                bb[s] = ok ? vb : 0.0;
                xx[s] = ok ? vx : 0.0;
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                sb[s][lane] = bb[s];
                sx[s][lane] = xx[s];
                b2 += bb[s] * bb[s];
            }
        }
        const double bn = sqrt(Row16::sum(b2));
        int iters = 0;
        bool conv = bn == 0.0;
        if (conv)
#pragma unroll
            for (int s = 0; s < S; ++s) sx[s][lane] = 0.0;
        const bool act = have && !conv;
        if (g.pick && g.x0) {
            // start from x0 or from b, whichever has the smaller residual
            double x[S], r[S], q[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                x[s] = sb[s][lane];
                q[s] = sx[s][lane];
            }
            const double rd = residual<Row16>(op, g.alpha, x, sb, r), rg = residual<Row16>(op, g.alpha, q, sb, r);
            if (act && rd < rg)
#pragma unroll
                for (int s = 0; s < S; ++s) sx[s][lane] = x[s];
        }
        gmres_lanes<Row16, Op, M, VR>(op, g.alpha, g.rtol * bn, g.restart, g.max_restarts, act, sx, sb, sv, sH[row],
                                      conv, iters);
        asm volatile("" : "+v"(el));
#pragma unroll
        for (int s = 0; s < S; ++s) {
            long o5, o3;
            if (node(s, o5, o3)) g.x[o5] = sx[s][lane];
        }
        copy_uv<N, FULL>(g, nz, nxy, col, have, el);
        if (e == 0 && have && g.iters) g.iters[col] = conv ? iters : -iters - 1;
        wave_sync();
    }
}

// Schur form, four columns per wave, restart length M.  N unknowns per lane,
// so the basis leaves room for two waves per SIMD (orders above 4: one).
// Measured on the 147,456 columns above (14.6 steps): 0.76 ms per solve against
// 3.17 with one column per wave.
template <int N, bool FULL, int M>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(N <= 4 ? 2 : 1, N <= 4 ? 2 : 1)))
gmres_schur_elem_kernel(const HeviParams h, const GmresArgs g, const int ngrp)
{
    using Op = SchurOp<N, FULL>;
    constexpr int S = N;
    __shared__ double sc[Op::NC][kColElems];
    __shared__ double sx[S][64], sb[S][64];
    __shared__ double sH[4][M * (M + 1)];
    const int lane = threadIdx.x, e = lane % 16, row = lane / 16;
    const int nz = h.nz;
    fill_coefficients<N, FULL>(h, sc, Op::TDL);
    __syncthreads();
    const Op op{sc, DMat<N>(h.cst + kCstD), h.g, e};
    const long nxy = (long)h.nx * h.ny, U = nxy * nz;
    for (GroupWalk walk(ngrp); walk.at < walk.end; walk.at += walk.step) {
        const long col = (long)walk.at * 4 + row;
        const bool have = col < nxy;
        int el = e;
        asm volatile("" : "+v"(el));
        // b of the lane's levels (index N: the top level of lane 15, FULL)
        double br[N + 1], bt[N + 1], bw[N + 1];
        auto load_b = [&]() {
#pragma unroll
            for (int l = 0; l <= N; ++l) {
                const int k = el * N + l;
                const bool ok = have && k < nz && (l < N || (FULL && k == nz - 1));
                const long I = (have ? col : 0) + (long)(k < nz ? k : nz - 1) * nxy;
                const double a = g.b[I], w = g.b[3 * U + I], t = g.b[4 * U + I];
                br[l] = ok ? a : 0.0;
                bw[l] = ok ? w : 0.0;
                bt[l] = ok ? t : 0.0;
            }
        };
        auto interior = [&](int l) { return el * N + l > 0 && el * N + l < nz - 1; };
        load_b();
        const double bn = sqrt(Row16::sum(dot(br, br) + dot(bw, bw) + dot(bt, bt)));
        int iters = 0;
        bool conv = bn == 0.0;
        const bool act = have && !conv;
        const double beta = g.alpha * g.alpha;
        {
            // reduced right-hand side: b_w + alpha L_w(b_rho + alpha L_rw w_wall, b_th + alpha L_tw w_wall)
            double cf[Op::NC], w[N + 1], r[N + 1], t[N + 1], y[N], xd[S], xg[S];
            op.coefficients(cf);
#pragma unroll
            for (int l = 0; l <= N; ++l) w[l] = interior(l) ? 0.0 : bw[l];
            op.chain(g.alpha, w, br, bt, cf, r, t, y);
#pragma unroll
            for (int l = 0; l < N; ++l) {
                const int k = el * N + l;
                const double x0 = g.x0 ? g.x0[U + (have ? col : 0) + (long)(k < nz ? k : nz - 1) * nxy] : bw[l];
                sb[l][lane] = interior(l) ? bw[l] + g.alpha * y[l] : 0.0;
                xd[l] = interior(l) ? bw[l] : 0.0;
                xg[l] = interior(l) && have && !conv ? x0 : 0.0;
                sx[l][lane] = xg[l];
            }
            if (g.pick && g.x0) {
                // start from x0 or from b_w, whichever has the smaller residual
                double q[S];
                const double rd = residual<Row16>(op, beta, xd, sb, q), rg = residual<Row16>(op, beta, xg, sb, q);
                if (act && rd < rg)
#pragma unroll
                    for (int l = 0; l < N; ++l) sx[l][lane] = xd[l];
            }
        }
        // finite (or NaN): a right-hand side with an infinity has an infinite
        // residual, which must not pass for a solution
        const double tol = g.rtol * bn > DBL_MAX ? DBL_MAX : g.rtol * bn;
        gmres_lanes<Row16, Op, M, M>(op, beta, tol, g.restart, g.max_restarts, act, sx, sb, nullptr, sH[row], conv,
                                     iters);
        asm volatile("" : "+v"(el));
        // rho' and theta' from the full w column
        load_b();
        {
            double cf[Op::NC], w[N + 1], r[N + 1], t[N + 1], y[N];
            op.coefficients(cf);
#pragma unroll
            for (int l = 0; l < N; ++l) w[l] = interior(l) ? sx[l][lane] : bw[l];
            w[N] = bw[N];
            op.chain(g.alpha, w, br, bt, cf, r, t, y);
#pragma unroll
            for (int l = 0; l <= N; ++l) {
                const int k = el * N + l;
                if (have && k < nz && (l < N || (FULL && k == nz - 1))) {
                    const long I = col + (long)k * nxy;
                    g.x[I] = r[l];
                    g.x[3 * U + I] = w[l];
                    g.x[4 * U + I] = t[l];
                }
            }
        }
        copy_uv<N, FULL>(g, nz, nxy, col, have, el);
        if (e == 0 && have && g.iters) g.iters[col] = conv ? iters : -iters - 1;
        wave_sync();
    }
}

// ---------------------------------------------------------------- two lanes per element
// Full form with two columns per wave, 32 lanes each, for restart lengths
// whose basis does not fit the registers of 16 lanes.  Lane 2 e + f of a
// column: f = 0 holds w on the N levels of element e and theta' on the lower
// H = ceil(N / 2), f = 1 rho' on the N levels and theta' on the others, so
// that both stencil inputs of L_v (rho0 w in lane 0, p'_L in lane 1) are
// contracted with D by the same instructions; the results change lanes (rho'
// rows need d(rho0 w)/dz, w rows dp'_L/dz).  The top level is level 0 of
// lanes 2 nelz + f when nelz < 16; with 16 elements (FULL) one extra slot holds
// it: theta' in lane 29, w in lane 30, rho' in lane 31.  Measured at restart 20
// (17,760 columns, n_z = 49, 40 steps): 1.25 ms per solve against 7.18 with
// one column per wave and the basis in LDS; at restart 10 the one-lane form
// was the faster one of the two (2.63 ms against 3.55 on 147,456 columns).
// Bound: the latency of its own chain in one wave per SIMD (36 KB of LDS hold the
// six other vectors: four waves to a CU, so those columns are 8.7 rounds of waves):
// VALU active in 52 % of the wave's cycles, 2 % wait to issue, under 1 % for LDS.
template <int N>
struct HalfCf {   // a lane's coefficients
    static constexpr int H = (N + 1) / 2;
    static constexpr int C1 = 0;            // f = 0: rho0; f = 1: gamma p0 / rho0
    static constexpr int C2 = N;            // f = 0: 0;    f = 1: gamma p0 / theta0
    static constexpr int CY = 2 * N;        // f = 0: 1 / rho0 (0 on the walls); f = 1: 1
    static constexpr int DT = 3 * N;        // d theta0 / dz of the lane's theta' levels
    static constexpr int H2 = 3 * N + H;    // 2 / h
    static constexpr int WB = H2 + 1;       // w_hi 2 / h of the bottom level
    static constexpr int WT = H2 + 2;       // w_lo 2 / h of the element's top level
    static constexpr int T1 = H2 + 3;       // FULL: lanes 30, 31: C1 of the top level
    static constexpr int T2 = H2 + 4;       // FULL: lane 31: C2 of the top level
    static constexpr int TD = H2 + 5;       // FULL: lane 29: d theta0 / dz of the top level
    static constexpr int COUNT = H2 + 6;
};

template <int N, bool FULL>
__device__ __forceinline__ void fill_half_coefficients(const HeviParams &h, double (*sc)[32])
{
    using C = HalfCf<N>;
    const int nz = h.nz, nelz = (nz - 1) / N;
    for (int i = threadIdx.x; i < C::COUNT * 32; i += 64) {
        const int c = i / 32, ln = i % 32, e = ln / 2, f = ln % 2;
        const bool elem = e < nelz;
        double v = 0.0;
        if (c < C::H2) {
            const int l = c < C::DT ? c % N : (c - C::DT) + f * C::H;
            const int k = e * N + l;
            if (l < N && (elem || (e == nelz && l == 0))) {
                const double *L = h.lev + (long)k * kLevW;
                if (c < C::C2) v = f ? h.gamma * L[2] * L[7] : L[0];
                else if (c < C::CY) v = f ? h.gamma * L[2] * L[8] : 0.0;
                else if (c < C::DT) v = f ? 1.0 : (k == 0 || k == nz - 1) ? 0.0 : L[7];
                else v = L[3];
            }
        } else {
            const double *T = h.lev + (long)(nz - 1) * kLevW;
            if (c == C::H2 && elem) v = h.hz2[e];
            if (c == C::WB && elem) v = h.hz2[e] * h.lev[(long)(e * N) * kLevW + 6];
            if (c == C::WT && elem) v = h.hz2[e] * h.lev[(long)(e * N + N) * kLevW + 5];
            if (FULL && c == C::T1 && e == kColElems - 1) v = f ? h.gamma * T[2] * T[7] : T[0];
            if (FULL && c == C::T2 && ln == 31) v = h.gamma * T[2] * T[8];
            if (FULL && c == C::TD && ln == 29) v = T[3];
        }
        sc[c][ln] = v;
    }
}

template <int N, bool FULL>
struct HalfOp {
    using C = HalfCf<N>;
    static constexpr int H = C::H, XT = N + H, S = XT + (FULL ? 1 : 0), NC = C::COUNT;
    static constexpr bool NAN_ENDS = false;
    const double (*sc)[32];
    DMat<N> D;
    double gg;   // g in the lanes of rho', 0 in those of w
    int ln;
    __device__ __forceinline__ void coefficients(double (&c)[NC]) const
    {
        int l = ln;   // laundered: read anew each time rather than kept in registers
        asm volatile("" : "+v"(l));
#pragma unroll
        for (int i = 0; i < (FULL ? C::COUNT : C::T1); ++i) c[i] = sc[i][l];
    }
    __device__ __forceinline__ void apply(const double (&x)[S], const double (&c)[NC], double (&y)[S]) const
    {
        const bool f1 = ln & 1, first = ln < 2, last = ln >= 30;
        double F[N + 1], d[N + 1], z[N];
#pragma unroll
        for (int l = 0; l < N; ++l) {
            const double th = l < H ? lane_move<kSwapPair>(x[N + (l < H ? l : 0)]) : x[N + (l < H ? 0 : l - H)];
            F[l] = c[C::C1 + l] * x[l] + c[C::C2 + l] * th;
        }
        // level 0 of the element above (the wave shift crosses into the other
        // column at the ends of a half: masked there)
        const double up = lane_move<kWaveShl1>(lane_move<kWaveShl1>(F[0]));
        F[N] = last ? 0.0 : up;
        if constexpr (FULL) F[N] += c[C::T1] * x[XT] + c[C::T2] * lane_move<kRowShr2>(x[XT]);
        D.contract(F, d);
        const double tN = c[C::WT] * d[N];
        const double dn = lane_move<kWaveShr1>(lane_move<kWaveShr1>(tN));
        z[0] = c[C::WB] * d[0] + (first ? 0.0 : dn) + gg * x[0];
#pragma unroll
        for (int l = 1; l < N; ++l) z[l] = c[C::H2] * d[l] + gg * x[l];
#pragma unroll
        for (int l = 0; l < N; ++l) y[l] = -c[C::CY + l] * lane_move<kSwapPair>(z[l]);
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const double wo = H + i < N ? lane_move<kSwapPair>(x[H + i < N ? H + i : 0]) : 0.0;
            y[N + i] = -c[C::DT + i] * (f1 ? wo : x[i]);
        }
        if constexpr (FULL) {
            // rho' row of the top level in lane 31, theta' row in lane 29, w row zero
            const double yr = lane_move<kSwapPair>(tN), yt = c[C::TD] * lane_move<kRowShl1>(x[XT]);
            y[XT] = ln == 31 ? -yr : -yt;
        }
    }
};

template <int N, bool FULL, int M, int VR>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1)))
gmres_half_kernel(const HeviParams h, const GmresArgs g, const int ngrp)
{
    using Op = HalfOp<N, FULL>;
    constexpr int H = Op::H, S = Op::S, XT = Op::XT, ML = M > VR ? M - VR : 0;
    __shared__ double sc[Op::NC][32];
    __shared__ double sx[S][64], sb[S][64];
    __shared__ double sv[ML ? ML * S : 1][64];
    __shared__ double sH[2][M * (M + 1)];
    const int lane = threadIdx.x, ln = lane % 32, half = lane / 32;
    const bool f1 = ln & 1;
    const int nz = h.nz;
    fill_half_coefficients<N, FULL>(h, sc);
    __syncthreads();
    const Op op{sc, DMat<N>(h.cst + kCstD), f1 ? h.g : 0.0, ln};
    const long nxy = (long)h.nx * h.ny, U = nxy * nz;
    for (GroupWalk walk(ngrp); walk.at < walk.end; walk.at += walk.step) {
        const long col = (long)walk.at * 2 + half;
        const bool have = col < nxy;
        int el = ln / 2;
        asm volatile("" : "+v"(el));
        // node of slot s, as in the one-lane form
        auto node = [&](int s, long &o5, long &o3) {
            int fld, k;   // fld: 0 rho', 1 w, 2 theta'
            bool ok;
            if (FULL && s == XT) {
                fld = 31 - ln;
                ok = fld < 3;
                fld = ok ? fld : 0;
                k = nz - 1;
            } else if (s < N) {
                fld = f1 ? 0 : 1;
                k = el * N + s;
                ok = k < nz;
            } else {
                const int l = s - N + (f1 ? H : 0);
                fld = 2;
                k = el * N + l;
                ok = l < N && k < nz;
            }
            const long o = (long)(k < nz ? k : nz - 1) * nxy + (have ? col : 0);
            o5 = (fld == 0 ? 0 : (fld + 2) * U) + o;
            o3 = fld * U + o;
            return ok && have;
        };
        double b2 = 0.0;
        {
            const double *x0 = g.x0 ? g.x0 : g.b;
            double bb[S], xx[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                long o5, o3;
                const bool ok = node(s, o5, o3);
                const double vb = g.b[o5], vx = x0[g.x0 ? o3 : o5];
                bb[s] = ok ? vb : 0.0;
                xx[s] = ok ? vx : 0.0;
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                sb[s][lane] = bb[s];
                sx[s][lane] = xx[s];
                b2 += bb[s] * bb[s];
            }
        }
        const double bn = sqrt(Half32::sum(b2));
        int iters = 0;
        bool conv = bn == 0.0;
        if (conv)
#pragma unroll
            for (int s = 0; s < S; ++s) sx[s][lane] = 0.0;
        const bool act = have && !conv;
        gmres_lanes<Half32, Op, M, VR>(op, g.alpha, g.rtol * bn, g.restart, g.max_restarts, act, sx, sb, sv,
                                       sH[half], conv, iters);
        asm volatile("" : "+v"(el));
#pragma unroll
        for (int s = 0; s < S; ++s) {
            long o5, o3;
            if (node(s, o5, o3)) g.x[o5] = sx[s][lane];
        }
        // u and v rows are the identity: lane f copies field 1 + f
        {
            const long fo = (f1 ? 2 : 1) * U + (have ? col : 0);
            double c[N + 1];
#pragma unroll
            for (int l = 0; l <= N; ++l) {
                const int k = el * N + l;
                c[l] = g.b[fo + (long)(k < nz ? k : nz - 1) * nxy];
            }
#pragma unroll
            for (int l = 0; l <= N; ++l) {
                const int k = el * N + l;
                if (have && k < nz && (l < N || (FULL && k == nz - 1))) g.x[fo + (long)k * nxy] = c[l];
            }
        }
        if (ln == 0 && have && g.iters) g.iters[col] = conv ? iters : -iters - 1;
        wave_sync();
    }
}

int wave_grid(int ngrp)
{
    return ngrp < 4096 ? (ngrp + kXcds - 1) / kXcds * kXcds : 4096;
}

template <int N, bool FULL>
void launch_forms(const HeviParams &h, const GmresArgs &g, hipStream_t s)
{
    // basis vectors kept in registers at order N (the rest in LDS): the most
    // that fit 512 registers without scratch; of the 20 of the half form 14
    // (orders 5 and 6 then spill 76 to 236 bytes a lane): 14 and 16 measured
    // alike at order 4 (3.41 ms per HEVI step, 2.84 now), 12 and 10 slower
    // (4.7: their LDS vectors leave three waves per CU instead of four)
    constexpr int VR = N <= 4 ? kGmresRegM : N == 5 ? 8 : 6;
    constexpr int VRH = 14;
    const long ncol = (long)h.nx * h.ny;
    const int n4 = (int)((ncol + 3) / 4), n2 = (int)((ncol + 1) / 2);
    const dim3 b(64);
    if (g.schur)
        hipLaunchKernelGGL((gmres_schur_elem_kernel<N, FULL, kGmresRegM>), dim3(wave_grid(n4)), b, 0, s, h, g, n4);
    else if (g.restart > kGmresRegM)
        hipLaunchKernelGGL((gmres_half_kernel<N, FULL, kGmresColM, VRH>), dim3(wave_grid(n2)), b, 0, s, h, g, n2);
    else
        hipLaunchKernelGGL((gmres_elem_kernel<N, FULL, kGmresRegM, VR>), dim3(wave_grid(n4)), b, 0, s, h, g, n4);
}

}  // namespace

// Which solves run here and which one column per wave (nh_hevi.hip).  A wave's
// time in this file hardly depends on how many of its lanes have an element,
// while the other forms get faster with fewer unknowns, and with a SIMD for
// every column there it is the length of one solve that counts, not the
// number of instructions.  So short columns and small lattices go there where
// that measured faster; times there / here on columns of 1 to 16 elements,
// 9 to 16384 columns, alpha 0.3 and 2, to 1e-8:
//   full form, restart 10 (registers there, 3 n_z <= 256): up to 1024 columns 0.95-0.99,
//     0.85-0.97, 0.77-0.9 and 0.68-0.99 at orders 2 to 5 up to the elements of the table
//     (1.0-1.2 above); up to 2048 columns 0.82-0.94 (order 4) and 0.85-0.96 (5) up to
//     half as many; with more 1.05-2.6.  Order 6: 0.61-0.95 up to 10 elements on any
//     lattice (1.0 at up to 2048 of them, 10 elements), 0.92-1.29 above.
//   restart 11 to 20: 1.0-5.5 while the lattice gives every wave slot one wave (four to a
//     CU, at orders 5 and 6 three); on more columns 0.49-0.95 with one element, 0.64-1.05 with two,
//     0.78-1.1 with three at restarts up to 16, and while few slots get a second wave
//     0.81-0.95 with three and four (1.4 at orders 5 and 6 from 2304 columns on); 1.0-8.7 above.
//   restart below 10: 1.05-11 but for order 6 on more than 2048 columns: 0.66-0.97 up to
//     three elements, 0.7-0.93 up to six at restarts 1 to 3.
//   Schur form: 1.0-4.4 but for order 6, up to 1024 columns of one or two elements: 0.9-0.99.
bool gmres_lanes_ok(const HeviParams &h, const GmresArgs &g)
{
    const int e = (h.nz - 1) / h.N, N = h.N;
    const long ncol = (long)h.nx * h.ny;
    if (e > kColElems || g.restart > kGmresColM) return false;
    if (g.schur) return !(N == 6 && e <= 2 && ncol <= 1024);
    if (g.restart > kGmresRegM)
        return ncol <= (N <= 4 ? 2048 : 1536) || e > (ncol <= 2304 ? 4 : ncol <= 3072 || g.restart <= 16 ? 3 : 2);
    if (g.restart < kGmresRegM) return N < 6 || ncol <= 2048 || e > (g.restart <= 3 ? 6 : 3);
    if (3 * h.nz > 64 * kGmresRegSlots) return true;
    if (N == 6) return e > 10;
    static const int few[6] = {0, 0, 8, 10, 6, 12};
    const int top = ncol <= 1024 ? few[N] : ncol <= 2048 && N >= 4 ? few[N] / 2 : 0;
    return e > top;
}

hipError_t launch_gmres_lanes(const HeviParams &h, const GmresArgs &g0, hipStream_t s)
{
    GmresArgs g = g0;
    g.pick = g0.restart == kGmresRegM && g0.pick;   // the choice of start is an option of restart 10
    const bool full = (h.nz - 1) / h.N == kColElems;
    switch (h.N) {
#define NH_COL(NN)                                      \
    case NN:                                            \
        if (full) launch_forms<NN, true>(h, g, s);      \
        else launch_forms<NN, false>(h, g, s);          \
        break;
        NH_COL(2) NH_COL(3) NH_COL(4) NH_COL(5) NH_COL(6)
#undef NH_COL
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace nh
