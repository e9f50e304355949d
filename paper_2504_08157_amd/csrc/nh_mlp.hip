// gfx950 kernels of the per-column MLP that predicts the initial guess of
// the HEVI column solves: feature extraction and resampling, FP16 MFMA
// forward GEMMs with FP32 accumulation, FP32 backward, Adam.
//
// Network: x (208: 198 features zero-padded) -> SiLU(W1 x + b1) (256)
//          -> SiLU(W2 h1 + b2) (256) -> y = W3 h2 + b3 + S x (256: 195 used),
// with a linear bypass S [256][208]: the exact map from the features to the
// correction is linear for a fixed column grid and alpha ((I - alpha L_v)^-1
// - I), the hidden layers carry its dependence on those.
// Features of a column with right-hand side b (fields rho', w, theta' on the
// n_z lattice levels): the default start x0 = b leaves the residual
// r = alpha L_v b, and the exact correction x - b = (I - alpha L_v)^-1 r is a
// linear function of r alone.  r is made dimensionless level by level
// (rho'/rho0, w/c0 with c0 = sqrt(gamma p0 / rho0), theta'/theta0), divided
// by one column scale s (RMS of the dimensionless r over the column's 3 n_z
// values) and resampled linearly in z to the 65 canonical levels (LGL nodes
// of 16 equal order-4 elements of the column): features 0 .. 194; then 3
// scalars (alpha / 10, 100 alpha c0(z_0) / H, log10 H / 5), zeros to 207.
// s itself is not a feature: the correction is homogeneous of degree one in
// r, so the map from r / s does not depend on s.  The correction is thus predicted
// relative to its own size, not to the size of b.
// Output: the dimensionless correction on the canonical levels,
// x0 = b + D s resample^-1(y), with the w correction zero on the walls.
#include "nh_internal.h"

#include <hip/hip_fp16.h>
#include <math.h>

namespace nh {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- features
// canonical level c of a column with lattice levels z[0..nz-1]: interval and weight
__device__ __forceinline__ void canon_interp(const double *z, int nz, double zc, int *k0, double *t)
{
    int lo = 0, hi = nz - 1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (z[mid] <= zc) lo = mid; else hi = mid;
    }
    *k0 = lo;
    *t = (zc - z[lo]) / (z[lo + 1] - z[lo]);
    if (*t < 0.0) *t = 0.0;
    if (*t > 1.0) *t = 1.0;
}

// Dimension factor of field f (0: rho', 1: w, 2: theta') at lattice level k.
__device__ __forceinline__ double dim_factor(const MlpColParams &p, int f, int k)
{
    const double *L = p.lev + (long)k * kLevW;
    if (f == 0) return L[0];
    if (f == 2) return L[1];
    return sqrt(p.gamma * L[2] / L[0]);
}

// 64 columns per workgroup of 512 threads: lane = column (every load reads
// 64 consecutive columns of one level, coalesced), the 8 waves split the
// levels of the scale sum and the canonical levels of the resampling; the
// features of the 64 columns are assembled in LDS and written out as whole
// rows.  The interpolation intervals of the canonical levels and the
// inverse dimension factors of every level are tabulated in LDS first
// (dynamic LDS: 3 n_z doubles).  The residual of the start is rscale * lb
// (fields 0, 3, 4 of [5][U]); the targets are the correction x - base of
// that start, base = b ([5][U]) or a previous guess ([3][U], base3).
__global__ void __launch_bounds__(512) mlp_features_kernel(MlpColParams p, const double *__restrict__ base,
                                                           bool base3, const double *__restrict__ lb,
                                                           double rscale, const double *__restrict__ x, long col0,
                                                           long ncol, _Float16 *__restrict__ feat,
                                                           double *__restrict__ scale, float *__restrict__ tgt)
{
    constexpr int NWV = 8;   // waves
    __shared__ _Float16 sf[64][kMlpIn];
    __shared__ double spart[NWV][64];
    __shared__ int sk0[kMlpNC];
    __shared__ double st[kMlpNC];
    extern __shared__ double sdinv[];   // [3][n_z]
    const int nz = p.nz;
    const long nxy = (long)p.nx * p.ny;
    const long U = nxy * nz;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int fld[3] = {0, 3, 4};
    const double H = p.z[nz - 1] - p.z[0];
    for (int i = threadIdx.x; i < 3 * nz; i += 64 * NWV) sdinv[i] = 1.0 / dim_factor(p, i / nz, i % nz);
    for (int c = threadIdx.x; c < kMlpNC; c += 64 * NWV)
        canon_interp(p.z, nz, p.z[0] + H * p.zc[c], &sk0[c], &st[c]);
    __syncthreads();
    const long r0 = (long)blockIdx.x * 64;
    const long r = r0 + lane;
    const bool ok = r < ncol;
    const long col = col0 + (ok ? r : 0);
    // s = RMS over the column of the dimensionless residual
    double a = 0.0;
#pragma unroll 4
    for (int k = q; k < nz; k += NWV) {
        const long I = col + (long)k * nxy;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const double l = rscale * lb[fld[f] * U + I] * sdinv[f * nz + k];
            a += l * l;
        }
    }
    spart[q][lane] = a;
    __syncthreads();
    double ssum = 0.0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) ssum += spart[w][lane];
    const double s = sqrt(ssum / (3.0 * nz)) + 1e-300;
#pragma unroll 3
    for (int c = q; c < kMlpNC; c += NWV) {
        const int k0 = sk0[c];
        const double t = st[c];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const long I0 = fld[f] * U + col + (long)k0 * nxy, I1 = I0 + nxy;
            const double d0 = sdinv[f * nz + k0], d1 = sdinv[f * nz + k0 + 1];
            const double vl = (1.0 - t) * (rscale * lb[I0] * d0) + t * (rscale * lb[I1] * d1);
            sf[lane][f * kMlpNC + c] = (_Float16)(vl / s);
            if (tgt && ok) {
                const long B0 = (base3 ? f : fld[f]) * U + col + (long)k0 * nxy, B1 = B0 + nxy;
                const double vx = (1.0 - t) * ((x[I0] - base[B0]) * d0) + t * ((x[I1] - base[B1]) * d1);
                tgt[r * kMlpOut + f * kMlpNC + c] = (float)(vx / s);
            }
        }
    }
    if (q == 0) {
        sf[lane][kMlpNF] = (_Float16)(p.alpha / 10.0);
        sf[lane][kMlpNF + 1] = (_Float16)(100.0 * p.alpha * dim_factor(p, 1, 0) / H);
        sf[lane][kMlpNF + 2] = (_Float16)(log10(H) / 5.0);
        for (int i = kMlpNF + 3; i < kMlpIn; ++i) sf[lane][i] = (_Float16)0.0f;
        if (ok) scale[r] = s;
    } else if (tgt && ok) {
        for (int i = kMlpNF + q - 1; i < kMlpOut; i += NWV - 1) tgt[r * kMlpOut + i] = 0.0f;
    }
    __syncthreads();
    // rows of 208 halves = 104 words; threads write consecutive words
    const long nrow = ncol - r0 < 64 ? ncol - r0 : 64;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(&sf[0][0]);
    uint32_t *dst = reinterpret_cast<uint32_t *>(feat + r0 * kMlpIn);
    for (long i = threadIdx.x; i < nrow * (kMlpIn / 2); i += 64 * NWV) dst[i] = src[i];
}

// x0 = b + D s (y resampled from the canonical to the lattice levels); the
// w correction is zero on the bottom and top levels, and a non-finite
// prediction falls back to x0 = b.  64 columns per workgroup of 512
// threads: the used outputs of the 64 rows of y are staged in LDS, lane =
// column (b reads and x0 writes coalesced), the 8 waves split the levels.
// Per-level tables (dynamic LDS: 4 n_z doubles and n_z ints): the canonical
// interval and weight of each lattice level and its dimension factors.
__global__ void __launch_bounds__(512) mlp_guess_kernel(MlpColParams p, const double *__restrict__ b, long col0,
                                                        long ncol, const float *__restrict__ y,
                                                        const double *__restrict__ scale, double *__restrict__ x0)
{
    __shared__ float sy[64][kMlpNF + 1];
    extern __shared__ double sg[];
    const int nz = p.nz;
    double *tg = sg;              // [n_z] interpolation weight
    double *dg = sg + nz;         // [3][n_z] dimension factors
    int *lg = (int *)(sg + 4 * nz);   // [n_z] canonical interval
    const long nxy = (long)p.nx * p.ny;
    const long U = nxy * nz;
    const int fld[3] = {0, 3, 4};
    const double H = p.z[nz - 1] - p.z[0];
    for (int k = threadIdx.x; k < nz; k += 512) {
        const double zh = (p.z[k] - p.z[0]) / H;
        int lo = 0, hi = kMlpNC - 1;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (p.zc[mid] <= zh) lo = mid; else hi = mid;
        }
        double t = (zh - p.zc[lo]) / (p.zc[lo + 1] - p.zc[lo]);
        if (t < 0.0) t = 0.0;
        if (t > 1.0) t = 1.0;
        lg[k] = lo;
        tg[k] = t;
        for (int f = 0; f < 3; ++f) dg[f * nz + k] = dim_factor(p, f, k);
    }
    const long r0 = (long)blockIdx.x * 64;
    const long nrow = ncol - r0 < 64 ? ncol - r0 : 64;
    for (long i = threadIdx.x; i < nrow * kMlpNF; i += 512) {
        const long rr = i / kMlpNF;
        const int c = (int)(i - rr * kMlpNF);
        sy[rr][c] = y[(r0 + rr) * kMlpOut + c];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    if (lane >= nrow) return;
    const long r = r0 + lane;
    const double s = scale[r];
#pragma unroll 2
    for (int k = q; k < nz; k += 8) {
        const long I = col0 + r + (long)k * nxy;
        const int lo = lg[k];
        const double t = tg[k];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const float *yr = &sy[lane][f * kMlpNC];
            double d = (1.0 - t) * yr[lo] + t * yr[lo + 1];
            if (!isfinite(d) || (f == 1 && (k == 0 || k == nz - 1))) d = 0.0;
            x0[f * U + I] = b[fld[f] * U + I] + dg[f * nz + k] * s * d;
        }
    }
}

// acc += A B^T over one 32-wide k slice held as 8 halves per lane, as two
// v_mfma_f32_16x16x16_f16 (halves 0-3, then 4-7 of both operands: the same
// k values pair up).  The single-instruction v_mfma_f32_16x16x32_f16 form
// gave run-to-run different results in the fused inference kernel although
// its LDS accesses are race-free between barriers; that build spills MFMA
// operands and rewrites their registers right behind the instruction, so
// it is not used.
__device__ __forceinline__ float4v mfma_k32(const half8 &a, const half8 &b, float4v c)
{
    const half4 al = {a[0], a[1], a[2], a[3]}, ah = {a[4], a[5], a[6], a[7]};
    const half4 bl = {b[0], b[1], b[2], b[3]}, bh = {b[4], b[5], b[6], b[7]};
    c = __builtin_amdgcn_mfma_f32_16x16x16f16(al, bl, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16f16(ah, bh, c, 0, 0, 0);
}

// ---------------------------------------------------------------- forward GEMM (MFMA)
// C[M x 256] = A[M x K] W[256 x K]^T (+ A2[M x K2] W2[256 x K2]^T) + bias,
// FP16 operands, FP32 accumulation on v_mfma_f32_16x16x16_f16 (two per
// 32-wide K slice, one for a 16-wide remainder).  Workgroup: 64 rows and all 256
// outputs, 4 waves (wave w: outputs 64 w .. 64 w + 63, 4 x 4 MFMA tiles).
// The K loop stages 32-wide slices of A (64 x 32, shared by the 4 waves) in
// LDS; each wave loads its own W fragments straight from memory (W is a
// few hundred KB and stays in L2).  The next slice of both is loaded into
// registers while the current one is multiplied.  A lane's A and B operands
// hold the same 8 (or 4) k values, so the pairing inside the instruction is
// consistent.  The optional second product (the linear bypass of the last
// layer) is accumulated first, into the same registers.  Epilogue: Z (FP32
// pre-activation, skipped when null) and, when act != 0, H = SiLU(Z) in
// FP16.  Requires M % 64 == 0, K % 16 == 0, K2 % 16 == 0.
__global__ void __launch_bounds__(256) gemm_rows_kernel(const _Float16 *__restrict__ A,
                                                        const _Float16 *__restrict__ W,
                                                        const float *__restrict__ bias, int K,
                                                        const _Float16 *__restrict__ A2,
                                                        const _Float16 *__restrict__ W2, int K2,
                                                        float *__restrict__ Z, _Float16 *__restrict__ Hout, int act)
{
    __shared__ half8 sA[64 * 4];    // [row][k octet]
    half4 *sA4 = reinterpret_cast<half4 *>(sA);
    const int t = threadIdx.x, wave = t / 64, lane = t % 64;
    const long m0 = (long)blockIdx.x * 64;
    const int r16 = lane % 16, g = lane / 16;
    float4v acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = float4v{0.f, 0.f, 0.f, 0.f};

    auto run = [&](const _Float16 *Ap, const _Float16 *Wp, int KK) {
        const int K32 = KK & ~31;
        // thread t stages octet t % 4 of A row t / 4; lane (r16, g) of wave w
        // reads k octet g of W rows 64 w + 16 c + r16
        const _Float16 *ga = Ap + (m0 + t / 4) * KK + (t % 4) * 8;
        const _Float16 *gw = Wp + (long)(64 * wave + r16) * KK + 8 * g;
        if (K32 > 0) {
            half8 ra = *(const half8 *)ga;
            half8 bv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) bv[c] = *(const half8 *)(gw + (long)16 * c * KK);
            for (int k = 0; k < K32; k += 32) {
                __syncthreads();   // the previous slice has been read
                sA[t] = ra;
                __syncthreads();
                half8 bn[4];
                if (k + 32 < K32) {
                    ra = *(const half8 *)(ga + k + 32);
#pragma unroll
                    for (int c = 0; c < 4; ++c) bn[c] = *(const half8 *)(gw + (long)16 * c * KK + k + 32);
                }
                half8 av[4];
#pragma unroll
                for (int a = 0; a < 4; ++a) av[a] = sA[(16 * a + r16) * 4 + g];
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[a][c] = mfma_k32(av[a], bv[c], acc[a][c]);
                if (k + 32 < K32)
#pragma unroll
                    for (int c = 0; c < 4; ++c) bv[c] = bn[c];
            }
        }
        if (KK > K32) {
            // 16-wide remainder: quads instead of octets
            const half4 ra = *(const half4 *)(Ap + (m0 + t / 4) * KK + K32 + (t % 4) * 4);
            const _Float16 *gw4 = Wp + (long)(64 * wave + r16) * KK + K32 + 4 * g;
            half4 bv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) bv[c] = *(const half4 *)(gw4 + (long)16 * c * KK);
            __syncthreads();
            sA4[t] = ra;
            __syncthreads();
            half4 av[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) av[a] = sA4[(16 * a + r16) * 4 + g];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(av[a], bv[c], acc[a][c], 0, 0, 0);
        }
    };
    // the bypass product first (the fused inference kernel accumulates in
    // the same order)
    if (A2) run(A2, W2, K2);
    run(A, W, K);

    // output layout: lane holds rows 4 (lane / 16) + i, column lane % 16 of each 16 x 16 tile
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long row = m0 + 16 * a + 4 * g + i;
                const int col = 64 * wave + 16 * c + r16;
                const float z = acc[a][c][i] + bias[col];
                if (Z) Z[row * 256 + col] = z;
                if (act) Hout[row * 256 + col] = (_Float16)(z / (1.0f + expf(-z)));
            }
}

// ---------------------------------------------------------------- fused inference
// The guess x0 of 64 columns per workgroup of 512 threads (8 waves) with
// everything between the right-hand side and x0 kept in LDS: the features
// of the 64 columns (computed as in mlp_features_kernel), the three layers
// on v_mfma_f32_16x16x16_f16 with the A operands read from LDS (wave w:
// outputs 32 w .. 32 w + 31 of the 64 rows; W fragments from memory, where
// they stay L2 resident), and the resampling of the output to the lattice
// levels (as in mlp_guess_kernel).  Layer 1 and the linear bypass share one
// pass over the features, after which one LDS region holds in turn the
// features, H1, H2 and the output rows (about 58 KB per workgroup, two
// workgroups per CU).  The MFMA operands and the order of accumulation are
// those of gemm_rows_kernel, so the guess equals that of the separate
// kernels.
constexpr int kLdF = kMlpIn + 8;    // LDS row of the features (halves), padded
constexpr int kLdH = kMlpHid + 8;   // LDS row of the activations (halves), padded
// the shared region: features, then H1, H2, output rows (the largest)
constexpr int kRegBytes = 64 * (kMlpNF + 1) * 4;
static_assert(64 * kLdF * 2 <= kRegBytes && 64 * kLdH * 2 <= kRegBytes && kRegBytes % 16 == 0, "region sizes");

// x0 = base + D s (network of the residual r of the start base,
// dimensionless) per column: base is b ([5][U], fields 0, 3, 4), whose
// residual is r = alpha L_v b (first pass), or the previous guess ([3][U],
// base3), whose residual is r = b - base + alpha L_v base (refinement pass).
// NV = 0: r is read from lb (fields 0, 3, 4 of [5][U]) times rscale.
// NV = N > 0: r is computed here -- each wave walks a contiguous chunk of the
// column's levels with lv_walk -- and kept dimensionless as FP32 rows
// [3][n_z][64] in the shared region until the resampling (n_z <= 65, the
// region's size).  x0 may be base (each element is read before it is
// written, by the same thread; the walk only reads the workgroup's own
// columns).
constexpr int kMlpFusedNz = kRegBytes / (3 * 64 * 4);

template <int NV>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) mlp_infer_kernel(MlpColParams p, HeviParams hp,
                                                        MlpWeights wt, const double *base, bool base3,
                                                        const double *b, const double *lb, double rscale, long col0,
                                                        long ncol, double *x0)
{
    constexpr int NWV = 8;
    __shared__ __align__(16) unsigned char sreg[kRegBytes];
    _Float16 *sf = reinterpret_cast<_Float16 *>(sreg);   // features [64][kLdF]
    _Float16 *sh = reinterpret_cast<_Float16 *>(sreg);   // H1, then H2 [64][kLdH]
    __shared__ double spart[NWV][64];
    __shared__ double sscale[64];
    __shared__ int sk0[kMlpNC];
    __shared__ double st[kMlpNC];
    extern __shared__ double stab[];
    const int nz = p.nz;
    double *sdinv = stab;              // [3][n_z] inverse dimension factors
    double *dg = stab + 3 * nz;        // [3][n_z] dimension factors
    double *tg = stab + 6 * nz;        // [n_z] canonical weight of each lattice level
    int *lg = (int *)(stab + 7 * nz);  // [n_z] canonical interval of each lattice level
    float *sy = reinterpret_cast<float *>(sreg);   // [64][kMlpNF + 1] outputs, after the last layer

    const long nxy = (long)p.nx * p.ny;
    const long U = nxy * nz;
    const int tid = threadIdx.x, lane = tid & 63, q = tid >> 6;
    const int fld[3] = {0, 3, 4};
    const double H = p.z[nz - 1] - p.z[0];

    // ---- tables
    for (int i = tid; i < 3 * nz; i += 64 * NWV) {
        sdinv[i] = 1.0 / dim_factor(p, i / nz, i % nz);
        dg[i] = dim_factor(p, i / nz, i % nz);
    }
    for (int c = tid; c < kMlpNC; c += 64 * NWV) canon_interp(p.z, nz, p.z[0] + H * p.zc[c], &sk0[c], &st[c]);
    for (int k = tid; k < nz; k += 64 * NWV) {
        const double zh = (p.z[k] - p.z[0]) / H;
        int lo = 0, hi = kMlpNC - 1;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (p.zc[mid] <= zh) lo = mid; else hi = mid;
        }
        double t = (zh - p.zc[lo]) / (p.zc[lo + 1] - p.zc[lo]);
        if (t < 0.0) t = 0.0;
        if (t > 1.0) t = 1.0;
        lg[k] = lo;
        tg[k] = t;
    }
    __syncthreads();

    // ---- features (lane = column, the waves split the levels)
    const long r0 = (long)blockIdx.x * 64;
    const long nrow = ncol - r0 < 64 ? ncol - r0 : 64;
    const long r = r0 + lane;
    const long col = col0 + (lane < nrow ? r : r0);
    float *rbuf = reinterpret_cast<float *>(sreg);   // NV > 0: residual rows [3][n_z][64]
    {
        double a = 0.0;
        if constexpr (NV > 0) {
            auto resid = [&](int k, double l0, double l3, double l4, double xr, double xw, double xt) {
                const long I = col + (long)k * nxy;
                double v[3] = {p.alpha * l0, p.alpha * l3, p.alpha * l4};
                if (base3) {
                    v[0] = b[I] - xr + v[0];
                    v[1] = b[3 * U + I] - xw + v[1];
                    v[2] = b[4 * U + I] - xt + v[2];
                }
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const double d = v[f] * sdinv[f * nz + k];
                    rbuf[(f * nz + k) * 64 + lane] = (float)d;
                    a += d * d;
                }
            };
            // a contiguous chunk of levels per wave, walked with a window
            // (computing each level from its own 2N+1 neighbours instead
            // measured slower: 0.57 against 0.38 ms per pass)
            const long xw = base3 ? U : 3 * U, xt = base3 ? 2 * U : 4 * U;
            const int chunk = (nz + NWV - 1) / NWV;
            const int ka = q * chunk, kb = min(nz, ka + chunk);
            if (ka < kb) lv_walk<NV>(hp, col, ka, kb, base, xw, xt, resid);
        } else {
#pragma unroll 4
            for (int k = q; k < nz; k += NWV) {
                const long I = col + (long)k * nxy;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const double l = rscale * lb[fld[f] * U + I] * sdinv[f * nz + k];
                    a += l * l;
                }
            }
        }
        spart[q][lane] = a;
    }
    __syncthreads();
    double ssum = 0.0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) ssum += spart[w][lane];
    const double s = sqrt(ssum / (3.0 * nz)) + 1e-300;
    _Float16 *fr = sf + lane * kLdF;
    if constexpr (NV > 0) {
        // canonical levels c = q, q + 8, ... of this lane's column from the
        // residual rows, held in registers until every wave has read them
        constexpr int NCW = (kMlpNC + NWV - 1) / NWV;
        _Float16 hv[NCW][3];
#pragma unroll
        for (int j = 0; j < NCW; ++j) {
            const int c = q + j * NWV;
            if (c < kMlpNC) {
                const int k0 = sk0[c];
                const double t = st[c];
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const double v0 = rbuf[(f * nz + k0) * 64 + lane], v1 = rbuf[(f * nz + k0 + 1) * 64 + lane];
                    hv[j][f] = (_Float16)(((1.0 - t) * v0 + t * v1) / s);
                }
            }
        }
        __syncthreads();   // every wave has read the residual rows
#pragma unroll
        for (int j = 0; j < NCW; ++j) {
            const int c = q + j * NWV;
            if (c < kMlpNC)
#pragma unroll
                for (int f = 0; f < 3; ++f) fr[f * kMlpNC + c] = hv[j][f];
        }
    } else {
#pragma unroll 3
        for (int c = q; c < kMlpNC; c += NWV) {
            const int k0 = sk0[c];
            const double t = st[c];
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                const long I0 = fld[f] * U + col + (long)k0 * nxy, I1 = I0 + nxy;
                const double d0 = sdinv[f * nz + k0], d1 = sdinv[f * nz + k0 + 1];
                const double vl = (1.0 - t) * (rscale * lb[I0] * d0) + t * (rscale * lb[I1] * d1);
                fr[f * kMlpNC + c] = (_Float16)(vl / s);
            }
        }
    }
    if (q == 0) {
        fr[kMlpNF] = (_Float16)(p.alpha / 10.0);
        fr[kMlpNF + 1] = (_Float16)(100.0 * p.alpha * dim_factor(p, 1, 0) / H);
        fr[kMlpNF + 2] = (_Float16)(log10(H) / 5.0);
        for (int i = kMlpNF + 3; i < kMlpIn; ++i) fr[i] = (_Float16)0.0f;
        sscale[lane] = s;
    }
    __syncthreads();

    // ---- layers
    const int wave = q, r16 = lane % 16, g = lane / 16;
    float4v acc[4][2], acc3[4][2];   // current layer; last layer (bypass first)
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            acc[a][c] = float4v{0.f, 0.f, 0.f, 0.f};
            acc3[a][c] = float4v{0.f, 0.f, 0.f, 0.f};
        }
    // C += S[64 x KK] (LDS, row stride ld) Wp[32 w .. 32 w + 31][KK]^T for
    // up to two (W, C) pairs sharing the A fragments
    auto mma = [&](const _Float16 *S, int ld, int KK, const _Float16 *Wa, float4v (&Ca)[4][2],
                   const _Float16 *Wb, float4v (&Cb)[4][2]) __attribute__((always_inline)) {
        const int K32 = KK & ~31;
        const long wrow = (long)(32 * wave + r16) * KK;
        if (K32 > 0) {
            half8 ba[2], bb[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                ba[c] = *(const half8 *)(Wa + wrow + (long)16 * c * KK + 8 * g);
                if (Wb) bb[c] = *(const half8 *)(Wb + wrow + (long)16 * c * KK + 8 * g);
            }
#pragma unroll 1
            for (int k = 0; k < K32; k += 32) {
                half8 na[2], nb[2];
                if (k + 32 < K32)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        na[c] = *(const half8 *)(Wa + wrow + (long)16 * c * KK + k + 32 + 8 * g);
                        if (Wb) nb[c] = *(const half8 *)(Wb + wrow + (long)16 * c * KK + k + 32 + 8 * g);
                    }
                half8 av[4];
#pragma unroll
                for (int a = 0; a < 4; ++a) av[a] = *(const half8 *)(S + (16 * a + r16) * ld + k + 8 * g);
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        Ca[a][c] = mfma_k32(av[a], ba[c], Ca[a][c]);
                        if (Wb) Cb[a][c] = mfma_k32(av[a], bb[c], Cb[a][c]);
                    }
                if (k + 32 < K32)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        ba[c] = na[c];
                        if (Wb) bb[c] = nb[c];
                    }
            }
        }
        if (KK > K32) {
            half4 ba[2], bb[2], av[4];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                ba[c] = *(const half4 *)(Wa + wrow + (long)16 * c * KK + K32 + 4 * g);
                if (Wb) bb[c] = *(const half4 *)(Wb + wrow + (long)16 * c * KK + K32 + 4 * g);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) av[a] = *(const half4 *)(S + (16 * a + r16) * ld + K32 + 4 * g);
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    Ca[a][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(av[a], ba[c], Ca[a][c], 0, 0, 0);
                    if (Wb) Cb[a][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(av[a], bb[c], Cb[a][c], 0, 0, 0);
                }
        }
    };
    // H = SiLU(acc + bias) into the activation rows (lane: rows 4 g + i,
    // column r16 of each tile); acc is cleared for the next layer
    auto store_h = [&](const float *bias) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 16 * a + 4 * g + i, cl = 32 * wave + 16 * c + r16;
                    const float z = acc[a][c][i] + bias[cl];
                    sh[row * kLdH + cl] = (_Float16)(z / (1.0f + expf(-z)));
                }
                acc[a][c] = float4v{0.f, 0.f, 0.f, 0.f};
            }
    };
    // layer 1 and the bypass of the last layer: one pass over the features
    mma(sf, kLdF, kMlpIn, wt.W[3], acc3, wt.W[0], acc);
    __syncthreads();   // every wave has read the features
    store_h(wt.bias[0]);
    __syncthreads();
    mma(sh, kLdH, kMlpHid, wt.W[1], acc, nullptr, acc);
    __syncthreads();   // every wave has read H1
    store_h(wt.bias[1]);
    __syncthreads();
    mma(sh, kLdH, kMlpHid, wt.W[2], acc3, nullptr, acc3);
    __syncthreads();   // every wave has read H2
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * a + 4 * g + i, cl = 32 * wave + 16 * c + r16;
                if (cl < kMlpNF) sy[row * (kMlpNF + 1) + cl] = acc3[a][c][i] + wt.bias[2][cl];
            }
    __syncthreads();

    // ---- resampling to the lattice levels (lane = column, the waves split the levels)
    if (lane >= nrow) return;
    const double sc = sscale[lane];
#pragma unroll 2
    for (int k = q; k < nz; k += NWV) {
        const long I = col0 + r + (long)k * nxy;
        const int lo = lg[k];
        const double t = tg[k];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const float *yr = sy + lane * (kMlpNF + 1) + f * kMlpNC;
            double d = (1.0 - t) * yr[lo] + t * yr[lo + 1];
            if (!isfinite(d) || (f == 1 && (k == 0 || k == nz - 1))) d = 0.0;
            x0[f * U + I] = base[(base3 ? f : fld[f]) * U + I] + dg[f * nz + k] * sc * d;
        }
    }
}

// ---------------------------------------------------------------- training, row part
// Everything of a training step that is local to a batch row, for R rows per
// workgroup of 8 waves: the three layers (FWD; FP16 MFMA, the operands and the
// order of accumulation of gemm_rows_kernel), the gradient of the mean squared
// error dY = 2 (Y - T) / n with a loss partial per workgroup, and the chain
//   dZ2 = (dY W3) SiLU'(Z2),   dZ1 = (dZ2 W2) SiLU'(Z1)
// on v_mfma_f32_16x16x4_f32 (FP32 products and accumulation).  Without FWD
// (nh_mlp_backward) dY, Z1 and Z2 are read instead of computed.  Written for the
// weight gradients and for a later nh_mlp_backward: Z1, Z2, H1, H2, dY, dZ2,
// dZ1.  Row tiles stay in LDS from layer to layer; wave w owns output columns
// 32 w .. 32 w + 31, lane r16 of column tile c the column 32 w + 2 r16 + c, so that
// a lane's two columns are one 8-byte access and the weights of the backward
// products, stored with that index fastest, are read in pairs.  A wave loads a
// layer's whole weight strip into registers (64 VGPRs) before it multiplies:
// one exposed L2 latency per layer.
// Bound: the FP32 products, 2 x 256 x 256 x 2 flops per row (13.7 us for 8192 rows
// at the 157 TFLOP/s of the FP32 matrix units), and the layer-by-layer chain of two
// waves per SIMD around them: 56 us for 8192 rows, where the separate products, SiLU
// gradients and loss took 190 us (a training step of 8192 rows: 532 us before, 104 now).
constexpr int kTrX = kMlpIn + 8;    // LDS row of the features (halves)
constexpr int kTrH = kMlpHid + 8;   // LDS row of the activations (halves)
constexpr int kTrD = kMlpHid + 4;   // LDS row of the FP32 gradients

// a caller's targets and output gradients are aligned to their elements only
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

struct TrainRows {
    const _Float16 *X;                       // [M][kMlpIn]
    const float *T;                          // [M][kMlpOut] targets (FWD)
    MlpWeights wt;
    float *Z1, *Z2, *dY, *dZ2, *dZ1;         // [M][256]
    _Float16 *H1, *H2;                       // [M][256]
    const float *dYin;                       // the caller's dY (without FWD)
    float *part;                             // [workgroups] loss partials (FWD)
    float scale;                             // 1 / n of the loss
};

__device__ __forceinline__ float silu_grad(float z)
{
    const float sg = 1.f / (1.f + expf(-z));
    return sg * (1.f + z * (1.f - sg));
}

template <int R, bool FWD>
__global__ void __launch_bounds__(512) mlp_train_rows_kernel(const TrainRows p)
{
    static_assert(kMlpHid == 256 && kMlpOut == 256 && (R == 16 || R == 32), "8 waves x 32 columns");
    constexpr int RA = R / 16;
    __shared__ __align__(16) _Float16 sX[FWD ? R * kTrX : 8];
    __shared__ __align__(16) _Float16 sH[FWD ? R * kTrH : 8];
    __shared__ __align__(16) float sD[R * kTrD];
    __shared__ float sloss[8];
    const int t = threadIdx.x, wave = t / 64, lane = t % 64, r16 = lane % 16, g = lane / 16;
    const long m0 = (long)blockIdx.x * R;
    const int n0 = 32 * wave + 2 * r16;   // the lane's columns n0, n0 + 1

    float z1[RA][2][4], z2[RA][2][4];
    if constexpr (FWD) {
        for (int i = t; i < R * (kMlpIn / 8); i += 512) {
            const int r = i / (kMlpIn / 8), o = i % (kMlpIn / 8);
            *(half8 *)(sX + r * kTrX + 8 * o) = *(const half8 *)(p.X + (m0 + r) * kMlpIn + 8 * o);
        }
        // weight strip of the wave: rows n0, n0 + 1 of W [256][KK]
        constexpr int KX = kMlpIn / 32, KH = kMlpHid / 32;
        static_assert(kMlpIn % 32 == 16 && kMlpHid % 32 == 0, "one 16-wide remainder in the feature layers");
        auto load_h = [&](const _Float16 *W, half8 (&w8)[KH][2]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < KH; ++k)
#pragma unroll
                for (int c = 0; c < 2; ++c) w8[k][c] = *(const half8 *)(W + (long)(n0 + c) * kMlpHid + 32 * k + 8 * g);
        };
        auto load_x = [&](const _Float16 *W, half8 (&w8)[KX][2], half4 (&w4)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int k = 0; k < KX; ++k) w8[k][c] = *(const half8 *)(W + (long)(n0 + c) * kMlpIn + 32 * k + 8 * g);
                w4[c] = *(const half4 *)(W + (long)(n0 + c) * kMlpIn + 32 * KX + 4 * g);
            }
        };
        auto mul_x = [&](const half8 (&w8)[KX][2], const half4 (&w4)[2], float4v (&acc)[RA][2])
                         __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < KX; ++k)
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    const half8 av = *(const half8 *)(sX + (16 * a + r16) * kTrX + 32 * k + 8 * g);
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[a][c] = mfma_k32(av, w8[k][c], acc[a][c]);
                }
#pragma unroll
            for (int a = 0; a < RA; ++a) {
                const half4 av = *(const half4 *)(sX + (16 * a + r16) * kTrX + 32 * KX + 4 * g);
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(av, w4[c], acc[a][c], 0, 0, 0);
            }
        };
        auto mul_h = [&](const half8 (&w8)[KH][2], float4v (&acc)[RA][2]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < KH; ++k)
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    const half8 av = *(const half8 *)(sH + (16 * a + r16) * kTrH + 32 * k + 8 * g);
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[a][c] = mfma_k32(av, w8[k][c], acc[a][c]);
                }
        };
        auto clear = [&](float4v (&acc)[RA][2]) __attribute__((always_inline)) {
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[a][c] = float4v{0.f, 0.f, 0.f, 0.f};
        };
        // z = acc + bias to registers and memory, SiLU(z) to LDS and memory
        auto layer_out = [&](const float4v (&acc)[RA][2], const float *bias, float (&z)[RA][2][4], float *Z,
                             _Float16 *Hg) __attribute__((always_inline)) {
            const float b0 = bias[n0], b1 = bias[n0 + 1];
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 16 * a + 4 * g + i;
                    const float u = acc[a][0][i] + b0, v = acc[a][1][i] + b1;
                    z[a][0][i] = u;
                    z[a][1][i] = v;
                    *(float2 *)(Z + (m0 + row) * 256 + n0) = make_float2(u, v);
                    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
                    const half2v h = {(_Float16)(u / (1.0f + expf(-u))), (_Float16)(v / (1.0f + expf(-v)))};
                    *(half2v *)(sH + row * kTrH + n0) = h;
                    *(half2v *)(Hg + (m0 + row) * 256 + n0) = h;
                }
        };
        float4v acc[RA][2], acc3[RA][2];
        clear(acc);
        clear(acc3);
        half8 wa[KX][2], wb[KX][2], wh[KH][2];
        half4 wa4[2], wb4[2];
        load_x(p.wt.W[0], wa, wa4);
        load_x(p.wt.W[3], wb, wb4);
        __syncthreads();
        mul_x(wa, wa4, acc);
        load_h(p.wt.W[1], wh);
        mul_x(wb, wb4, acc3);   // the bypass is accumulated first
        layer_out(acc, p.wt.bias[0], z1, p.Z1, p.H1);
        __syncthreads();
        clear(acc);
        mul_h(wh, acc);
        load_h(p.wt.W[2], wh);
        __syncthreads();        // every wave has read H1
        layer_out(acc, p.wt.bias[1], z2, p.Z2, p.H2);
        __syncthreads();
        mul_h(wh, acc3);
        float loss = 0.f;
        {
            const float b0 = p.wt.bias[2][n0], b1 = p.wt.bias[2][n0 + 1];
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 16 * a + 4 * g + i;
                    const float2u tt = *(const float2u *)(p.T + (m0 + row) * 256 + n0);
                    const float d0 = (acc3[a][0][i] + b0) - tt.x, d1 = (acc3[a][1][i] + b1) - tt.y;
                    loss += d0 * d0 + d1 * d1;
                    const float2 dy = make_float2(2.f * d0 * p.scale, 2.f * d1 * p.scale);
                    *(float2 *)(sD + row * kTrD + n0) = dy;
                    *(float2 *)(p.dY + (m0 + row) * 256 + n0) = dy;
                }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o);
        if (lane == 0) sloss[wave] = loss;
        __syncthreads();
        if (t == 0) {
            float l = 0.f;
#pragma unroll
            for (int w = 0; w < 8; ++w) l += sloss[w];
            p.part[blockIdx.x] = l;
        }
    } else {
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * a + 4 * g + i;
                const long o = (m0 + row) * 256 + n0;
                const float2 u = *(const float2 *)(p.Z1 + o), v = *(const float2 *)(p.Z2 + o);
                z1[a][0][i] = u.x;
                z1[a][1][i] = u.y;
                z2[a][0][i] = v.x;
                z2[a][1][i] = v.y;
                const float2u dy = *(const float2u *)(p.dYin + o);
                *(float2 *)(sD + row * kTrD + n0) = make_float2(dy.x, dy.y);
            }
        __syncthreads();
    }

    // acc[m][n] = sum_k sD[m][k] W[k][n], W [256][256] FP16 with n fastest: in
    // each block of 16 k, lane quarter g holds k = 4 g + i for the i-th product
    // (the same k in both operands)
    auto chain = [&](const _Float16 *W, float4v (&acc)[RA][2]) __attribute__((always_inline)) {
        typedef _Float16 half2v __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int c = 0; c < 2; ++c) acc[a][c] = float4v{0.f, 0.f, 0.f, 0.f};
        constexpr int KB = 8;   // blocks of 16 k whose weights are in registers at a time
        half2v w[KB][4];
        auto load = [&](int kb0) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    w[b][i] = *(const half2v *)(W + (long)(16 * (kb0 + b) + 4 * g + i) * 256 + n0);
        };
        load(0);
#pragma unroll
        for (int kb0 = 0; kb0 < 16; kb0 += KB) {
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float4v av[RA];
#pragma unroll
                for (int a = 0; a < RA; ++a)
                    av[a] = *(const float4v *)(sD + (16 * a + r16) * kTrD + 16 * (kb0 + b) + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int a = 0; a < RA; ++a)
                            acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a][i], (float)w[b][i][c], acc[a][c],
                                                                             0, 0, 0);
            }
            if (kb0 + KB < 16) load(kb0 + KB);
        }
    };
    float4v d[RA][2];
    chain(p.wt.W[2], d);
    __syncthreads();   // every wave has read dY
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 16 * a + 4 * g + i;
            const float2 dz = make_float2(d[a][0][i] * silu_grad(z2[a][0][i]), d[a][1][i] * silu_grad(z2[a][1][i]));
            *(float2 *)(sD + row * kTrD + n0) = dz;
            *(float2 *)(p.dZ2 + (m0 + row) * 256 + n0) = dz;
        }
    __syncthreads();
    chain(p.wt.W[1], d);
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 16 * a + 4 * g + i;
            *(float2 *)(p.dZ1 + (m0 + row) * 256 + n0) =
                make_float2(d[a][0][i] * silu_grad(z1[a][0][i]), d[a][1][i] * silu_grad(z1[a][1][i]));
        }
}

// ---------------------------------------------------------------- training, batch sums
// The four weight gradients and three bias gradients in one launch:
//   dS = dY^T X, dW3 = dY^T H2, dW2 = dZ2^T H1, dW1 = dZ1^T X, db = column sums,
// FP32 products and accumulation on v_mfma_f32_16x16x4_f32 (lane l: A row l % 16 and
// B column l % 16 at k = l / 16).  Workgroup: a 64 x 64 tile of one gradient over
// one slice of the batch, 4 waves of 2 x 2 MFMA tiles; chunks of 32 batch rows go
// through LDS as FP32, the next chunk in registers during the products; rows of
// kBkLd floats so that the four k rows a wave reads fall in distinct banks.
// The workgroups of a gradient's first column tile also sum the columns of A.
// Slice z writes its share of the whole gradient vector to part + z nparam;
// train_update_kernel adds the slices in order (deterministic).
// One launch instead of four (and no separate column sums) keeps up to 1024
// workgroups in flight, four to a CU, which is what hides the staging latency.
// 3.9 GFLOP at 8192 rows, 25 us at 157 TFLOP/s: 48 us measured (seven launches with
// their sums and the column sums took 330 us).
constexpr int kBkK = 32, kBkLd = 80;
constexpr int kGradTiles = 4 * 16;   // 4 x 4 tiles of 64 x 64 per gradient (the last column tile of 208 is partial)

struct GradJob {
    const float *A;        // [M][256]
    const _Float16 *B;     // [M][No]
    int No;
    long off, boff;        // offsets of the gradient and of the bias gradient (-1: none) in the parameter vector
};
struct GradJobs {
    GradJob j[4];
};

__global__ void __launch_bounds__(256) mlp_grads_kernel(const GradJobs jobs, int M, int kslice, long nparam,
                                                        float *__restrict__ part)
{
    __shared__ __align__(16) float As[kBkK][kBkLd];
    __shared__ __align__(16) float Bs[kBkK][kBkLd];
    const int t = threadIdx.x, wave = t / 64, lane = t % 64, r16 = lane % 16, kq = lane / 16;
    const GradJob J = jobs.j[blockIdx.x / 16];
    const int m0 = 64 * ((blockIdx.x % 16) / 4), n0 = 64 * (blockIdx.x % 4);
    const int kb = blockIdx.y * kslice, ke = min(M, kb + kslice);   // kslice and M are multiples of 32
    float *out = part + (long)blockIdx.y * nparam;
    const int wm = 32 * (wave / 2), wn = 32 * (wave % 2);
    const bool bias = J.boff >= 0 && n0 == 0;
    // staging: A rows t / 16 and t / 16 + 16, four columns; B row t / 8, eight columns
    const float *ga = J.A + m0 + 4 * (t % 16);
    const bool bin = n0 + 8 * (t % 8) < J.No;
    const _Float16 *gb = J.B + (bin ? n0 + 8 * (t % 8) : 0);
    float4v ra[2];
    half8 rb;
    auto load = [&](int k0) __attribute__((always_inline)) {
        ra[0] = *(const float4u *)(ga + (long)(k0 + t / 16) * 256);
        ra[1] = *(const float4u *)(ga + (long)(k0 + 16 + t / 16) * 256);
        rb = *(const half8 *)(gb + (long)(k0 + t / 8) * J.No);
    };
    float4v acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = float4v{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    if (kb < ke) load(kb);
    for (int k0 = kb; k0 < ke; k0 += kBkK) {
        __syncthreads();   // the previous chunk has been read
        *(float4v *)&As[t / 16][4 * (t % 16)] = ra[0];
        *(float4v *)&As[16 + t / 16][4 * (t % 16)] = ra[1];
        float4v b0, b1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b0[i] = bin ? (float)rb[i] : 0.f;
            b1[i] = bin ? (float)rb[4 + i] : 0.f;
        }
        *(float4v *)&Bs[t / 8][8 * (t % 8)] = b0;
        *(float4v *)&Bs[t / 8][8 * (t % 8) + 4] = b1;
        __syncthreads();
        if (k0 + kBkK < ke) load(k0 + kBkK);
        if (bias)
#pragma unroll
            for (int i = 0; i < 8; ++i) bsum += As[8 * wave + i][lane];
#pragma unroll
        for (int kk = 0; kk < kBkK; kk += 4) {
            float a[2], b[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                a[x] = As[kk + kq][wm + 16 * x + r16];
                b[x] = Bs[kk + kq][wn + 16 * x + r16];
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[x], b[y], acc[x][y], 0, 0, 0);
        }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = m0 + wm + 16 * x + 4 * kq + i, col = n0 + wn + 16 * y + r16;
                if (col < J.No) out[J.off + (long)row * J.No + col] = acc[x][y][i];
            }
    if (bias) {
        __syncthreads();   // As has been read
        As[wave][lane] = bsum;
        __syncthreads();
        if (wave == 0) out[J.boff + m0 + lane] = ((As[0][lane] + As[1][lane]) + As[2][lane]) + As[3][lane];
    }
}

struct AdamArgs {
    float *w, *m, *v;
    _Float16 *wh;
    float lr, b1, b2, eps, c1, c2;
    long ndecay;
    float wd;
};

__device__ __forceinline__ void adam_update(const AdamArgs &a, long i, float gi)
{
    const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
    const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
    a.m[i] = mi;
    a.v[i] = vi;
    float u = (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
    if (i < a.ndecay) u += a.wd * a.w[i];
    const float wi = a.w[i] - a.lr * u;
    a.w[i] = wi;
    a.wh[i] = (_Float16)wi;
}

// g = the slices of part added in order; with ADAM the update with it; and, in
// the first workgroup, the loss: scale times the sum of its nloss partials
// (lane l the entries l, l + 64, ... in order, then a fixed butterfly).
template <bool ADAM>
__global__ void __launch_bounds__(256) train_update_kernel(long n, const float *__restrict__ part, int slices,
                                                           float *__restrict__ grad, const AdamArgs a,
                                                           const float *__restrict__ lpart, int nloss, float scale,
                                                           float *__restrict__ loss, float *__restrict__ loss2)
{
    const long i = blockIdx.x * 256L + threadIdx.x;
    if (ADAM && blockIdx.x == 0 && threadIdx.x < 64) {
        float l = 0.f;
        for (int k = threadIdx.x; k < nloss; k += 64) l += lpart[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
        if (threadIdx.x == 0) {
            *loss = l * scale;
            if (loss2) *loss2 = l * scale;
        }
    }
    if (i >= n) return;
    float s = 0.f;
    int z = 0;
    for (; z + 4 <= slices; z += 4) {
        const float p0 = part[z * n + i], p1 = part[(z + 1) * n + i], p2 = part[(z + 2) * n + i],
                    p3 = part[(z + 3) * n + i];
        s = (((s + p0) + p1) + p2) + p3;
    }
    for (; z < slices; ++z) s += part[z * n + i];
    grad[i] = s;
    if constexpr (ADAM) adam_update(a, i, s);
}

// Adam on FP32 masters (Kingma & Ba), then FP16 copies.  The first ndecay
// parameters also take decoupled weight decay wd (Loshchilov & Hutter):
// w -= lr (m_hat / (sqrt(v_hat) + eps) + wd w).
__global__ void adam_kernel(long n, const float *__restrict__ g, const AdamArgs a)
{
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
        adam_update(a, i, g[i]);
}

__global__ void to_half_kernel(long n, const float *__restrict__ w, _Float16 *__restrict__ wh)
{
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
        wh[i] = (_Float16)w[i];
}

static int grid_for(long n, int block)
{
    long gsz = (n + block - 1) / block;
    if (gsz > 65535) gsz = 65535;
    if (gsz < 1) gsz = 1;
    return (int)gsz;
}

// ---------------------------------------------------------------- launchers
hipError_t launch_mlp_features(const MlpColParams &p, const double *base, bool base3, const double *lb,
                               double rscale, const double *x, long col0, long ncol, void *feat, double *scale,
                               float *tgt, hipStream_t s)
{
    const int grid = (int)((ncol + 63) / 64);
    const size_t lds = sizeof(double) * 3 * (size_t)p.nz;
    hipLaunchKernelGGL(mlp_features_kernel, dim3(grid), dim3(512), lds, s, p, base, base3, lb, rscale, x, col0,
                       ncol, (_Float16 *)feat, scale, tgt);
    return hipGetLastError();
}

hipError_t launch_mlp_guess(const MlpColParams &p, const double *b, long col0, long ncol, const float *y,
                            const double *scale, double *x0, hipStream_t s)
{
    const int grid = (int)((ncol + 63) / 64);
    const size_t lds = (sizeof(double) * 4 + sizeof(int)) * (size_t)p.nz;
    hipLaunchKernelGGL(mlp_guess_kernel, dim3(grid), dim3(512), lds, s, p, b, col0, ncol, y, scale, x0);
    return hipGetLastError();
}

hipError_t launch_mlp_infer(const MlpColParams &p, const HeviParams &hp, const MlpNet &net, const double *base,
                            bool base3, const double *b, const double *lb, double rscale, long col0, long ncol,
                            double *x0, hipStream_t s)
{
    MlpWeights wt;
    for (int i = 0; i < 4; ++i) wt.W[i] = (const _Float16 *)net.wh[i];
    for (int i = 0; i < 3; ++i) wt.bias[i] = net.b[i];
    const int grid = (int)((ncol + 63) / 64);
    const size_t lds = (sizeof(double) * 7 + sizeof(int)) * (size_t)p.nz;
    const int nv = lb ? 0 : hp.N;
    if (nv > 0 && p.nz > kMlpFusedNz) return hipErrorInvalidValue;
#define NH_INFER(NN)                                                                                           \
    hipLaunchKernelGGL(mlp_infer_kernel<NN>, dim3(grid), dim3(512), lds, s, p, hp, wt, base, base3, b, lb, rscale, \
                       col0, ncol, x0)
    switch (nv) {
    case 0: NH_INFER(0); break;
    case 1: NH_INFER(1); break;
    case 2: NH_INFER(2); break;
    case 3: NH_INFER(3); break;
    case 4: NH_INFER(4); break;
    case 5: NH_INFER(5); break;
    case 6: NH_INFER(6); break;
    default: return hipErrorInvalidValue;
    }
#undef NH_INFER
    return hipGetLastError();
}

int mlp_fused_max_nz() { return kMlpFusedNz; }

hipError_t mlp_forward(const MlpNet &net, int M, const void *X, hipStream_t s, bool keep_z)
{
    static_assert(kMlpHid == 256 && kMlpOut == 256, "gemm_rows_kernel computes 256 outputs");
    const dim3 blk(256), grid(M / 64);
    const _Float16 *none = nullptr;
    hipLaunchKernelGGL(gemm_rows_kernel, grid, blk, 0, s, (const _Float16 *)X, (const _Float16 *)net.wh[0], net.b[0],
                       kMlpIn, none, none, 0, keep_z ? net.Z1 : nullptr, (_Float16 *)net.H1, 1);
    hipLaunchKernelGGL(gemm_rows_kernel, grid, blk, 0, s, (const _Float16 *)net.H1, (const _Float16 *)net.wh[1],
                       net.b[1], kMlpHid, none, none, 0, keep_z ? net.Z2 : nullptr, (_Float16 *)net.H2, 1);
    hipLaunchKernelGGL(gemm_rows_kernel, grid, blk, 0, s, (const _Float16 *)net.H2, (const _Float16 *)net.wh[2],
                       net.b[2], kMlpHid, (const _Float16 *)X, (const _Float16 *)net.wh[3], kMlpIn, net.Y,
                       (_Float16 *)nullptr, 0);
    return hipGetLastError();
}

// Rows per workgroup of the row part: 32 (the weights of each layer are read
// once per 32 rows), 16 while each workgroup then has a CU to itself.  A
// training step with 16 and with 32 rows: 46.2 and 59.7 us (batch 1024), 61.0 and
// 73.8 (4096), 97.6 and 86.4 (6144), 107.7 and 99.0 (8192).
static int train_rows(int M) { return M > 4096 ? 32 : 16; }

template <bool FWD>
static void launch_train_rows(const TrainRows &r, int M, hipStream_t s)
{
    if (train_rows(M) == 32)
        hipLaunchKernelGGL((mlp_train_rows_kernel<32, FWD>), dim3(M / 32), dim3(512), 0, s, r);
    else
        hipLaunchKernelGGL((mlp_train_rows_kernel<16, FWD>), dim3(M / 16), dim3(512), 0, s, r);
}

static TrainRows train_rows_args(const MlpNet &net, const void *X)
{
    TrainRows r{};
    r.X = (const _Float16 *)X;
    for (int i = 0; i < 4; ++i) r.wt.W[i] = (const _Float16 *)net.wh[i];
    for (int i = 0; i < 3; ++i) r.wt.bias[i] = net.b[i];
    r.Z1 = net.Z1; r.Z2 = net.Z2; r.dY = net.dY; r.dZ2 = net.dZ2; r.dZ1 = net.dZ1;
    r.H1 = (_Float16 *)net.H1; r.H2 = (_Float16 *)net.H2;
    r.part = net.part;
    return r;
}

// Batch slices of the weight gradients: 128 rows or more each, at most
// kMlpSlices (the partial sums of 16 slices are 15 MB).  A training step with
// slices of 64, 128 and 256 rows: 38.4, 39.0 and 41.8 us (batch 256), 48.3, 46.2
// and 45.7 (1024), no difference from 4096 on.
static int grad_slices(int M)
{
    const int n = M / 128;
    return n < 1 ? 1 : n > kMlpSlices ? kMlpSlices : n;
}

static hipError_t weight_grads(const MlpNet &net, int M, const void *X, const float *dY, int slices, hipStream_t s)
{
    const _Float16 *Xh = (const _Float16 *)X;
    auto off = [&](const float *p) { return (long)(p - net.grad); };
    GradJobs j;
    j.j[0] = {dY, Xh, kMlpIn, off(net.gw[3]), -1};
    j.j[1] = {dY, (const _Float16 *)net.H2, kMlpHid, off(net.gw[2]), off(net.gb[2])};
    j.j[2] = {net.dZ2, (const _Float16 *)net.H1, kMlpHid, off(net.gw[1]), off(net.gb[1])};
    j.j[3] = {net.dZ1, Xh, kMlpIn, off(net.gw[0]), off(net.gb[0])};
    const int kslice = ((M + slices - 1) / slices + kBkK - 1) / kBkK * kBkK;
    hipLaunchKernelGGL(mlp_grads_kernel, dim3(kGradTiles, slices), dim3(256), 0, s, j, M, kslice, net.nparam,
                       net.part_k);
    return hipGetLastError();
}

static AdamArgs adam_args(const MlpNet &net, float lr, float b1, float b2, float eps, int step, float wd)
{
    AdamArgs a{};
    a.w = net.master; a.m = net.m; a.v = net.v; a.wh = (_Float16 *)net.half;
    a.lr = lr; a.b1 = b1; a.b2 = b2; a.eps = eps;
    a.c1 = 1.f - powf(b1, (float)step);
    a.c2 = 1.f - powf(b2, (float)step);
    // the hidden path (W1, b1, W2, b2, W3, b3) precedes the bypass S
    a.ndecay = wd > 0.f ? net.nparam - (long)kMlpOut * kMlpIn : 0;
    a.wd = wd;
    return a;
}

hipError_t mlp_backward(const MlpNet &net, int M, const void *X, const float *dY, hipStream_t s)
{
    TrainRows r = train_rows_args(net, X);
    r.dYin = dY;
    launch_train_rows<false>(r, M, s);
    const int slices = grad_slices(M);
    hipError_t e = weight_grads(net, M, X, dY, slices, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((train_update_kernel<false>), dim3((unsigned)((net.nparam + 255) / 256)), dim3(256), 0, s,
                       net.nparam, net.part_k, slices, net.grad, AdamArgs{}, nullptr, 0, 0.f, nullptr, nullptr);
    return hipGetLastError();
}

// One training step in three launches: everything local to a row, the weight
// gradients, their sums with the Adam update and the loss.
hipError_t mlp_train_step(const MlpNet &net, int M, const void *X, const float *T, float lr, float b1, float b2,
                          float eps, int step, float wd, float *loss2, hipStream_t s)
{
    TrainRows r = train_rows_args(net, X);
    r.T = T;
    r.scale = 1.0f / ((float)M * kMlpOut);
    launch_train_rows<true>(r, M, s);
    const int slices = grad_slices(M);
    hipError_t e = weight_grads(net, M, X, net.dY, slices, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((train_update_kernel<true>), dim3((unsigned)((net.nparam + 255) / 256)), dim3(256), 0, s,
                       net.nparam, net.part_k, slices, net.grad, adam_args(net, lr, b1, b2, eps, step, wd), net.part,
                       M / train_rows(M), r.scale, net.loss, loss2);
    return hipGetLastError();
}

hipError_t mlp_adam(const MlpNet &net, float lr, float b1, float b2, float eps, int step, float wd, hipStream_t s)
{
    hipLaunchKernelGGL(adam_kernel, dim3(grid_for(net.nparam, 256)), dim3(256), 0, s, net.nparam, net.grad,
                       adam_args(net, lr, b1, b2, eps, step, wd));
    return hipGetLastError();
}

hipError_t mlp_sync_half(const MlpNet &net, hipStream_t s)
{
    hipLaunchKernelGGL(to_half_kernel, dim3(grid_for(net.nparam, 256)), dim3(256), 0, s, net.nparam, net.master,
                       (_Float16 *)net.half);
    return hipGetLastError();
}

}  // namespace nh
