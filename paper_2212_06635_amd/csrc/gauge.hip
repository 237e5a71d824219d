// Gauge-field and clover set-up kernels (run once per gauge field / mass).
//
//  * link compression: rows 0 and 1 of every SU(3) link are kept (row 2 is
//    conj(row0 x row1), rebuilt in registers by the stencil kernels), split
//    by the parity of the site the link starts at, in the site-major layout.
//  * clover term: F_{mu nu} from the four plaquette leaves, F = (Q - Q^+)/8,
//    T = i kappa csw sum_{mu<nu} sigma_{mu nu} F_{mu nu}.  In the chiral
//    basis sigma_{kl} = -eps_{klm} diag(s_m, s_m) and sigma_{k4} = diag(s_k,
//    -s_k) (s = Pauli matrices), so each chirality block is
//      T_chi = i kappa csw (s_1 (x) G_1 + s_2 (x) G_2 + s_3 (x) G_3),
//      G_1 = -F_yz +- F_xt,  G_2 = F_xz +- F_yt,  G_3 = -F_xy +- F_zt
//    (+ for chirality 0 = spins 0,1, - for chirality 1).  T is stored as its
//    structured blocks (load_ct): H = i kappa csw G_3, K = i kappa csw
//    (G_1 + i G_2).  A clover term given by the caller is stored as A = 1 + T
//    in general Hermitian 6x6 blocks.
//  * site inverses through (A + i nu)^{-1} = (A - i nu)(A^2 + nu^2)^{-1},
//    with the Hermitian positive A^2 + nu^2 inverted by Cholesky, all in
//    FP64; where that fails (two flavours: A^2 + nubar^2 - epsbar^2 need not be
//    positive on rough fields) by elimination with pivoting on its factors.
#include "tmx_device.h"
#include "tmx_kernels.h"

namespace tmx {

using cd = cx<double>;

struct M3 {
    cd m[9];
};

__device__ __forceinline__ M3 mul(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cd s{0, 0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(s, a.m[3 * i + k], b.m[3 * k + j]);
            c.m[3 * i + j] = s;
        }
    return c;
}

// a * b^dagger
__device__ __forceinline__ M3 mul_nd(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cd s{0, 0};
#pragma unroll
            for (int k = 0; k < 3; ++k) s = s + a.m[3 * i + k] * conj(b.m[3 * j + k]);
            c.m[3 * i + j] = s;
        }
    return c;
}

// a^dagger * b
__device__ __forceinline__ M3 mul_dn(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cd s{0, 0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac_conj(s, a.m[3 * k + i], b.m[3 * k + j]);
            c.m[3 * i + j] = s;
        }
    return c;
}

// ---------------------------------------------------------------------------
// link compression
// ---------------------------------------------------------------------------
__global__ void pack_links_kernel(const double *canon, double *links64, Geom g)
{
    const long V = 2L * g.Vh;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= V) return;
    int x[4];
    long r = i;
    x[0] = (int)(r % g.L[0]);
    r /= g.L[0];
    x[1] = (int)(r % g.L[1]);
    r /= g.L[1];
    x[2] = (int)(r % g.L[2]);
    x[3] = (int)(r / g.L[2]);
    const int p = (x[0] + x[1] + x[2] + x[3]) & 1;
    const int s = cb_index(g, x);
    double2 *out = reinterpret_cast<double2 *>(links64);
    const double2 *in = reinterpret_cast<const double2 *>(canon);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
#pragma unroll
        for (int k = 0; k < 6; ++k) out[((long)(p * 4 + mu) * 6 + k) * g.Vh + s] = in[(i * 4 + mu) * 9 + k];
}

hipError_t launch_pack_links(const double *canon, double *links64, Geom g, hipStream_t st)
{
    const long V = 2L * g.Vh;
    hipLaunchKernelGGL(pack_links_kernel, dim3((V + 255) / 256), dim3(256), 0, st, canon, links64, g);
    return hipGetLastError();
}

__global__ void convert_links_kernel(const double *links64, void *dst, int prec, long Vh)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 8 * Vh) return;
    const long pm = t / Vh, s = t - pm * Vh;  // (p*4+mu), site
    const double2 *in = reinterpret_cast<const double2 *>(links64) + pm * 6 * Vh;
    float v[12];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        double2 d = in[k * Vh + s];
        v[2 * k] = (float)d.x;
        v[2 * k + 1] = (float)d.y;
    }
    if (prec == F32) {
        float4 *o = static_cast<float4 *>(dst) + pm * 3 * Vh;
#pragma unroll
        for (int k = 0; k < 3; ++k) o[k * Vh + s] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    } else {
        uint2 *o = static_cast<uint2 *>(dst) + pm * 3 * Vh;
#pragma unroll
        for (int k = 0; k < 3; ++k) o[k * Vh + s] = f_to_h4(v + 4 * k);
    }
}

hipError_t launch_convert_links(const double *links64, void *dst, int prec, Geom g, hipStream_t st)
{
    const long n = 8L * g.Vh;
    hipLaunchKernelGGL(convert_links_kernel, dim3((n + 255) / 256), dim3(256), 0, st, links64, dst, prec,
                       (long)g.Vh);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// clover term
// ---------------------------------------------------------------------------
__device__ __forceinline__ M3 link_at(const double *links64, const Geom &g, const int x[4], int mu)
{
    const int p = (x[0] + x[1] + x[2] + x[3]) & 1;
    LinkPtr U{links64, g.Vh};
    M3 u;
    load_link<F64, false>(U, p, mu, cb_index(g, x), u.m);
    return u;
}

__device__ __forceinline__ void step(const Geom &g, const int x[4], int mu, int d, int y[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = x[k];
    y[mu] += d;
    if (y[mu] < 0) y[mu] += g.L[mu];
    if (y[mu] >= g.L[mu]) y[mu] -= g.L[mu];
}

// F_{mu nu}(x) = (Q - Q^+)/8 with Q the sum of the four leaves.  Q and Q^+
// enter alike, so a leaf may be replaced by minus its adjoint: two leaves then
// end in the same link and share its product (10 products instead of 12).
// f: the imaginary parts of the diagonal of F, then F_10, F_20, F_21.
__device__ __forceinline__ void field_strength(const double *U, const Geom &g, const int x[4], int mu, int nu,
                                               double f[9])
{
    int xpm[4], xpn[4], xmm[4], xmn[4], xmmpn[4], xmmmn[4], xpmmn[4];
    step(g, x, mu, +1, xpm);
    step(g, x, nu, +1, xpn);
    step(g, x, mu, -1, xmm);
    step(g, x, nu, -1, xmn);
    step(g, xmm, nu, +1, xmmpn);
    step(g, xmm, nu, -1, xmmmn);
    step(g, xpm, nu, -1, xpmmn);
    M3 Q;
    const M3 un = link_at(U, g, x, nu), vn = link_at(U, g, xmn, nu);
    {
        // [U_nu(x-nu)^+ U_mu(x-nu) U_nu(x+mu-nu) - U_nu(x) U_mu(x+nu) U_nu(x+mu)^+] U_mu(x)^+
        M3 s = mul(mul_dn(vn, link_at(U, g, xmn, mu)), link_at(U, g, xpmmn, nu));
        const M3 t = mul_nd(mul(un, link_at(U, g, xpn, mu)), link_at(U, g, xpm, nu));
#pragma unroll
        for (int k = 0; k < 9; ++k) s.m[k] = s.m[k] - t.m[k];
        Q = mul_nd(s, link_at(U, g, x, mu));
    }
    {
        // [U_nu(x) U_mu(x-mu+nu)^+ U_nu(x-mu)^+ - U_nu(x-nu)^+ U_mu(x-mu-nu)^+ U_nu(x-mu-nu)] U_mu(x-mu)
        M3 s = mul_nd(mul_nd(un, link_at(U, g, xmmpn, mu)), link_at(U, g, xmm, nu));
        const M3 w = mul(link_at(U, g, xmmmn, mu), vn);  // (U_mu U_nu)^+ = U_nu^+ U_mu^+
        const M3 t = mul_dn(w, link_at(U, g, xmmmn, nu));
#pragma unroll
        for (int k = 0; k < 9; ++k) s.m[k] = s.m[k] - t.m[k];
        const M3 r = mul(s, link_at(U, g, xmm, mu));
#pragma unroll
        for (int k = 0; k < 9; ++k) Q.m[k] = Q.m[k] + r.m[k];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) f[i] = 0.25 * Q.m[4 * i].im;
    int k = 3;
#pragma unroll
    for (int i = 1; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
            const cd v = 0.125 * (Q.m[3 * i + j] - conj(Q.m[3 * j + i]));
            f[k] = v.re;
            f[k + 1] = v.im;
            k += 2;
        }
}

// packed Hermitian store: 36 reals per chirality (d0..d5, 15 lower (re,im))
__device__ __forceinline__ void store_herm(double *clov64, long stride, long s, int chir, const cd A[6][6])
{
    double a[36];
#pragma unroll
    for (int i = 0; i < 6; ++i) a[i] = A[i][i].re;
    int k = 6;
#pragma unroll
    for (int i = 1; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
            a[k] = A[i][j].re;
            a[k + 1] = A[i][j].im;
            k += 2;
        }
    store_seq<F64, 36>(clov64 + (size_t)chir * 18 * stride * 2, stride, s, a);
}

__device__ __forceinline__ void load_herm(const double *clov64, long stride, long s, int chir, cd A[6][6])
{
    double a[36];
    load_seq<F64, 36>(clov64 + (size_t)chir * 18 * stride * 2, stride, s, a);
#pragma unroll
    for (int i = 0; i < 6; ++i) A[i][i] = cd{a[i], 0.0};
    int k = 6;
#pragma unroll
    for (int i = 1; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
            A[i][j] = cd{a[k], a[k + 1]};
            A[j][i] = cd{a[k], -a[k + 1]};
            k += 2;
        }
}

// A = 1 + T of one chirality from the structured (ct) or general storage
__device__ __forceinline__ void load_block(const double *clov64, int ct, long stride, long s, int chir, cd A[6][6])
{
    if (!ct) {
        load_herm(clov64, stride, s, chir, A);
        return;
    }
    double a[28];
    load_ct<F64>(clov64, stride, s, chir, a);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        A[i][i] = cd{1.0 + ct_diag(a, i), 0.0};
#pragma unroll
        for (int j = 0; j < i; ++j) {
            A[i][j] = ct_lower(a, i, j);
            A[j][i] = conj(A[i][j]);
        }
    }
}

// whether elimination on 1 + T (structured block a) keeps every pivot at 1/8 or more
__device__ __forceinline__ bool pivots_bounded(const double a[28])
{
    cd A[6][6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        A[i][i] = cd{1.0 + ct_diag(a, i), 0.0};
#pragma unroll
        for (int j = 0; j < i; ++j) A[i][j] = ct_lower(a, i, j);
    }
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        ok = ok && A[k][k].re >= 0.125;  // false for a NaN too
        const double d = 1.0 / A[k][k].re;
#pragma unroll
        for (int i = k + 1; i < 6; ++i) {
            const cd f = d * A[i][k];
#pragma unroll
            for (int j = k + 1; j <= i; ++j) cmsub(A[i][j], f, conj(A[j][k]));
        }
    }
    return ok;
}

// clov64 layout: [parity][56 reals as 28 double2][Vh].  Six waves per 64 sites
// of one parity, one plane each (a thread that took all six planes held the
// results of five while computing the sixth: 1.6 kB of scratch a lane); the
// nine reals of each F meet in LDS and two waves write one chirality each.
// The links are read through the caches (each serves 24 plaquette leaves of
// its neighbourhood) with both parities of a region on one XCD: 4.74 -> 1.68 ms
// at 32^3x64 (2.19 ms with streaming loads and no XCD order), 314 -> 96 us at
// 16^3x32.
__global__ void __launch_bounds__(384) clover_build_kernel(const double *links64, double *clov64, Geom g, double kappa,
                                                           double csw)
{
    __shared__ double F[6][9][64];  // plane order: xy, xz, xt, yz, yt, zt
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int b = xcd_block(1), p = b & 1;  // both parities of a region on one XCD
    const int s0 = (b >> 1) * 64 + lane;
    const int s = s0 < g.Vh ? s0 : g.Vh - 1;
    int x[4];
    cb_coords(g, s, p, x);
    {
        const int mu = w < 3 ? 0 : (w < 5 ? 1 : 2), nu = w < 3 ? w + 1 : (w < 5 ? w - 1 : 3);
        double f[9];
        field_strength(links64, g, x, mu, nu, f);
#pragma unroll
        for (int k = 0; k < 9; ++k) F[w][k][lane] = f[k];
    }
    __syncthreads();
    if (w >= 2 || s0 >= g.Vh) return;
    const double kc = kappa * csw, sg = w == 0 ? 1.0 : -1.0;
    double g1[9], g2[9], g3[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        g1[k] = -F[3][k][lane] + sg * F[2][k][lane];
        g2[k] = F[1][k][lane] + sg * F[4][k][lane];
        g3[k] = -F[0][k][lane] + sg * F[5][k][lane];
    }
    // T = i kc [[G3, G1 - i G2], [G1 + i G2, -G3]] = [[H, K^+], [K, -H]]
    double a[28];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        a[i] = -kc * g3[i];
        a[4 + 2 * i] = -kc * g3[4 + 2 * i];
        a[5 + 2 * i] = kc * g3[3 + 2 * i];
        // K_ii = kc (i G1 - G2)_ii
        a[10 + 8 * i] = -kc * g1[i];
        a[11 + 8 * i] = -kc * g2[i];
    }
    int k = 3;
#pragma unroll
    for (int i = 1; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
            const int lo = 10 + 2 * (3 * i + j), up = 10 + 2 * (3 * j + i);
            a[lo] = kc * (-g1[k + 1] - g2[k]);
            a[lo + 1] = kc * (g1[k] - g2[k + 1]);
            a[up] = kc * (-g1[k + 1] + g2[k]);  // G_ji = -conj(G_ij)
            a[up + 1] = kc * (-g1[k] - g2[k + 1]);
            k += 2;
        }
    a[3] = 0.0;
    if (p == 0 && pivots_bounded(a)) a[3] = 1.0;
    store_seq<F64, 28>(clov64 + ((size_t)p * 28 + w * 14) * g.Vh * 2, g.Vh, s, a);
}

hipError_t launch_clover_build(const double *links64, double *clov64, Geom g, double kappa, double csw,
                               hipStream_t st)
{
    const long nb = 2L * ((g.Vh + 63) / 64);
    hipLaunchKernelGGL(clover_build_kernel, dim3((unsigned)nb), dim3(384), 0, st, links64, clov64, g, kappa, csw);
    return hipGetLastError();
}

// four reals per thread (one vector of the FP32 / FP16 layout)
__global__ void convert_ct_kernel(const double *src, void *dst, int prec, long Vh)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 28 * Vh) return;  // both parities, both chiralities, 7 vectors
    const long q = t / Vh, s = t - q * Vh;
    const double2 *in = reinterpret_cast<const double2 *>(src);
    const double2 lo = in[2 * q * Vh + s], hi = in[(2 * q + 1) * Vh + s];
    const float v[4] = {(float)lo.x, (float)lo.y, (float)hi.x, (float)hi.y};
    if (prec == F32)
        static_cast<float4 *>(dst)[q * Vh + s] = make_float4(v[0], v[1], v[2], v[3]);
    else
        static_cast<uint2 *>(dst)[q * Vh + s] = f_to_h4(v);
}

hipError_t launch_convert_ct(const double *src, void *dst, int prec, long Vh, hipStream_t st)
{
    const long n = 28 * Vh;
    hipLaunchKernelGGL(convert_ct_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, prec, Vh);
    return hipGetLastError();
}

// thread per (parity, site): both chirality blocks of A = 1 + T as 72 halves
__global__ void __launch_bounds__(256) convert_ct_general16_kernel(const double *src, void *dst, long Vh)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * Vh) return;
    const long p = t / Vh, s = t - p * Vh;
    float o[72];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        double a[28];
        load_ct<F64>(src + (size_t)p * 28 * Vh * 2, Vh, s, c, a);
        float *q = o + 36 * c;
#pragma unroll
        for (int i = 0; i < 6; ++i) q[i] = (float)(1.0 + ct_diag(a, i));
        int k = 6;
#pragma unroll
        for (int i = 1; i < 6; ++i)
#pragma unroll
            for (int j = 0; j < i; ++j) {
                const cd l = ct_lower(a, i, j);
                q[k] = (float)l.re;
                q[k + 1] = (float)l.im;
                k += 2;
            }
    }
    // through FP32, like every FP16 field (launch_convert_seq): keep the compiler
    // from rounding FP64 to binary16 in one step
#pragma unroll
    for (int i = 0; i < 72; ++i) asm volatile("" : "+v"(o[i]));
    store_seq<F16, 72>(static_cast<char *>(dst) + (size_t)p * 72 * 2 * Vh, Vh, s, o);
}

hipError_t launch_convert_ct_general16(const double *src, void *dst, long Vh, hipStream_t st)
{
    hipLaunchKernelGGL(convert_ct_general16_kernel, dim3((unsigned)((2 * Vh + 255) / 256)), dim3(256), 0, st, src, dst,
                       Vh);
    return hipGetLastError();
}

// canonical T: [lex][chir][6][6] complex128, A = 1 + T
__global__ void __launch_bounds__(128) clover_from_canon_kernel(const double *canonT, double *clov64, int ct, Geom g, int to_canon)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2L * g.Vh) return;
    int x[4];
    long r = i;
    x[0] = (int)(r % g.L[0]);
    r /= g.L[0];
    x[1] = (int)(r % g.L[1]);
    r /= g.L[1];
    x[2] = (int)(r % g.L[2]);
    x[3] = (int)(r / g.L[2]);
    const int p = (x[0] + x[1] + x[2] + x[3]) & 1;
    const int s = cb_index(g, x);
    double *base = clov64 + (size_t)p * (ct ? 28 : 36) * g.Vh * 2;
    const double2 *cin = reinterpret_cast<const double2 *>(canonT) + i * 72;
    double2 *cout = reinterpret_cast<double2 *>(const_cast<double *>(canonT)) + i * 72;
    for (int chir = 0; chir < 2; ++chir) {
        cd A[6][6];
        if (to_canon) {
            load_block(base, ct, g.Vh, s, chir, A);
            for (int a = 0; a < 6; ++a)
                for (int b = 0; b < 6; ++b) {
                    cd v = A[a][b];
                    if (a == b) v.re -= 1.0;
                    cout[chir * 36 + 6 * a + b] = make_double2(v.re, v.im);
                }
        } else {
            for (int a = 0; a < 6; ++a)
                for (int b = 0; b < 6; ++b) {
                    double2 v = cin[chir * 36 + 6 * a + b];
                    A[a][b] = cd{v.x + (a == b ? 1.0 : 0.0), v.y};
                }
            store_herm(base, g.Vh, s, chir, A);
        }
    }
}

hipError_t launch_clover_from_canonical(const double *canonT, double *clov64, Geom g, hipStream_t st)
{
    const long n = 2L * g.Vh;
    hipLaunchKernelGGL(clover_from_canon_kernel, dim3((n + 127) / 128), dim3(128), 0, st, canonT, clov64, 0, g, 0);
    return hipGetLastError();
}

hipError_t launch_clover_to_canonical(const double *clov64, int ct, double *canonT, Geom g, hipStream_t st)
{
    const long n = 2L * g.Vh;
    hipLaunchKernelGGL(clover_from_canon_kernel, dim3((n + 127) / 128), dim3(128), 0, st, canonT,
                       const_cast<double *>(clov64), ct, g, 1);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// site inverses
// ---------------------------------------------------------------------------
// S^{-1} for Hermitian positive definite 6x6 S via Cholesky S = L L^+:
// S^{-1} = L^{-+} L^{-1}.  False (no usable result) where S is not positive, or
// a pivot has lost half its digits.
__device__ __forceinline__ bool hpd_inverse(const cd S[6][6], cd Sinv[6][6])
{
    cd Lm[6][6];
    double dinv[6];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) Lm[i][j] = cd{0, 0};
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double d = S[j][j].re;
#pragma unroll
        for (int k = 0; k < j; ++k) d -= Lm[j][k].re * Lm[j][k].re + Lm[j][k].im * Lm[j][k].im;
        ok = ok && d > 1e-8 * S[j][j].re;
        d = sqrt(d);
        Lm[j][j] = cd{d, 0};
        dinv[j] = 1.0 / d;
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            cd v = S[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) {
                // v -= L[i][k] conj(L[j][k])
                const cd a = Lm[i][k], b = Lm[j][k];
                v.re -= a.re * b.re + a.im * b.im;
                v.im -= a.im * b.re - a.re * b.im;
            }
            Lm[i][j] = dinv[j] * v;
        }
    }
    // W = L^{-1} (lower triangular)
    cd W[6][6];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) W[i][j] = cd{0, 0};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        W[i][i] = cd{dinv[i], 0};
#pragma unroll
        for (int j = 0; j < i; ++j) {
            cd v{0, 0};
#pragma unroll
            for (int k = j; k < i; ++k) cmac(v, Lm[i][k], W[k][j]);
            W[i][j] = -dinv[i] * v;
        }
    }
    // Sinv = W^+ W
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            cd v{0, 0};
#pragma unroll
            for (int k = (i > j ? i : j); k < 6; ++k) cmac_conj(v, W[k][i], W[k][j]);
            Sinv[i][j] = v;
        }
    return ok;
}

// (A^2 - z^2)^{-1} = (A - z)^{-1} (A + z)^{-1} for any Hermitian A of the clover
// field: elimination with partial pivoting, one factor after the other.  Rows
// are indexed at run time, so the matrix lives in scratch; only fields rough
// enough to have eigenvalues of A near or below |z| need it.
__device__ __forceinline__ void inverse_pivot(const double *clov, int ct, long stride, long s, int chir, cd z,
                                              cd Sinv[6][6])
{
    cd m[6][12];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) m[i][6 + j] = cd{i == j ? 1.0 : 0.0, 0.0};
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        {
            cd A[6][6];
            load_block(clov, ct, stride, s, chir, A);
            const cd sh = pass == 0 ? z : -z;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int j = 0; j < 6; ++j) m[i][j] = i == j ? A[i][j] + sh : A[i][j];
        }
#pragma unroll 1
        for (int k = 0; k < 6; ++k) {
            int r = k;
            double best = -1.0;
#pragma unroll 1
            for (int i = k; i < 6; ++i) {
                const double n = m[i][k].re * m[i][k].re + m[i][k].im * m[i][k].im;
                if (n > best) {
                    best = n;
                    r = i;
                }
            }
            const cd p{m[r][k].re / best, -m[r][k].im / best};
#pragma unroll 1
            for (int j = k; j < 12; ++j) {  // row k = pivot row / pivot
                const cd t = m[r][j];
                m[r][j] = m[k][j];
                m[k][j] = t * p;
            }
#pragma unroll 1
            for (int i = 0; i < 6; ++i) {
                if (i == k) continue;
                const cd f = m[i][k];
#pragma unroll 1
                for (int j = k; j < 12; ++j) m[i][j] = m[i][j] - f * m[k][j];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) Sinv[i][j] = m[i][6 + j];
}

// A^2 + c (Hermitian positive for c > -lambda_min(A^2))
__device__ __forceinline__ void herm_square_shift(const cd A[6][6], double c, cd S[6][6])
{
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            cd v{i == j ? c : 0.0, 0};
#pragma unroll
            for (int k = 0; k < 6; ++k) cmac(v, A[i][k], A[k][j]);
            S[i][j] = v;
        }
}

// thread per (even site, chirality); inv64 layout [72 reals per chirality as
// 36 double2, chirality-major][Vh]
__global__ void __launch_bounds__(64) clover_inv_kernel(const double *clov_even, int ct, double *inv64, long Vh, double nu)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * Vh) return;
    const int chir = (int)(t / Vh);
    const long s = t - chir * Vh;
    cd A[6][6], S[6][6], Si[6][6];
    load_block(clov_even, ct, Vh, s, chir, A);
    const double tw = chir == 0 ? nu : -nu;  // i nu gamma5 on this chirality
    herm_square_shift(A, tw * tw, S);
    if (!hpd_inverse(S, Si)) inverse_pivot(clov_even, ct, Vh, s, chir, cd{0.0, tw}, Si);
    // (A + i tw)^{-1} = (A - i tw) S^{-1}
    double out[72];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            cd v{0, 0};
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                cd a = A[i][k];
                if (i == k) a.im -= tw;
                cmac(v, a, Si[k][j]);
            }
            out[12 * i + 2 * j] = v.re;
            out[12 * i + 2 * j + 1] = v.im;
        }
    store_seq<F64, 72>(inv64 + (size_t)chir * 36 * Vh * 2, Vh, s, out);
}

hipError_t launch_clover_inv(const double *clov64_even, int ct, double *inv64, Geom g, double nu, hipStream_t st)
{
    const long n = 2L * g.Vh;
    hipLaunchKernelGGL(clover_inv_kernel, dim3((n + 63) / 64), dim3(64), 0, st, clov64_even, ct, inv64, (long)g.Vh,
                       nu);
    return hipGetLastError();
}

__global__ void __launch_bounds__(64) clover_inv_nd_kernel(const double *clov_even, int ct, double *invnd64, long Vh, double c)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * Vh) return;
    const int chir = (int)(t / Vh);
    const long s = t - chir * Vh;
    cd A[6][6], S[6][6], Si[6][6];
    load_block(clov_even, ct, Vh, s, chir, A);
    herm_square_shift(A, c, S);
    if (!hpd_inverse(S, Si))
        inverse_pivot(clov_even, ct, Vh, s, chir, c < 0.0 ? cd{sqrt(-c), 0.0} : cd{0.0, sqrt(c)}, Si);
    store_herm(invnd64, Vh, s, chir, Si);
}

hipError_t launch_clover_inv_nd(const double *clov64_even, int ct, double *invnd64, Geom g, double nubar, double epst,
                                hipStream_t st)
{
    const long n = 2L * g.Vh;
    hipLaunchKernelGGL(clover_inv_nd_kernel, dim3((n + 63) / 64), dim3(64), 0, st, clov64_even, ct, invnd64,
                       (long)g.Vh, nubar * nubar - epst * epst);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// precision conversion of per-site real sequences (8 reals per thread)
// ---------------------------------------------------------------------------
__global__ void convert_seq_kernel(const double *src, void *dst, int prec, int nchunk, long nsite)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nchunk * nsite) return;
    const long c = t / nsite, s = t - c * nsite;
    const double2 *in = reinterpret_cast<const double2 *>(src);
    float v[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double2 d = in[(4 * c + k) * nsite + s];
        v[2 * k] = (float)d.x;
        v[2 * k + 1] = (float)d.y;
    }
    if (prec == F32) {
        float4 *o = static_cast<float4 *>(dst);
        o[(2 * c) * nsite + s] = make_float4(v[0], v[1], v[2], v[3]);
        o[(2 * c + 1) * nsite + s] = make_float4(v[4], v[5], v[6], v[7]);
    } else {
        uint4 *o = static_cast<uint4 *>(dst);
        o[c * nsite + s] = f_to_h8(v);
    }
}

hipError_t launch_convert_seq(const double *src, void *dst, int prec, int nreal, long nsite, hipStream_t st)
{
    const int nchunk = nreal / 8;
    const long n = nchunk * nsite;
    hipLaunchKernelGGL(convert_seq_kernel, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, prec, nchunk, nsite);
    return hipGetLastError();
}

}  // namespace tmx
