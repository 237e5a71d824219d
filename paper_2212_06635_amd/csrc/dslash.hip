// Wilson twisted-mass clover stencil kernels (gfx950).
//
// One launch computes, for every site s of the output parity p and every
// right-hand side r (slot t = s * nrhs + r; a launch may take a group of the
// right-hand sides, see dslash_kernel):
//
//   MODE_INV  (first half of the Schur operator, "K1"):
//       out = B_p^{-1}(sgn) (H in)(s)
//     degenerate: B^{-1} = (A + i sgn nu g5)^{-1}, a stored full 6x6 per
//     chirality (the -nu inverse is its adjoint);
//     two flavours: (A + X)^{-1} = (A - X) (A^2 + nubar^2 - epst^2)^{-1},
//     X = i sgn nubar g5 tau3 - epst tau1, with A and the Hermitian inverse
//     factor stored.
//   MODE_NRM (MODE_DIAG that also writes |out|^2 + nsig |x|^2 of every slot).
//   MODE_RES (MODE_DIAG with a residual epilogue, for the solvers):
//       rout = rin - alpha (out + sigma p)(s),  nrm = |rout|^2
//       in FP64: saves the pass that wrote the operator's result and the one
//       that read it back with r (3 of the 15 spinors of vector traffic in a
//       CG iteration).
//   MODE_SOLVE (K1 with the site block inverted in the kernel):
//       out = B_p^{-1}(sgn) (H in)(s) by elimination on the stored A itself.
//       The stencils are bound by HBM bytes (a wave spends some 130k cycles
//       mostly waiting, against about 4k for the two eliminations), so 56
//       reals of site data instead of the inverse's 144 is what counts: with
//       the structured A in K2 (56 instead of 72) the FP64 Mhat at 32^3x64
//       went from 772 to 633 us, the FP16 MP-CG from 66.1 to 58.9 ms.
//       Two flavours (FP64, many sites, nubar <= epst): two Hermitian
//       eliminations, A -+ del, on the one A instead of A and the stored
//       inverse factor; N at 24^3x48 717 -> 675 us.
//       Not in FP32: there the stored inverse, formed in FP64 and rounded
//       once, is the more accurate one.
//   MODE_DIAG (second half, "K2", or one parity of the full operator D):
//       out = (A_p + X(sgn)) x(s) - kfac (H in)(s)
//     with X = i sgn nu g5 (degenerate) or the two-flavour X above; for the
//     mass-preconditioned operator (one flavour) i rho x is added to the
//     final output.
//
// H is the Wilson hopping term with the spin projectors (1 -+ gamma_mu) of
// the chiral basis written out per direction: the projected half spinor
// h = psi_upper + sgn * a_mu psi_lower is transported, and the lower spin
// components are rebuilt as sgn * a_mu^dagger (U h), where gamma_mu =
// [[0, a_mu], [a_mu^dagger, 0]], a_k = -i sigma_k, a_4 = 1.
//
// Optional gamma5 on the hopping input (g5in), on the diagonal input (g5x)
// and on the output (g5out) implement the
// adjoint Mhat^dagger = g5 Mhat(-sgn) g5 and the normal operator without
// extra passes.
#include <type_traits>

#include "tmx_device.h"
#include "tmx_kernels.h"

namespace tmx {



// transported half spinor k = bc W h of a hop, h the projection of psi by
// (1 + sgn gamma_mu), W = U (fwd) or U^dagger (bwd): k0, k1 its two spins
template <int MU, int SGN, bool DAG, typename R>
__device__ __forceinline__ void hop_half(const cx<R> u[9], R bc, const cx<R> psi[12], cx<R> k0[3], cx<R> k1[3])
{
    // half spinor h[spin 0/1][colour]
    cx<R> h0[3], h1[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<R> p0 = psi[c], p1 = psi[3 + c], p2 = psi[6 + c], p3 = psi[9 + c];
        cx<R> a0, a1;  // a_mu psi_lower
        if constexpr (MU == 0) {
            a0 = -imul(p3);
            a1 = -imul(p2);
        } else if constexpr (MU == 1) {
            a0 = -p3;
            a1 = p2;
        } else if constexpr (MU == 2) {
            a0 = -imul(p2);
            a1 = imul(p3);
        } else {
            a0 = p2;
            a1 = p3;
        }
        if constexpr (SGN > 0) {
            h0[c] = p0 + a0;
            h1[c] = p1 + a1;
        } else {
            h0[c] = p0 - a0;
            h1[c] = p1 - a1;
        }
    }
    // k = W h
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        k0[a] = cx<R>{0, 0};
        k1[a] = cx<R>{0, 0};
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if constexpr (DAG) {
                cmac_conj(k0[a], u[3 * b + a], h0[b]);
                cmac_conj(k1[a], u[3 * b + a], h1[b]);
            } else {
                cmac(k0[a], u[3 * a + b], h0[b]);
                cmac(k1[a], u[3 * a + b], h1[b]);
            }
        }
        k0[a] = bc * k0[a];
        k1[a] = bc * k1[a];
    }
}

// lower spins of a hop from its half spinor: (l0, l1) += sgn * a_mu^dagger (k0, k1)
template <int MU, int SGN, typename R>
__device__ __forceinline__ void hop_lower(const cx<R> k0[3], const cx<R> k1[3], cx<R> *low)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        cx<R> l0, l1;
        if constexpr (MU == 0) {
            l0 = imul(k1[c]);
            l1 = imul(k0[c]);
        } else if constexpr (MU == 1) {
            l0 = k1[c];
            l1 = -k0[c];
        } else if constexpr (MU == 2) {
            l0 = imul(k0[c]);
            l1 = -imul(k1[c]);
        } else {
            l0 = k0[c];
            l1 = k1[c];
        }
        if constexpr (SGN > 0) {
            low[c] = low[c] + l0;
            low[3 + c] = low[3 + c] + l1;
        } else {
            low[c] = low[c] - l0;
            low[3 + c] = low[3 + c] - l1;
        }
    }
}

// acc += (1 + sgn gamma_mu) * bc * W psi
template <int MU, int SGN, bool DAG, typename R>
__device__ __forceinline__ void hop_term(const cx<R> u[9], R bc, const cx<R> psi[12], cx<R> acc[12])
{
    cx<R> k0[3], k1[3];
    hop_half<MU, SGN, DAG>(u, bc, psi, k0, k1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        acc[c] = acc[c] + k0[c];
        acc[3 + c] = acc[3 + c] + k1[c];
    }
    hop_lower<MU, SGN>(k0, k1, acc + 6);
}

template <int P, typename R>
__device__ __forceinline__ void load_spinor_g5(const SpinorPtr &f, int flav, long slot, bool g5, cx<R> v[12])
{
    load_spinor<P>(f, flav, slot, v);
    if (g5) {
#pragma unroll
        for (int k = 6; k < 12; ++k) v[k] = -v[k];
    }
}

// accumulate (H in)(s) for all flavours
template <int P, int NF, int MU, bool NT, typename R>
__device__ __forceinline__ void hop_dir(const DslashArgs &a, const int x[4], int s, long rhs, cx<R> acc[NF][12])
{
    const Geom &g = a.g;
    const int p = a.parity;
    // forward: (1 - gamma_mu) U_mu(x) psi(x + mu)
    {
        int y[4] = {x[0], x[1], x[2], x[3]};
        R bc = R(1);
        if (++y[MU] == g.L[MU]) {
            y[MU] = 0;
            if (MU == 3) bc = R(a.t_bc);
        }
        const int n = cb_index(g, y);
        cx<R> u[9];
        load_link<P, NT>(a.U, p, MU, s, u);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            cx<R> psi[12];
            load_spinor_g5<P>(a.in, f, (long)n * a.nrhs + rhs, a.g5in, psi);
            hop_term<MU, -1, false>(u, bc, psi, acc[f]);
        }
        // one flavour, and two flavours in FP32: the forward and backward hops
        // of a direction share a fence, so both neighbours' loads are in
        // flight together (FP64: 220 VGPRs, two waves per SIMD; 1-4 % faster
        // than a fence per hop); FP64 and FP16 two-flavour kernels keep a
        // fence per hop (FP16: 5 % slower paired)
        if constexpr (NF != 1 && P != F32) {
#pragma unroll
            for (int f = 0; f < NF; ++f) reg_fence(acc[f], 12);
        }
    }
    // backward: (1 + gamma_mu) U_mu(x - mu)^dagger psi(x - mu)
    {
        int y[4] = {x[0], x[1], x[2], x[3]};
        R bc = R(1);
        if (--y[MU] < 0) {
            y[MU] = g.L[MU] - 1;
            if (MU == 3) bc = R(a.t_bc);
        }
        const int n = cb_index(g, y);
        cx<R> u[9];
        load_link<P, NT>(a.U, 1 - p, MU, n, u);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            cx<R> psi[12];
            load_spinor_g5<P>(a.in, f, (long)n * a.nrhs + rhs, a.g5in, psi);
            hop_term<MU, +1, true>(u, bc, psi, acc[f]);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) reg_fence(acc[f], 12);
    }
}

// A is DslashArgs for applications and DslashFused for a solver's kernels
template <class A> constexpr bool FUSED = std::is_same_v<A, DslashFused>;

template <int P, int NF, int MODE, bool CT, bool NT = true, class A>
__device__ __forceinline__ void dslash_slot(const A &a, int s, long rhs);

// Whether a launch enqueued ahead is not wanted any more.  Kernel arguments are
// not loaded ahead of a branch they lie behind, so a check in front of
// everything made their miss a serial one more per launch; the empty asm asks for
// those of the check and the first ones the hops need together with those of
// u.
__device__ __forceinline__ bool stopped(const DslashFused &a, long &u)
{
    const int *stop = a.stop;
    const int it = a.it;
    asm volatile(""
                 : "+v"(u)
                 : "s"(stop), "s"(it), "s"(a.in.d), "s"(a.U.d), "s"(a.out.d), "s"(a.clov), "s"(a.parity), "s"(a.nrhs),
                   "s"(a.t_bc), "s"(a.g5in));
    return stop && *stop < it;
}

// Thread i takes the work items i, i + G, ..., i + (SPT - 1) G (G the grid's
// thread count); item u is right-hand side r0 + u % rg of site u / rg.  SPT
// is a template parameter: a runtime loop costs registers (and occupancy)
// even when it runs once.
template <int P, int NF, int MODE, int SPT, bool CT, class A>
__global__ void __launch_bounds__(256) dslash_kernel(A a)
{
    const long rg = a.rg;
    const long n = (long)a.g.Vh * rg;
    long u = (long)xcd_block(a.xcd) * blockDim.x + threadIdx.x;
    if constexpr (FUSED<A>)
        if (stopped(a, u)) return;
    if constexpr (SPT == 1) {
        if (u >= n) return;
        const int s = (int)(u / rg);
        dslash_slot<P, NF, MODE, CT>(a, s, a.r0 + (u - (long)s * rg));
    } else {
        const long G = (long)gridDim.x * blockDim.x;
        for (int k = 0; k < SPT && u < n; ++k, u += G) {
            const int s = (int)(u / rg);
            dslash_slot<P, NF, MODE, CT>(a, s, a.r0 + (u - (long)s * rg));
        }
    }
}

// Two first halves at once, for the force terms: out = B^{-1}(sgn) (H in) and
// out2 = B^{-1}(-sgn) (H in2) with the other setting of g5in.  Workgroups
// 2i and 2i + 1 (with the XCD order, on one XCD at about the same time) take
// the same sites, so links and site blocks, two thirds of the bytes, come
// from HBM once; they are therefore read through the caches, not past them.
// FP64 at 32^3x64, the pair: 663 us as two launches, 633 with streamed links,
// 572 with cached ones (the waves of the pair in one workgroup: 584); 2.0 GB
// at that size, so waits at two waves per SIMD are what is left.
template <int NF, int MODE, bool CT>
__global__ void __launch_bounds__(256) dslash_pair_kernel(DslashArgs a, SpinorPtr in2, SpinorPtr out2)
{
    const int blk = xcd_block(a.xcd);
    const long s = (long)(blk >> 1) * blockDim.x + threadIdx.x;
    if (s >= a.g.Vh) return;
    if (blk & 1) {
        a.in = in2;
        a.out = out2;
        a.sgn = -a.sgn;
        a.g5in = !a.g5in;
    }
    dslash_slot<F64, NF, MODE, CT, false>(a, (int)s, 0);
}

template <typename R> __device__ __forceinline__ void add_norm(double &n2, const cx<R> v[6])
{
#pragma unroll
    for (int k = 0; k < 6; ++k) n2 += (double)v[k].re * v[k].re + (double)v[k].im * v[k].im;
}

// (A_chir + i tw) v for both flavours (structured or general blocks)
template <int P, bool CT, typename R>
__device__ __forceinline__ void apply_clov(const void *clov, long cs, long s, int c, R tw0, const cx<R> *v0, cx<R> *o0,
                                           R tw1, const cx<R> *v1, cx<R> *o1)
{
    if constexpr (CT) {
        R b[28];
        load_ct<P>(clov, cs, s, c, b);
        ct_apply(b, tw0, v0, o0);
        ct_apply(b, tw1, v1, o1);
    } else {
        herm_apply_c<P>(clov, cs, s, c, tw0, v0, o0);
        herm_apply_c<P>(clov, cs, s, c, tw1, v1, o1);
    }
}

// one output slot: site s (of the output parity), right-hand side rhs; NT:
// links streamed past the caches
template <int P, int NF, int MODE, bool CT, bool NT, class A>
__device__ __forceinline__ void dslash_slot(const A &a, int s, long rhs)
{
    using R = typename RealOf<P>::type;
    const long t = (long)s * a.nrhs + rhs;  // slot of the output, the diagonal input and the norms
    int x[4];
    cb_coords(a.g, s, a.parity, x);

    cx<R> acc[NF][12];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[f][k] = cx<R>{0, 0};

    // one direction at a time (register fences inside hop_dir): holding every
    // neighbour's data at once would need ~4x the registers and drop
    // occupancy to one wave per SIMD.  t first: its neighbours are the
    // farthest in memory (most often past L2), so their loads go out first
    // (FP64 K1 1.4 % faster than x first)
    hop_dir<P, NF, 3, NT>(a, x, s, rhs, acc);
    hop_dir<P, NF, 2, NT>(a, x, s, rhs, acc);
    hop_dir<P, NF, 1, NT>(a, x, s, rhs, acc);
    hop_dir<P, NF, 0, NT>(a, x, s, rhs, acc);

    const long cs = a.g.Vh;  // clover stride
    // site-block epilogue, one chirality block at a time (register fences
    // keep the two blocks' matrices from being live together)
    cx<R> out[NF][12];
    double xn2 = 0.0;  // MODE_NRM with nsig: |x|^2
    if constexpr (MODE == MODE_SOLVE) {
        static_assert(CT, "the in-kernel solve takes structured blocks");
        const R nb = R(a.sgn * a.nu);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            R b[28];
            load_ct<P>(a.clov, cs, s, c, b);
            const R tw = c == 0 ? nb : -nb;
            if constexpr (NF == 1) {
#pragma unroll
                for (int k = 0; k < 6; ++k) out[0][6 * c + k] = acc[0][6 * c + k];
                ct_solve(b, tw, out[0] + 6 * c);
            } else {
                ct_inverse_nd(b, R(a.del), tw, R(a.epst), acc[0] + 6 * c, acc[1] + 6 * c, out[0] + 6 * c,
                              out[1] + 6 * c);
                reg_fence(out[1] + 6 * c, 6);
            }
            reg_fence(out[0] + 6 * c, 6);
        }
    } else if constexpr (MODE == MODE_INV) {
        if constexpr (NF == 1) {
            const bool dag = a.sgn < 0;
            full_apply<P>(a.inv, cs, s, 0, dag, acc[0], out[0]);
            reg_fence(out[0], 6);
            full_apply<P>(a.inv, cs, s, 1, dag, acc[0] + 6, out[0] + 6);
        } else {
            // (A + X)^{-1} acc = (A - X) t,  t_f = Binv acc_f  (per chirality)
            const R nb = R(a.sgn * a.nu), ep = R(a.epst);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const R tw = c == 0 ? nb : -nb;  // i nubar g5 tau3 on flavour 0
                cx<R> t0[6], t1[6];
                herm_apply_c<P>(a.inv, cs, s, c, R(0), acc[0] + 6 * c, t0);
                herm_apply_c<P>(a.inv, cs, s, c, R(0), acc[1] + 6 * c, t1);
                reg_fence(t0, 6);
                reg_fence(t1, 6);
                apply_clov<P, CT>(a.clov, cs, s, c, -tw, t0, out[0] + 6 * c, tw, t1, out[1] + 6 * c);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    out[0][6 * c + k] = out[0][6 * c + k] + ep * t1[k];
                    out[1][6 * c + k] = out[1][6 * c + k] + ep * t0[k];
                }
                reg_fence(out[0] + 6 * c, 6);
                reg_fence(out[1] + 6 * c, 6);
            }
        }
    } else {
        const R kf = R(a.kfac);
        const R nb = R(a.sgn * a.nu);
        const R g5s = a.g5x ? R(-1) : R(1);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const R tw = c == 0 ? nb : -nb;
            const R gx = c == 0 ? R(1) : g5s;  // gamma5 on the diagonal input
            if constexpr (NF == 1) {
                cx<R> xv[6];
                load_chiral<P>(a.x, 0, t, c, xv);
#pragma unroll
                for (int k = 0; k < 6; ++k) xv[k] = gx * xv[k];
                if constexpr (MODE == MODE_NRM)
                    if (a.nsig) add_norm(xn2, xv);
                if constexpr (CT) {
                    R b[28];
                    load_ct<P>(a.clov, cs, s, c, b);
                    ct_apply(b, tw, xv, out[0] + 6 * c);
                } else {
                    herm_apply_c<P>(a.clov, cs, s, c, tw, xv, out[0] + 6 * c);
                }
                if (a.rho != 0.0) {
                    // + i rho x on the final output: before the output gamma5,
                    // the lower chirality takes the opposite sign
                    const R rs = (c == 1 && a.g5out) ? R(-a.rho) : R(a.rho);
#pragma unroll
                    for (int k = 0; k < 6; ++k) out[0][6 * c + k] = out[0][6 * c + k] + rs * imul(gx * xv[k]);
                }
            } else {
                const R ep = R(a.epst);
                cx<R> x0[6], x1[6];
                load_chiral<P>(a.x, 0, t, c, x0);
                load_chiral<P>(a.x, 1, t, c, x1);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    x0[k] = gx * x0[k];
                    x1[k] = gx * x1[k];
                }
                if constexpr (MODE == MODE_NRM) {
                    if (a.nsig) {
                        add_norm(xn2, x0);
                        add_norm(xn2, x1);
                    }
                }
                apply_clov<P, CT>(a.clov, cs, s, c, tw, x0, out[0] + 6 * c, -tw, x1, out[1] + 6 * c);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    out[0][6 * c + k] = out[0][6 * c + k] - ep * x1[k];
                    out[1][6 * c + k] = out[1][6 * c + k] - ep * x0[k];
                }
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
#pragma unroll
                for (int k = 0; k < 6; ++k) out[f][6 * c + k] = out[f][6 * c + k] - kf * acc[f][6 * c + k];
                reg_fence(out[f] + 6 * c, 6);
            }
        }
    }
    if (a.g5out) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int k = 6; k < 12; ++k) out[f][k] = -out[f][k];
    }
    if constexpr (MODE == MODE_RES) {
        // a kernel of its own: in MODE_DIAG the residual's registers would
        // take the FP16 kernels from four waves per SIMD to three
        const double al = a.ralpha ? a.ralpha[rhs] : 1.0, sg = a.rsig ? a.rsig[rhs] : 0.0;
        double n2 = 0.0;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            cx<R> r[12];
            load_spinor<P, true>(a.rin, f, t, r);
            if (a.rsig) {
                cx<R> p[12];
                load_spinor<P, true>(a.rp, f, t, p);
#pragma unroll
                for (int k = 0; k < 12; ++k)
                    out[f][k] = cx<R>{(R)fma(sg, (double)p[k].re, (double)out[f][k].re),
                                      (R)fma(sg, (double)p[k].im, (double)out[f][k].im)};
            }
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                const double re = fma(-al, (double)out[f][k].re, (double)r[k].re);
                const double im = fma(-al, (double)out[f][k].im, (double)r[k].im);
                n2 += re * re + im * im;
                r[k] = cx<R>{(R)re, (R)im};
            }
            store_spinor<P, P != F16>(a.rout, f, t, r);
            if constexpr (P == F64) {
                if (a.rlo.d && a.rlo_prec == F32) store_spinor<F32>(a.rlo, f, t, r);
                if (a.rlo.d && a.rlo_prec == F16) store_spinor<F16>(a.rlo, f, t, r);
            }
        }
        a.nrm[t] = n2;
        return;
    }
    if constexpr (MODE == MODE_NRM) {
        double n2 = 0.0;
        if (a.nsig) n2 = a.nsig[rhs] * xn2;
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int k = 0; k < 12; ++k) n2 += (double)out[f][k].re * out[f][k].re + (double)out[f][k].im * out[f][k].im;
        a.nrm[t] = n2;
    }
    // the output is written once per sweep: non-temporal stores keep it from
    // displacing the neighbour spinors in L2 (FP16 outputs, 52 bytes a site,
    // measured no faster that way)
#pragma unroll
    for (int f = 0; f < NF; ++f) store_spinor<P, P != F16>(a.out, f, t, out[f]);
}

// ---------------------------------------------------------------------------
// split form: four waves per 64 slots, one lattice direction each
// ---------------------------------------------------------------------------
// One thread per slot takes its eight hops one direction after the other, each
// waiting for its loads: some 7 us a launch however few sites there are, and
// below about three waves per SIMD nothing else hides that.  Here wave w of a
// workgroup takes both hops of direction w for the same 64 slots and leaves
// the transported half spinors in LDS; after one barrier waves 0 and 1 sum
// them in the order of the plain form (the two forms differ by the rounding of
// products that the compiler fuses into sums in one of them) and finish one
// chirality each.  Site blocks and the other per-site operands
// are requested before the barrier.
template <int P, typename R> struct SplitShared {
    cx<R> k[8][6][64];    // hop, component of the half spinor, slot
    float amax[2][64]; // FP16 scales: largest component per chirality
    double n2[64];        // chirality 1's part of the norm
};

template <int P, int NF, int MU, typename R>
__device__ __forceinline__ void split_dir(const DslashArgs &a, const int x[4], int s, long rhs, int h, int lane,
                                          SplitShared<P, R> *sh)
{
    const Geom &g = a.g;
    const int p = a.parity;
    int y[4] = {x[0], x[1], x[2], x[3]}, z[4] = {x[0], x[1], x[2], x[3]};
    R bf = R(1), bb = R(1);
    if (++y[MU] == g.L[MU]) {
        y[MU] = 0;
        if (MU == 3) bf = R(a.t_bc);
    }
    if (--z[MU] < 0) {
        z[MU] = g.L[MU] - 1;
        if (MU == 3) bb = R(a.t_bc);
    }
    const int nf = cb_index(g, y), nb = cb_index(g, z);
    cx<R> u[9], v[9];
    load_link<P>(a.U, p, MU, s, u);
    load_link<P>(a.U, 1 - p, MU, nb, v);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        cx<R> psi[12], k[6];
        load_spinor_g5<P>(a.in, f, (long)nf * a.nrhs + rhs, a.g5in, psi);
        hop_half<MU, -1, false>(u, bf, psi, k, k + 3);
#pragma unroll
        for (int c = 0; c < 6; ++c) sh[f].k[h][c][lane] = k[c];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        cx<R> psi[12], k[6];
        load_spinor_g5<P>(a.in, f, (long)nb * a.nrhs + rhs, a.g5in, psi);
        hop_half<MU, +1, true>(v, bb, psi, k, k + 3);
#pragma unroll
        for (int c = 0; c < 6; ++c) sh[f].k[h + 1][c][lane] = k[c];
    }
}

// sum of the hops for chirality c, in the plain form's order (t, z, y, x)
template <int MU, int P, typename R>
__device__ __forceinline__ void split_sum_dir(const SplitShared<P, R> &sh, int h, int lane, int c, cx<R> acc[6])
{
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        cx<R> k[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) k[i] = sh.k[h + d][i][lane];
        if (c == 0) {
#pragma unroll
            for (int i = 0; i < 6; ++i) acc[i] = acc[i] + k[i];
        } else if (d == 0) {
            hop_lower<MU, -1>(k, k + 3, acc);
        } else {
            hop_lower<MU, +1>(k, k + 3, acc);
        }
    }
}

// store chirality c (6 components) of flavour f; FP16: `m` the scale of the slot
template <int P, bool NT, typename R>
__device__ __forceinline__ void store_chiral(const SpinorPtr &o, int f, long t, int c, const cx<R> v[6], float m)
{
    R q[12];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        q[2 * k] = v[k].re;
        q[2 * k + 1] = v[k].im;
    }
    char *base = static_cast<char *>(o.d) + (size_t)f * spinor_vecs<P>() * o.stride * 16;
    if constexpr (P == F16) {
        const float inv = m > 0.f ? 1.0f / m : 0.f;
        float z[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) z[k] = (float)q[k] * inv;
        uint4 *b = reinterpret_cast<uint4 *>(base);
        if (c == 0) {  // vector 0 and the first half of vector 1
            b[t] = f_to_h8(z);
            *reinterpret_cast<uint2 *>(b + o.stride + t) = f_to_h4(z + 8);
            o.nrm[f * o.stride + t] = m;
        } else {  // the second half of vector 1 and vector 2
            *(reinterpret_cast<uint2 *>(b + o.stride + t) + 1) = f_to_h4(z);
            b[2 * o.stride + t] = f_to_h8(z + 4);
        }
    } else {
        store_seq<P, 12, R, NT>(base + (size_t)c * (spinor_vecs<P>() / 2) * o.stride * 16, o.stride, t, q);
    }
}

template <typename R> __device__ __forceinline__ float chiral_max(const cx<R> v[6])
{
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < 6; ++k) m = fmaxf(m, fmaxf(fabsf((float)v[k].re), fabsf((float)v[k].im)));
    return m;
}

template <int P, int NF, int MODE, bool CT, class A>
__global__ void __launch_bounds__(256) dslash_split_kernel(A a)
{
    using R = typename RealOf<P>::type;
    extern __shared__ __align__(16) char split_lds[];
    auto *sh = reinterpret_cast<SplitShared<P, R> *>(split_lds);  // one per flavour
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long n = (long)a.g.Vh * a.rg;
    long u0 = (long)xcd_block(a.xcd) * 64 + lane;
    if constexpr (FUSED<A>)
        if (stopped(a, u0)) return;
    const bool live = u0 < n;
    const long u = live ? u0 : n - 1;  // the last workgroup's spare lanes repeat the last slot
    const int s = (int)(u / a.rg);
    const long rhs = a.r0 + (u - (long)s * a.rg);
    const long t = (long)s * a.nrhs + rhs;
    const long cs = a.g.Vh;
    const int c = w;  // chirality of waves 0 and 1 in the second part
    int x[4];
    cb_coords(a.g, s, a.parity, x);

    // per-site operands of the second part, requested first
    R b[28];
    if (w < 2) {
        if constexpr (CT && MODE != MODE_INV) load_ct<P>(a.clov, cs, s, c, b);
    }
    if (w == 0)
        split_dir<P, NF, 3>(a, x, s, rhs, 0, lane, sh);
    else if (w == 1)
        split_dir<P, NF, 2>(a, x, s, rhs, 2, lane, sh);
    else if (w == 2)
        split_dir<P, NF, 1>(a, x, s, rhs, 4, lane, sh);
    else
        split_dir<P, NF, 0>(a, x, s, rhs, 6, lane, sh);
    __syncthreads();

    cx<R> out[NF][6];
    double n2 = 0.0;
    if (w < 2) {
        cx<R> acc[NF][6];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int k = 0; k < 6; ++k) acc[f][k] = cx<R>{0, 0};
            split_sum_dir<3>(sh[f], 0, lane, c, acc[f]);
            split_sum_dir<2>(sh[f], 2, lane, c, acc[f]);
            split_sum_dir<1>(sh[f], 4, lane, c, acc[f]);
            split_sum_dir<0>(sh[f], 6, lane, c, acc[f]);
        }
        const R nb = R(a.sgn * a.nu), tw = c == 0 ? nb : -nb, ep = R(a.epst);
        if constexpr (MODE == MODE_SOLVE) {
            static_assert(NF == 1, "the two-flavour solve is for many sites only");
#pragma unroll
            for (int k = 0; k < 6; ++k) out[0][k] = acc[0][k];
            ct_solve(b, tw, out[0]);
        } else if constexpr (MODE == MODE_INV) {
            if constexpr (NF == 1) {
                full_apply<P>(a.inv, cs, s, c, a.sgn < 0, acc[0], out[0]);
            } else {
                cx<R> t0[6], t1[6];
                herm_apply_c<P>(a.inv, cs, s, c, R(0), acc[0], t0);
                herm_apply_c<P>(a.inv, cs, s, c, R(0), acc[1], t1);
                apply_clov<P, CT>(a.clov, cs, s, c, -tw, t0, out[0], tw, t1, out[1]);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    out[0][k] = out[0][k] + ep * t1[k];
                    out[1][k] = out[1][k] + ep * t0[k];
                }
            }
        } else {
            const R kf = R(a.kfac);
            const R gx = (c == 1 && a.g5x) ? R(-1) : R(1);
            double xn2 = 0.0;
            cx<R> xv[NF][6];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                load_chiral<P>(a.x, f, t, c, xv[f]);
#pragma unroll
                for (int k = 0; k < 6; ++k) xv[f][k] = gx * xv[f][k];
                if constexpr (MODE == MODE_NRM)
                    if (a.nsig) add_norm(xn2, xv[f]);
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const R tf = f == 0 ? tw : -tw;
                if constexpr (CT)
                    ct_apply(b, tf, xv[f], out[f]);
                else
                    herm_apply_c<P>(a.clov, cs, s, c, tf, xv[f], out[f]);
            }
            if constexpr (NF == 1) {
                if (a.rho != 0.0) {
                    const R rs = (c == 1 && a.g5out) ? R(-a.rho) : R(a.rho);
#pragma unroll
                    for (int k = 0; k < 6; ++k) out[0][k] = out[0][k] + rs * imul(gx * xv[0][k]);
                }
            } else {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    out[0][k] = out[0][k] - ep * xv[1][k];
                    out[1][k] = out[1][k] - ep * xv[0][k];
                }
            }
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int k = 0; k < 6; ++k) out[f][k] = out[f][k] - kf * acc[f][k];
            if constexpr (MODE == MODE_NRM)
                if (a.nsig) n2 = a.nsig[rhs] * xn2;
        }
        if (a.g5out && c == 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int k = 0; k < 6; ++k) out[f][k] = -out[f][k];
        }
        if constexpr (MODE == MODE_RES) {
            const double al = a.ralpha ? a.ralpha[rhs] : 1.0, sg = a.rsig ? a.rsig[rhs] : 0.0;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                cx<R> r[6];
                load_chiral<P>(a.rin, f, t, c, r);
                if (a.rsig) {
                    cx<R> p[6];
                    load_chiral<P>(a.rp, f, t, c, p);
#pragma unroll
                    for (int k = 0; k < 6; ++k)
                        out[f][k] = cx<R>{(R)fma(sg, (double)p[k].re, (double)out[f][k].re),
                                          (R)fma(sg, (double)p[k].im, (double)out[f][k].im)};
                }
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const double re = fma(-al, (double)out[f][k].re, (double)r[k].re);
                    const double im = fma(-al, (double)out[f][k].im, (double)r[k].im);
                    n2 += re * re + im * im;
                    out[f][k] = cx<R>{(R)re, (R)im};
                }
            }
        } else if constexpr (MODE == MODE_NRM) {
#pragma unroll
            for (int f = 0; f < NF; ++f) add_norm(n2, out[f]);
        }
        if constexpr (P == F16 || MODE == MODE_RES) {
#pragma unroll
            for (int f = 0; f < NF; ++f) sh[f].amax[c][lane] = chiral_max(out[f]);
        }
        if constexpr (MODE == MODE_RES || MODE == MODE_NRM) {
            if (c == 1) sh[0].n2[lane] = n2;
        }
    }
    if constexpr (P == F16 || MODE == MODE_RES || MODE == MODE_NRM) __syncthreads();
    if (w >= 2 || !live) return;
    if constexpr (MODE == MODE_RES || MODE == MODE_NRM) {
        if (c == 0) a.nrm[t] = n2 + sh[0].n2[lane];
    }
    SpinorPtr dst = a.out;
    if constexpr (MODE == MODE_RES) dst = a.rout;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        float m = 0.f;
        if constexpr (P == F16 || MODE == MODE_RES) m = fmaxf(sh[f].amax[0][lane], sh[f].amax[1][lane]);
        store_chiral<P, P != F16>(dst, f, t, c, out[f], m);
        if constexpr (P == F64 && MODE == MODE_RES) {
            if (a.rlo.d && a.rlo_prec == F32) store_chiral<F32, false>(a.rlo, f, t, c, out[f], m);
            if (a.rlo.d && a.rlo_prec == F16) store_chiral<F16, false>(a.rlo, f, t, c, out[f], m);
        }
    }
}

// Slots up to which the split form is the faster one.  Measured on N (two K1,
// two K2; us, plain -> split), one flavour FP64 / FP32 / FP16, then two flavours:
//    2048 slots  31 -> 23 / 28 -> 20 / 33 -> 23   46 -> 31 / 40 -> 30 / 49 -> 30
//   13824 slots  40 -> 30 / 34 -> 23 / 36 -> 24   65 -> 44 / 47 -> 35 / 56 -> 34
//   32768 slots  55 -> 54 / 39 -> 34 / 41 -> 29   86 -> 88 / 56 -> 47 / 63 -> 43
//   65536 slots  92 -> 99 / 51 -> 53 / 48 -> 42  158 -> 166 / 80 -> 92 / 73 -> 74
//  120960 slots 158 -> 180 / 86 -> 91 / 66 -> 69
// (beyond, the plain form's waves fill the chip and LDS and barriers only cost)
template <int P, int NF> static bool use_split(long n)
{
    return n <= (P == F64 ? 24576 : (P == F16 && NF == 1 ? 98304 : 49152));
}

template <int P, int NF, int MODE, bool CT, class A>
static hipError_t launch_one(const A &a, hipStream_t st, int block)
{
    using R = typename RealOf<P>::type;
    const long n = (long)a.g.Vh * a.rg;
    if (n == 0) return hipSuccess;
    if constexpr (!(MODE == MODE_SOLVE && NF == 2)) {  // that one is for many sites only
        if (use_split<P, NF>(n)) {
            hipLaunchKernelGGL((dslash_split_kernel<P, NF, MODE, CT, A>), dim3((unsigned)((n + 63) / 64)), dim3(256),
                               NF * sizeof(SplitShared<P, R>), st, a);
            return hipGetLastError();
        }
    }
    constexpr bool EPI = MODE == MODE_RES || MODE == MODE_NRM;  // one slot per thread
    const long per = block * (long)(EPI ? 1 : a.spt);
    const int grid = (int)((n + per - 1) / per);
    if constexpr (!EPI) {
        if (a.spt == 2) {
            hipLaunchKernelGGL((dslash_kernel<P, NF, MODE, 2, CT, A>), dim3(grid), dim3(block), 0, st, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((dslash_kernel<P, NF, MODE, 1, CT, A>), dim3(grid), dim3(block), 0, st, a);
    return hipGetLastError();
}

template <int NF, int MODE, bool CT>
static hipError_t launch_pair(const DslashArgs &a, const SpinorPtr &in2, const SpinorPtr &out2, hipStream_t st,
                              int block)
{
    const long grid = 2 * ((long)(a.g.Vh + block - 1) / block);
    hipLaunchKernelGGL((dslash_pair_kernel<NF, MODE, CT>), dim3((unsigned)grid), dim3(block), 0, st, a, in2, out2);
    return hipGetLastError();
}

template <int P, int NF, class A>
static hipError_t launch_mode(int mode, const A &a, hipStream_t st, int block)
{
    if (mode == MODE_SOLVE) {
        if constexpr (P == F64 || (P == F16 && NF == 1))  // FP32: the stored inverse, formed in FP64
            return a.ct ? launch_one<P, NF, MODE_SOLVE, true>(a, st, block) : hipErrorInvalidValue;
        else
            return hipErrorInvalidValue;
    }
    if (mode == MODE_INV) {
        if constexpr (NF == 1)  // reads the inverse only
            return launch_one<P, NF, MODE_INV, false>(a, st, block);
        else
            return a.ct ? launch_one<P, NF, MODE_INV, true>(a, st, block)
                        : launch_one<P, NF, MODE_INV, false>(a, st, block);
    }
    if constexpr (FUSED<A>) {
        if (mode == MODE_NRM)
            return a.ct ? launch_one<P, NF, MODE_NRM, true>(a, st, block) : launch_one<P, NF, MODE_NRM, false>(a, st, block);
        if (mode == MODE_RES)
            return a.ct ? launch_one<P, NF, MODE_RES, true>(a, st, block) : launch_one<P, NF, MODE_RES, false>(a, st, block);
        return hipErrorInvalidValue;
    } else {
        if (mode != MODE_DIAG) return hipErrorInvalidValue;
        return a.ct ? launch_one<P, NF, MODE_DIAG, true>(a, st, block) : launch_one<P, NF, MODE_DIAG, false>(a, st, block);
    }
}

template <class A>
static hipError_t launch_any(int prec, int nf, int mode, const A &a0, hipStream_t st, int block)
{
    if (block <= 0) block = 256;
    A a = a0;
    if (a.spt != 2) a.spt = 1;
    if (a.rg <= 0 || a.r0 < 0 || a.r0 + a.rg > a.nrhs) {
        a.r0 = 0;
        a.rg = a.nrhs;
    }
    if (prec == F64) return nf == 1 ? launch_mode<F64, 1>(mode, a, st, block) : launch_mode<F64, 2>(mode, a, st, block);
    if (prec == F32) return nf == 1 ? launch_mode<F32, 1>(mode, a, st, block) : launch_mode<F32, 2>(mode, a, st, block);
    if (prec == F16) return nf == 1 ? launch_mode<F16, 1>(mode, a, st, block) : launch_mode<F16, 2>(mode, a, st, block);
    return hipErrorInvalidValue;
}

hipError_t launch_dslash(int prec, int nf, int mode, const DslashArgs &a, hipStream_t st, int block)
{
    return launch_any(prec, nf, mode, a, st, block);
}

hipError_t launch_dslash_fused(int prec, int nf, int mode, const DslashFused &a, hipStream_t st, int block)
{
    return launch_any(prec, nf, mode, a, st, block);
}

hipError_t launch_dslash_pair(int nf, int mode, const DslashArgs &a0, SpinorPtr in2, SpinorPtr out2, hipStream_t st,
                              int block)
{
    if (block <= 0) block = 256;
    DslashArgs a = a0;
    a.spt = 1;
    a.r0 = 0;
    a.rg = 1;
    const bool inv = mode == MODE_INV;
    if (a.nrhs != 1 || (!inv && (mode != MODE_SOLVE || !a.ct))) return hipErrorInvalidValue;
    if (a.g.Vh == 0) return hipSuccess;
    if (nf == 1 ? use_split<F64, 1>(a.g.Vh) : use_split<F64, 2>(a.g.Vh)) {
        hipError_t e = launch_dslash(F64, nf, mode, a, st, block);
        if (e != hipSuccess) return e;
        a.in = in2;
        a.out = out2;
        a.sgn = -a.sgn;
        a.g5in = !a.g5in;
        return launch_dslash(F64, nf, mode, a, st, block);
    }
    if (!inv)
        return nf == 1 ? launch_pair<1, MODE_SOLVE, true>(a, in2, out2, st, block)
                       : launch_pair<2, MODE_SOLVE, true>(a, in2, out2, st, block);
    if (nf == 1) return launch_pair<1, MODE_INV, false>(a, in2, out2, st, block);
    return a.ct ? launch_pair<2, MODE_INV, true>(a, in2, out2, st, block) : launch_pair<2, MODE_INV, false>(a, in2, out2, st, block);
}

}  // namespace tmx
