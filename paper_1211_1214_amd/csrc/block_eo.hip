// Even-odd preconditioned Schwarz block solves: x_k = D_k(m)^-1 b_k for every block k of
// one colour, with D_k the Dirichlet block operator (Sec. 1 of the paper).  Inside a
// block the odd sites are eliminated (eo.h):
//     M_k = A_ee - 1/4 H^k_eo A_oo^-1 H^k_oe,  b'_e = b_e + 1/2 H^k_eo A_oo^-1 b_o,
//     x_o = A_oo^-1 (b_o + 1/2 H^k_oe x_e),
// H^k the hops inside block k.  Every kernel here runs one workgroup per (block, RHS); the
// block's even and odd sites occupy the same contiguous range of the two half fields.
//   k_blk_prep    FP64: b'_e, r_e = b'_e, x_e = 0, ||b_k||^2, ||r_e||^2
//   k_blk_lds, k_lds_lanes, k_blk_mr   persistent minimal residual in FP32 (FP16 storage) on M_k for r_e / ||r_e||, adds
//                 the correction to x_e in FP64 (blocks already converged return at once)
//   k_blk_lds (BI), k_blk_inner   the same by BiCGStab, in the LDS and in memory: where minimal residual converges slowly, in
//                 FP64, and on blocks whose hop masks k_blk_mr cannot hold
//   k_blk_resid   FP64: r_e = b'_e - M_k x_e and ||r_e||^2 (defect correction)
//   k_blk_recon   FP64: x_o, and (x_e, x_o) written to the full solution
// k_blk_prep_lds and k_blk_resid_lds are the FP64 passes of blocks whose parity fits the LDS.  The LDS-resident solvers
// also take whole small lattices as one block (WRAP) for the global solver.
#include <algorithm>
#include <type_traits>

#include "ddwc_internal.h"
#include "eo.h"
#include "uniform_mem.h"
#include "../../include/ddwc.h"

namespace ddwc {

constexpr int BE_MAX_THREADS = 256;  // FP64 kernels: prep, resid, recon and the FP64 inner solver
constexpr int BE_INNER_MAX = 768;    // FP32/FP16 inner solver: up to 12 waves (3 per SIMD at its VGPR use)

// Workgroup size of a block kernel of at most `cap` threads: `req` (a multiple of 64, from the
// schedule options) or, by default, enough waves for one block parity.
static int block_threads_for(const Geom& g, int req, int cap) {
    const int t = req > 0 ? ((req + 63) / 64) * 64 : ((g.hvb + 63) / 64) * 64;
    return t < cap ? t : cap;
}
int block_eo_threads(const Geom& g, int req) { return block_threads_for(g, req, BE_MAX_THREADS); }

// The persistent inner solver in FP32/FP16 storage runs up to BE_INNER_MAX threads: a 6^4 block
// parity (648 sites) is then one pass of 11 waves, and one such workgroup per CU keeps the
// block vectors in flight small enough for the last-level cache.
template <class S>
constexpr int be_inner_max() {
    return std::is_same<S, double>::value ? BE_MAX_THREADS : BE_INNER_MAX;
}

struct BlkIdx {
    int rank, rhs, B;
    unsigned h0;  // half index of the block's first site (both parities)
    size_t key;   // (rhs, rank) slot of the per-block arrays
};

// Workgroups are numbered block-major, RHS-minor and dealt to the 8 XCDs so that each XCD
// sweeps a contiguous range: the RHS of one block run on one XCD and share its links and
// clover in that XCD's L2.
__device__ __forceinline__ BlkIdx blk_idx(const Geom& g, int colour, int nrhs) {
    BlkIdx b;
    const int n = (int)gridDim.x;
    const int L = (n & 7) ? (int)blockIdx.x : ((int)blockIdx.x & 7) * (n >> 3) + ((int)blockIdx.x >> 3);
    b.rank = L / nrhs;
    b.rhs = L - b.rank * nrhs;
    b.B = colour * g.NBc + b.rank;
    b.h0 = (unsigned)b.B * g.hvb;
    b.key = (size_t)b.rhs * g.NBc + b.rank;
    return b;
}

// Storage S (double, float or H16; arithmetic in Traits<S>::real).  A vector of one RHS is a
// slab of slab_words<S>(n2) words: the word planes and, for H16, the plane of site scales.
template <class S>
__host__ __device__ __forceinline__ size_t slab_words(unsigned n2) {
    return (size_t)Traits<S>::NCW * n2 + (std::is_same<S, H16>::value ? n2 / 4 : 0);
}

// Direction loop of the in-block hops (hop_sum): unrolled for FP64 and FP32 storage, rolled for
// FP16 (unrolled it spills).
template <class S>
constexpr bool blk_hop_unroll() {
    return !std::is_same<S, H16>::value;
}

// Ainv (c + alpha H^k x) at odd half site j (x even).
template <class S>
__device__ __forceinline__ void odd_pass(unsigned n2, unsigned j, const typename Traits<S>::word* x,
                                         const typename Traits<S>::word* c, typename Traits<S>::real alpha,
                                         const EoFields<S>& F, const typename Traits<S>::kword* Ainv,
                                         cx<typename Traits<S>::real> w[12]) {
    typedef typename Traits<S>::real R;
    cx<R> acc[12];
    hop_sum<R, HOPS_INSIDE, blk_hop_unroll<S>()>(n2, j, x, F.U[1], F.U[0], F.nbr[1], acc, 8);
    if (c) {
        cx<R> cc[12];
        load_spinor(c, n2, j, cc);
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = cc[k] + alpha * acc[k];
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = alpha * acc[k];
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) w[k] = mk(R(0), R(0));
    apply_diag<R>(Ainv, n2, j, R(0), acc, w, R(0));
}

// [A_ee] c + beta H^k t at even half site i (t odd).
template <class S, bool USE_A>
__device__ __forceinline__ void even_pass(unsigned n2, unsigned i, const typename Traits<S>::word* c,
                                          const typename Traits<S>::word* t, typename Traits<S>::real beta,
                                          const EoFields<S>& F, typename Traits<S>::real mass4,
                                          cx<typename Traits<S>::real> y[12]) {
    typedef typename Traits<S>::real R;
    cx<R> cc[12];
    hop_sum<R, HOPS_INSIDE, blk_hop_unroll<S>()>(n2, i, t, F.U[0], F.U[1], F.nbr[0], y, 8);
    load_spinor(c, n2, i, cc);
    if (USE_A) {
        apply_diag<R>(F.K[0], n2, i, mass4, cc, y, beta);
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) y[k] = cc[k] + beta * y[k];
    }
}

__global__ __launch_bounds__(BE_MAX_THREADS) void k_blk_prep(Geom g, EoFields<double> F, const double2* __restrict__ Ainv,
                                                            const double2* __restrict__ b, double2* __restrict__ bpe,
                                                            double2* __restrict__ re, double2* __restrict__ xe,
                                                            double2* __restrict__ to, double* bb, double* rr,
                                                            int colour, int nrhs) {
    __shared__ double lds[16];
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const unsigned n2 = F.n2;
    const size_t of = (size_t)k.rhs * 12 * g.V, oh = (size_t)k.rhs * 12 * n2;
    double red[1] = {0};
    // odd pass: t_o = A_oo^-1 b_o ; ||b_o||^2
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned j = k.h0 + l, s = full_index(g, j, 1);
        cx<double> bo[12], w[12], z[12];
        load_spinor(b + of, g.V, s, bo);
        red[0] += acc_nrm(bo);
#pragma unroll
        for (int c = 0; c < 12; ++c) w[c] = z[c] = mk(0.0, 0.0);
        apply_diag<double>(Ainv, n2, j, 0.0, bo, w, 0.0);
        store_spinor(to + oh, n2, j, w);
    }
    __syncthreads();
    // even pass: b'_e = b_e + 1/2 H^k t_o ; r_e = b'_e ; x_e = 0 ; ||b_e||^2, ||r_e||^2
    double red2[1] = {0};
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned i = k.h0 + l, s = full_index(g, i, 0);
        cx<double> be[12], y[12], z[12];
        load_spinor(b + of, g.V, s, be);
        red[0] += acc_nrm(be);
        hop_sum<double, HOPS_INSIDE, true>(n2, i, to + oh, F.U[0], F.U[1], F.nbr[0], y, 8);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            y[c] = be[c] + 0.5 * y[c];
            z[c] = mk(0.0, 0.0);
        }
        store_spinor(bpe + oh, n2, i, y);
        store_spinor(re + oh, n2, i, y);
        store_spinor(xe + oh, n2, i, z);
        red2[0] += acc_nrm(y);
    }
    block_sum<1>(red, lds);
    block_sum<1>(red2, lds);
    if (threadIdx.x == 0) {
        bb[k.key] = red[0];
        rr[k.key] = red2[0];
    }
}

__global__ __launch_bounds__(BE_MAX_THREADS) void k_blk_resid(Geom g, EoFields<double> F, const double2* __restrict__ Ainv,
                                                             const double2* __restrict__ bpe, const double2* __restrict__ xe,
                                                             double2* __restrict__ re, double2* __restrict__ to, double* rr,
                                                             double mass4, int colour, int nrhs) {
    __shared__ double lds[16];
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const unsigned n2 = F.n2;
    const size_t oh = (size_t)k.rhs * 12 * n2;
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        cx<double> w[12];
        odd_pass<double>(n2, k.h0 + l, xe + oh, nullptr, 1.0, F, Ainv, w);
        store_spinor(to + oh, n2, k.h0 + l, w);
    }
    __syncthreads();
    double red[1] = {0};
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned i = k.h0 + l;
        cx<double> y[12], bv[12];
        even_pass<double, true>(n2, i, xe + oh, to + oh, -0.25, F, mass4, y);
        load_spinor(bpe + oh, n2, i, bv);
#pragma unroll
        for (int c = 0; c < 12; ++c) y[c] = bv[c] - y[c];
        store_spinor(re + oh, n2, i, y);
        red[0] += acc_nrm(y);
    }
    block_sum<1>(red, lds);
    if (threadIdx.x == 0) rr[k.key] = red[0];
}

// x = (x_e, x_o) on the blocks of the colour with x_o = A_oo^-1 (b_o + 1/2 H^k x_e), assembled
// from the two parts the FP64 passes already hold: to = A_oo^-1 b_o (k_blk_prep) and, when a
// residual pass ran on the final x_e, th = A_oo^-1 H^k x_e (k_blk_resid; th null when x_e = 0).
__global__ __launch_bounds__(BE_MAX_THREADS) void k_blk_recon(Geom g, const double2* __restrict__ to,
                                                             const double2* __restrict__ th,
                                                             const double2* __restrict__ xe, double2* __restrict__ x,
                                                             int colour, int nrhs) {
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const unsigned n2 = g.V / 2;
    const size_t of = (size_t)k.rhs * 12 * g.V, oh = (size_t)k.rhs * 12 * n2;
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned j = k.h0 + l;
        cx<double> w[12], e[12];
        load_spinor(to + oh, n2, j, w);
        if (th) {
            cx<double> h[12];
            load_spinor(th + oh, n2, j, h);
#pragma unroll
            for (int c = 0; c < 12; ++c) w[c] = w[c] + 0.5 * h[c];
        }
        store_spinor(x + of, g.V, full_index(g, j, 1), w);
        load_spinor(xe + oh, n2, j, e);
        store_spinor(x + of, g.V, full_index(g, j, 0), e);
    }
    // the solution is zero on the other colour: clear the block of the other colour with the same
    // rank (sites (B2 * Vb .. B2 * Vb + Vb) of the full field), so every such block is cleared once
    const unsigned s0 = (unsigned)((1 - colour) * g.NBc + k.rank) * (unsigned)g.Vb;
    const cx<double> z[12] = {};
#pragma unroll 1
    for (int l = threadIdx.x; l < g.Vb; l += blockDim.x) store_spinor(x + of, g.V, s0 + l, z);
}

template <class S>
struct BlkInner {
    typedef typename Traits<S>::word W;
    typedef typename Traits<typename Traits<S>::xs>::word XW;
    W *r, *rh, *p, *v, *t, *tmp;
    XW* e;  // the correction, in Traits<S>::xs
};

template <class R>
__device__ __forceinline__ cx<R> cdiv_r(cx<double> a, cx<double> b) {
    const double d = b.re * b.re + b.im * b.im;
    return mk((R)((a.re * b.re + a.im * b.im) / d), (R)((a.im * b.re - a.re * b.im) / d));
}

// v = M_k p on the block (two passes separated by a workgroup barrier), with the dot
// products requested: (rh, v) when DOT1, (v, p) and (v, v) when DOT2.
template <class S, int DOT>
__device__ __forceinline__ void apply_Mk(const Geom& g, const EoFields<S>& F, const typename Traits<S>::kword* Ainv,
                                         unsigned h0, size_t oR, const typename Traits<S>::word* in,
                                         typename Traits<S>::word* tmp, typename Traits<S>::word* out,
                                         const typename Traits<S>::word* rh, typename Traits<S>::real mass4,
                                         double red[3]) {
    typedef typename Traits<S>::real R;
    const unsigned n2 = F.n2;
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        cx<R> w[12];
        odd_pass<S>(n2, h0 + l, in + oR, nullptr, R(1), F, Ainv, w);
        store_spinor(tmp + oR, n2, h0 + l, w);
    }
    __syncthreads();
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned i = h0 + l;
        cx<R> y[12];
        even_pass<S, true>(n2, i, in + oR, tmp + oR, R(-0.25), F, mass4, y);
        store_spinor(out + oR, n2, i, y);
        if (DOT == 1) {
            cx<R> h[12];
            load_spinor(rh + oR, n2, i, h);
            acc_dot(h, y, red[0], red[1]);
        } else {
            cx<R> c[12];
            load_spinor(in + oR, n2, i, c);
            acc_dot(y, c, red[0], red[1]);
            red[2] += acc_nrm(y);
        }
    }
}

template <class S>
__global__ __launch_bounds__(be_inner_max<S>()) void k_blk_inner(Geom g, EoFields<S> F,
                                                             const typename Traits<S>::kword* __restrict__ Ainv,
                                                             const double2* __restrict__ re, double2* __restrict__ xe,
                                                             BlkInner<S> w, const double* __restrict__ bb,
                                                             const double* __restrict__ rr, double mass4, double tol,
                                                             double inner_floor, int maxit, int* iters, int colour,
                                                             int nrhs) {
    __shared__ double lds[3 * 16];
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const double b2 = bb[k.key], r2 = rr[k.key];
    if (!(b2 > 0) || !(r2 > tol * tol * b2) || !isfinite(r2)) return;  // uniform over the workgroup
    const unsigned n2 = F.n2;
    typedef typename Traits<S>::real R;
    typedef typename Traits<S>::xs XS;
    const size_t oh = (size_t)k.rhs * 12 * n2, oR = (size_t)k.rhs * slab_words<S>(n2),
                 oX = (size_t)k.rhs * Traits<XS>::NCW * n2;
    const R m4 = (R)mass4;
    const double rn = sqrt(r2), sc = 1.0 / rn;
    double eps = BI_AIM * tol * sqrt(b2) / rn;
    if (eps < inner_floor) eps = inner_floor;
    double red[3] = {0, 0, 0};
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned i = k.h0 + l;
        cx<double> a[12];
        cx<R> q[12];
        cx<XS> z[12];
        load_spinor(re + oh, n2, i, a);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            q[c] = mk((R)(sc * a[c].re), (R)(sc * a[c].im));
            z[c] = mk(XS(0), XS(0));
        }
        store_spinor(w.r + oR, n2, i, q);
        store_spinor(w.rh + oR, n2, i, q);
        store_spinor(w.p + oR, n2, i, q);
        store_spinor(w.e + oX, n2, i, z);
        red[0] += acc_nrm(q);
    }
    block_sum<1>(red, lds);
    cx<double> rho = mk(red[0], 0.0);
    const double thr2 = eps * eps * red[0];
    int it = 0;
    while (it < maxit) {
        red[0] = red[1] = red[2] = 0;
        apply_Mk<S, 1>(g, F, Ainv, k.h0, oR, w.p, w.tmp, w.v, w.rh, m4, red);
        block_sum<2>(red, lds);
        if (!(red[0] * red[0] + red[1] * red[1] > 0)) break;
        const cx<R> alpha = cdiv_r<R>(rho, mk(red[0], red[1]));
        // s = r - alpha v (kept in r)
#pragma unroll 1
        for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
            const unsigned i = k.h0 + l;
            cx<R> a[12], vv[12];
            load_spinor(w.r + oR, n2, i, a);
            load_spinor(w.v + oR, n2, i, vv);
#pragma unroll
            for (int c = 0; c < 12; ++c) a[c] = a[c] - alpha * vv[c];
            store_spinor(w.r + oR, n2, i, a);
        }
        __syncthreads();
        red[0] = red[1] = red[2] = 0;
        apply_Mk<S, 2>(g, F, Ainv, k.h0, oR, w.r, w.tmp, w.t, nullptr, m4, red);
        block_sum<3>(red, lds);
        cx<R> omega = mk(R(0), R(0));
        if (red[2] > 0) omega = mk((R)(red[0] / red[2]), (R)(red[1] / red[2]));
        // e += alpha p + omega s ; r = s - omega t ; (rh, r), (r, r)
        red[0] = red[1] = red[2] = 0;
#pragma unroll 1
        for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
            const unsigned i = k.h0 + l;
            cx<XS> ee[12];
            cx<R> pp[12], ss[12], tt[12];
            load_spinor(w.e + oX, n2, i, ee);
            load_spinor(w.p + oR, n2, i, pp);
            load_spinor(w.r + oR, n2, i, ss);
            load_spinor(w.t + oR, n2, i, tt);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                const cx<R> d = alpha * pp[c] + omega * ss[c];
                ee[c] = ee[c] + mk((XS)d.re, (XS)d.im);
                ss[c] = ss[c] - omega * tt[c];
            }
            store_spinor(w.e + oX, n2, i, ee);
            store_spinor(w.r + oR, n2, i, ss);
            load_spinor(w.rh + oR, n2, i, pp);
            acc_dot(pp, ss, red[0], red[1]);
            red[2] += acc_nrm(ss);
        }
        block_sum<3>(red, lds);
        ++it;
        if (red[2] <= thr2 || !isfinite(red[2])) break;
        if (omega.re == R(0) && omega.im == R(0)) break;
        const double d1 = rho.re * rho.re + rho.im * rho.im;
        if (!(d1 > 0)) break;
        const cx<double> q = mk((red[0] * rho.re + red[1] * rho.im) / d1, (red[1] * rho.re - red[0] * rho.im) / d1);
        const double d2 = (double)omega.re * omega.re + (double)omega.im * omega.im;
        const cx<double> ao = mk(((double)alpha.re * omega.re + (double)alpha.im * omega.im) / d2,
                                 ((double)alpha.im * omega.re - (double)alpha.re * omega.im) / d2);
        const cx<R> beta = mk((R)(q.re * ao.re - q.im * ao.im), (R)(q.re * ao.im + q.im * ao.re));
        rho = mk(red[0], red[1]);
#pragma unroll 1
        for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
            const unsigned i = k.h0 + l;
            cx<R> a[12], pp[12], vv[12];
            load_spinor(w.r + oR, n2, i, a);
            load_spinor(w.p + oR, n2, i, pp);
            load_spinor(w.v + oR, n2, i, vv);
#pragma unroll
            for (int c = 0; c < 12; ++c) pp[c] = a[c] + beta * (pp[c] - omega * vv[c]);
            store_spinor(w.p + oR, n2, i, pp);
        }
        __syncthreads();
    }
    // x_e += ||r_e|| e in FP64
#pragma unroll 1
    for (int l = threadIdx.x; l < g.hvb; l += blockDim.x) {
        const unsigned i = k.h0 + l;
        cx<XS> e[12];
        cx<double> x[12];
        load_spinor(w.e + oX, n2, i, e);
        load_spinor(xe + oh, n2, i, x);
#pragma unroll
        for (int c = 0; c < 12; ++c) x[c] = x[c] + mk(rn * (double)e[c].re, rn * (double)e[c].im);
        store_spinor(xe + oh, n2, i, x);
    }
    if (threadIdx.x == 0) iters[k.key] += it;
}

// ------------------------------------------------------------------ LDS-resident inner solver
// Minimal residual on M_k, one workgroup per (block, RHS), for block parities of at most BL_MAX sites:
//     t = M_k r, omega = (t, r) / (t, t), e += omega r, r -= omega t.
// The Dirichlet operators of the blocks are well conditioned, and it needs as many operator applications
// as BiCGStab (to 2e-6: 19 against 20 at kappa = 0.1205, 22 / 22 at 0.125, 26 / 24 at 0.129; 6^4 blocks, eps = 0.3 links)
// with one vector kept beside r.  A block whose residual falls by less than the gain expected of BL_WINDOW steps
// is left where it stands and marked in the second half of iters, and the caller goes on with BI: BiCGStab in the same
// layout, with p (then s) as the operand and rh, p and e as slabs, r in registers until s is formed and v in its
// place until p is updated.
//
// One thread per local half index l < hvb owns the even site and the odd site of that index.  r (the
// operand of M_k; even sites) and the odd intermediate A_oo^-1 H^k_oe r are staged in LDS
// (2 x (hvb + 1) x 96 bytes, 124 KB for a 6^4 block), so the in-block neighbour gathers of both passes
// are LDS reads; e stays in registers.  Links (packed, five loads each) and clover are read from
// global memory: the RHS of one block run on one XCD and share them in its L2.  Arithmetic FP32, dot
// products accumulated in FP64.
//
// What bounds it: one 11-wave workgroup per CU (6^4) issues vector loads and ALU work in barrier-
// separated phases, 1.7 KB of links and clover and 3300 vector
// instructions a site and step.  Time per launch at 48x24^3,
// 6^4, 12 RHS, one colour (to 2e-6, then to tol = 1e-10): BiCGStab with entry-major links (nine 8-byte
// loads each), five global vectors, conditional hops and shuffle reductions 5677 us; 4883 us with r and v in
// registers and branch-free hops; 4296 us with the packed links; 4002 us with the exchanging
// reduction; 3500 us with minimal residual to a quarter of tol, 3990 us to MR_AIM_LDS of it.  With no global loads but the same LDS reads and ALU work the BiCGStab
// took 3000 us: the load path, 64 bytes a cycle and CU, is the rest.
constexpr int BL_MAX = 768;     // 12 waves: 3 per SIMD at up to 168 VGPRs
constexpr int BL_WINDOW = 8;    // steps
// The fall of ||r|| in a window below which a block is left to BiCGStab: 0.1 decades a step, where the two meet.  One colour
// to 1e-10, BiCGStab alone / minimal residual left at 0.05 decades a step for k_blk_inner / this: 6^4 blocks of
// 24x12^3, 12 RHS, kappa 0.13 1.71 / 1.30 / 1.40, 0.14 2.17 / 2.39 / 1.60, 0.16 6.53 / 9.59 / 5.37 ms; 4^4 of 16^4, 8 RHS,
// 0.14 1.22 / 0.96 / 1.01, 0.15 1.39 / 1.33 / 1.49, 0.16 1.65 / 2.42 / 1.27 ms.  In k_blk_mr with FP32 storage 0.15 decades
// (BiCGStab alone / this): 8^4 of 16^4, 8 RHS, 0.1205 4.9 / 4.4, 0.13 6.7 / 7.0, 0.14 9.7 / 9.8 ms.  A whole lattice (WRAP) goes on
// by launches of the global solver, at two to four times the time an iteration, so it stays until 0.05 decades a step
// (4^4, 8 RHS, kappa 0.13: 3.03 / - / 1.18 ms).
constexpr double BL_GAIN = 0.16, BL_GAIN_WRAP = 0.4, BM_GAIN32 = 0.06;

// Exchanges halves between a and b and adds, on the two dwords of each double: with W = 32 the lower 32
// lanes get a(lane) + a(lane + 32) and the upper ones b(lane - 32) + b(lane); with W = 16 the same
// within each pair of 16-lane rows.
template <int W>
__device__ __forceinline__ double swap_add(double a, double b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
    u2 p, q;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (W == 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false);
            p[i] = r[0], q[i] = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane16_swap(x[i], y[i], false, false);
            p[i] = r[0], q[i] = r[1];
        }
    }
    return __builtin_bit_cast(double, p) + __builtin_bit_cast(double, q);
}
// v(lane) + v(lane rotated by N inside its 16-lane row)
template <int N>
__device__ __forceinline__ double ror_add(double v) {
    typedef int i2 __attribute__((ext_vector_type(2)));
    const i2 x = __builtin_bit_cast(i2, v);
    i2 y;
#pragma unroll
    for (int i = 0; i < 2; ++i) y[i] = __builtin_amdgcn_update_dpp(0, x[i], 0x120 + N, 0xf, 0xf, false);
    return v + __builtin_bit_cast(double, y);
}
__device__ __forceinline__ double row_sum(double v) { return ror_add<1>(ror_add<2>(ror_add<4>(ror_add<8>(v)))); }

// Sums of NV <= 8 values over the workgroup (full waves, at most 16), in a fixed order, with one
// barrier.  Inside a wave the values are exchanged against each other, so that each step halves the
// values a lane carries (about 40 instructions for eight values, against 144 and the LDS permutes
// of one shuffle tree per value), and the waves' sums are added the same way, one value per
// 16-lane row.  lds holds 8 x 16 doubles, zero in the slots of waves that do not exist, and must not be the
// slot of the previous call (alternate two slots).
template <int NV>
__device__ __forceinline__ void wg_sums(double v[NV], double* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int NP = NV > 4 ? 4 : NV > 2 ? 2 : 1;  // values per half wave
    double h[4], w[2];
#pragma unroll
    for (int k = 0; k < NP; ++k) h[k] = swap_add<32>(v[k], k + NP < NV ? v[k + NP] : v[k]);
    constexpr int NQ = NP > 2 ? 2 : 1;  // values per row
#pragma unroll
    for (int k = 0; k < NQ; ++k) w[k] = row_sum(swap_add<16>(h[k], NP > NQ ? h[k + NQ] : h[k]));
    // row r = lane / 16 holds value NP (r / 2) + NQ (r % 2) + k (NP > NQ), the same in both rows of a half otherwise
    const int r = lane >> 4, k0 = NP * (r >> 1) + (NP > NQ ? NQ * (r & 1) : 0);
    if ((lane & 15) == 0) {
#pragma unroll
        for (int k = 0; k < NQ; ++k)
            if (k0 + k < NV) lds[(k0 + k) * 16 + wave] = w[k];
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NV; b += 4) {
        const double s = row_sum(lds[b * 16 + lane]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (b + k < NV) {
                typedef int i2 __attribute__((ext_vector_type(2)));
                const i2 x = __builtin_bit_cast(i2, s);
                i2 y;
                y[0] = __builtin_amdgcn_readlane(x[0], 16 * k);
                y[1] = __builtin_amdgcn_readlane(x[1], 16 * k);
                v[b + k] = __builtin_bit_cast(double, y);
            }
    }
}

// Block field in LDS, one 96-byte record per site: a record has one address register and the rest
// in the offsets of its six 16-byte words (consecutive lanes' words of a record pitch of 24 banks
// fall on distinct banks for the eight lanes that are served together).
__device__ __forceinline__ void lds_load(const float4* __restrict__ L, unsigned li, cx<float> q[12]) {
    const float4* p = L + li * 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float4 w = p[k];
        q[2 * k] = mk(w.x, w.y);
        q[2 * k + 1] = mk(w.z, w.w);
    }
}
__device__ __forceinline__ void lds_store(float4* __restrict__ L, unsigned li, const cx<float> q[12]) {
    float4* p = L + li * 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) p[k] = make_float4(q[2 * k].re, q[2 * k].im, q[2 * k + 1].re, q[2 * k + 1].im);
}

// Local half indices of the in-block neighbours of one site, packed two per register; a hop that
// leaves the block has index HV, the record of zeros after the block's sites in LDS.
// WRAP (the whole lattice): no hop leaves, and bit 15 marks one across an antiperiodic time boundary (d < 2).
template <bool WRAP>
struct BlkNbr {
    unsigned w[4];
    __device__ __forceinline__ unsigned operator[](int d) const {
        const unsigned e = (d & 1) ? w[d >> 1] >> 16 : w[d >> 1] & 0xffffu;
        return WRAP && d < 2 ? e & 0x7fffu : e;
    }
    __device__ __forceinline__ bool flip(int d) const { return WRAP && d < 2 && (w[d >> 1] & (d ? 0x80000000u : 0x8000u)); }
};
template <bool WRAP>
__device__ __forceinline__ BlkNbr<WRAP> blk_nbr(const int* __restrict__ nbr, unsigned n2, unsigned s, unsigned h0, unsigned HV,
                                          bool act) {
    BlkNbr<WRAP> b;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        unsigned li[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = at(nbr + (size_t)(2 * k + q) * n2, s);
            const unsigned t = (e < 0 ? (unsigned)~e : (unsigned)e) - h0;
            li[q] = act && t < HV ? t : HV;
            if (WRAP && e < 0) li[q] |= 0x8000u;
        }
        b.w[k] = li[0] | (li[1] << 16);
    }
    return b;
}

// acc = sum over the in-block hops of the site with link byte offset own and neighbours nb, of
// (1 -+ g_mu) W q(neighbour), q read from LDS; forward links Uf at own, backward links Ub at the
// neighbour (packed links; own and the operand's h0 + neighbour index the whole half field).  A hop that leaves the block
// reads the record of zeros (and some link of the block), so every hop runs without a branch: the
// waves of a block take nearly every hop for some lane anyway, and as straight-line code the link of hop
// d + 1 is loaded while d is computed.  (In-block hops never cross the time boundary,
// whose sign the table carries: there are at least two blocks per direction.)
template <bool WRAP>
__device__ __forceinline__ void lds_hops(unsigned n2, unsigned h0, unsigned own, BlkNbr<WRAP> nb, unsigned HV,
                                         const float4* __restrict__ L, const char* Uf, const char* Ub,
                                         cx<float> acc[12]) {
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = mk(0.f, 0.f);
    PackedLinks<float> pf(fresh(Uf), n2), pb(fresh(Ub), n2);
    cx<float> u[9];
    pf.next(reissue(own), u);
    // (opaque here, so that the sixteen addresses formed from nb are not kept across the iteration loop)
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(nb.w[k]));
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        cx<float> un[9], q[12];
        lds_load(L, nb[d], q);
        if (WRAP && d < 2) {
            const float sg = nb.flip(d) ? -1.f : 1.f;
#pragma unroll
            for (int c = 0; c < 12; ++c) q[c] = sg * q[c];
        }
        if (d + 1 < 8) {
            const unsigned t = reissue(nb[d + 1]);
            if ((d + 1) & 1)
                pb.next(byte_offset(h0 + (t < HV ? t : 0u), 16), un);
            else
                pf.next(reissue(own), un);
        }
        __builtin_amdgcn_sched_barrier(0);
        hop_dispatch<float>(d, u, q, acc);
        pin(acc);
#pragma unroll
        for (int k = 0; k < 9; ++k) u[k] = un[k];
    }
}

// WRAP: the same for the whole lattice as one block with its boundary conditions, one workgroup per RHS (hvb = V / 2).
template <bool WRAP, bool BI>
__global__ __launch_bounds__(BL_MAX) void k_blk_lds(Geom g, EoFields<float> F, const float4* __restrict__ Ainv,
                                                    const double2* re, double2* xe, float4* rhg, float4* pg, float4* eg,
                                                    const double* __restrict__ bb, const double* __restrict__ rr,
                                                    double mass4, double tol, double aim, double inner_floor, int maxit,
                                                    int* iters, int colour, int nrhs) {
    extern __shared__ float4 bl_lds[];
    __shared__ double red_lds[2][8 * 16];  // alternating slots of the workgroup reductions
    constexpr double GAIN = WRAP ? BL_GAIN_WRAP : BL_GAIN;
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const double b2 = bb[k.key], r2 = rr[k.key];
    if (!(b2 > 0) || !(r2 > tol * tol * b2) || !isfinite(r2)) return;  // uniform over the workgroup
    const unsigned n2 = F.n2, HV = (unsigned)g.hvb, h0 = k.h0;
    float4* op = bl_lds;          // operand of M_k on the even sites of the block
    float4* tp = bl_lds + 6 * (HV + 1);  // A_oo^-1 H^k_oe (operand) on the odd sites
    // l: local half index of this thread's even and odd site.  The last wave's threads past the block
    // run the same code on the record of zeros (their stores are masked), so that the passes have no
    // divergent branches.
    const bool act = threadIdx.x < HV;
    const unsigned l = act ? threadIdx.x : HV, lg = act ? threadIdx.x : 0u;
    const unsigned lo = byte_offset(lg, 16), own = byte_offset(h0 + lg, 16);  // its byte offsets in the planes
    const size_t oh = (size_t)k.rhs * 12 * n2 + h0;
    // everything below is addressed from the block's first site
    re += oh;
    xe += oh;
    const char *Ue = F.W[0], *Uo = F.W[1];
    const float4 *Ke = F.K[0] + h0, *Ko = Ainv + h0;
    const BlkNbr<WRAP> ne = blk_nbr<WRAP>(F.nbr[0], n2, h0 + lg, h0, HV, act), no = blk_nbr<WRAP>(F.nbr[1], n2, h0 + lg, h0, HV, act);
    for (unsigned k = threadIdx.x; k < 2 * 8 * 16; k += blockDim.x) red_lds[0][k] = 0;
    if (threadIdx.x < 12) (threadIdx.x < 6 ? op : tp)[HV * 6 + threadIdx.x % 6] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    const float m4 = (float)mass4;
    if (BI) {
        const size_t oR = (size_t)k.rhs * 6 * n2 + h0;
        rhg += oR;
        pg += oR;
        eg += oR;
    }
    // tp = A_oo^-1 H^k_oe q on the odd sites (q: operand in op)
    auto odd = [&]() {
        cx<float> acc[12], w[12];
        UDiag<float> K(fresh(Ko), n2, lo);
        lds_hops<WRAP>(n2, h0, own, no, HV, op, Uo, Ue, acc);
#pragma unroll
        for (int c = 0; c < 12; ++c) w[c] = mk(0.f, 0.f);
        K.off = reissue(lo), K.first();
        K.apply(0.f, acc, w, 0.f);
        if (act) lds_store(tp, l, w);
    };
    // y = (4 + m + C) c - 1/4 H^k_eo q_o on the even sites (c: this site's operand; q_o in tp)
    auto even = [&](cx<float> y[12], cx<float> c[12]) {
        UDiag<float> K(fresh(Ke), n2, lo);
        lds_hops<WRAP>(n2, h0, own, ne, HV, tp, Ue, Uo, y);
        lds_load(op, l, c);
        K.off = reissue(lo), K.first();
        K.apply(m4, c, y, -0.25f);
    };
    const double rn = sqrt(r2), sc = 1.0 / rn;
    double eps = aim * tol * sqrt(b2) / rn;
    if (eps < inner_floor) eps = inner_floor;
    int phase = 0;  // reduction slot
    double red[8];
    cx<float> r[12], e[12];  // (BI: v in r from s on; e, the correction, otherwise)
    {
        cx<double> a[12];
        uload_spinor(re, n2, lo, a);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            r[c] = act ? mk((float)(sc * a[c].re), (float)(sc * a[c].im)) : mk(0.f, 0.f);
            e[c] = mk(0.f, 0.f);
        }
        if (act) lds_store(op, l, r);
        if (BI && act) {
            ustore_spinor(fresh(rhg), n2, lo, r);
            ustore_spinor(fresh(pg), n2, lo, r);
            ustore_spinor(fresh(eg), n2, lo, e);
        }
        red[0] = acc_nrm(r);
    }
    wg_sums<1>(red, red_lds[phase ^= 1]);  // (its barrier also publishes the operand)
    const double thr2 = eps * eps * red[0];
    double window = red[0];  // ||r||^2 when the current window began
    cx<double> rho = mk(red[0], 0.0);
    int it = 0;
    bool slow = false;
    while (BI && it < maxit) {
        // v = M_k p, (rh, v)
        odd();
        __syncthreads();
        red[0] = red[1] = 0;
        cx<float> v[12];
        {
            cx<float> c[12], h[12];
            even(v, c);
            uload_spinor(fresh(rhg), n2, lo, h);
            if (act) acc_dot(h, v, red[0], red[1]);
        }
        wg_sums<2>(red, red_lds[phase ^= 1]);
        if (!(red[0] * red[0] + red[1] * red[1] > 0)) break;
        const cx<float> alpha = cdiv_r<float>(rho, mk(red[0], red[1]));
        // s = r - alpha v, staged as the operand
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const cx<float> sv = r[c] - alpha * v[c];
            r[c] = v[c];
            v[c] = sv;
        }
        if (act) lds_store(op, l, v);
        __syncthreads();
        // t = M_k s, (t, s), (t, t), (rh, s), (rh, t), (s, s)
        odd();
        __syncthreads();
        cx<float> t[12], pp[12];
        {
            cx<float> sv[12], h[12];
            even(t, sv);
            uload_spinor(fresh(rhg), n2, lo, h);
#pragma unroll
            for (int c = 0; c < 8; ++c) red[c] = 0;
            if (act) {
                acc_dot(t, sv, red[0], red[1]);
                red[2] = acc_nrm(t);
                acc_dot(h, sv, red[3], red[4]);
                acc_dot(h, t, red[5], red[6]);
                red[7] = acc_nrm(sv);
            }
            // (needed after the reduction)
            uload_spinor(fresh(eg), n2, lo, e);
            uload_spinor(fresh(pg), n2, lo, pp);
        }
        wg_sums<8>(red, red_lds[phase ^= 1]);
        ++it;
        cx<float> omega = mk(0.f, 0.f);
        if (red[2] > 0) omega = mk((float)(red[0] / red[2]), (float)(red[1] / red[2]));
        // r = s - omega t is orthogonal to t, so ||r||^2 = (s, s) - |(t, s)|^2 / (t, t); the next
        // rho = (rh, r) = (rh, s) - omega (rh, t): one reduction serves omega, the stopping test and
        // beta, and x, r and p are updated in one pass
        const double r2n = red[2] > 0 ? red[7] - (red[0] * red[0] + red[1] * red[1]) / red[2] : red[7];
        const cx<double> rn_ = mk(red[3] - ((double)omega.re * red[5] - (double)omega.im * red[6]),
                                  red[4] - ((double)omega.re * red[6] + (double)omega.im * red[5]));
        const double d1 = rho.re * rho.re + rho.im * rho.im;
        const double d2 = (double)omega.re * omega.re + (double)omega.im * omega.im;
        const bool stop = r2n <= thr2 || !isfinite(r2n) || !(d2 > 0) || !(d1 > 0);
        cx<float> beta = mk(0.f, 0.f);
        if (!stop) {
            const cx<double> q = mk((rn_.re * rho.re + rn_.im * rho.im) / d1, (rn_.im * rho.re - rn_.re * rho.im) / d1);
            const cx<double> ao = mk(((double)alpha.re * omega.re + (double)alpha.im * omega.im) / d2,
                                     ((double)alpha.im * omega.re - (double)alpha.re * omega.im) / d2);
            beta = mk((float)(q.re * ao.re - q.im * ao.im), (float)(q.re * ao.im + q.im * ao.re));
        }
        rho = rn_;
        // e += alpha p + omega s ; r = s - omega t ; p = r + beta (p - omega v), staged as the next operand
        lds_load(op, l, v);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            e[c] = e[c] + (alpha * pp[c] + omega * v[c]);
            v[c] = v[c] - omega * t[c];
        }
        if (act) ustore_spinor(fresh(eg), n2, lo, e);
        if (stop) break;
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            pp[c] = v[c] + beta * (pp[c] - omega * r[c]);
            r[c] = v[c];
        }
        if (act) {
            ustore_spinor(fresh(pg), n2, lo, pp);
            // (only this thread reads its own operand record after the last barrier)
            lds_store(op, l, pp);
        }
        __syncthreads();
    }
    while (!BI && it < maxit) {
        // t = M_k r, (t, r), (t, t), (r, r)
        odd();
        __syncthreads();
        cx<float> t[12];
        even(t, r);
        red[0] = red[1] = 0;
        acc_dot(t, r, red[0], red[1]);
        red[2] = acc_nrm(t);
        red[3] = acc_nrm(r);
        wg_sums<4>(red, red_lds[phase ^= 1]);
        ++it;
        slow = !(red[2] > 0);
        if (slow) break;
        // e += omega r, r -= omega t with the omega that minimises ||r||, staged as the next operand
        const cx<float> omega = mk((float)(red[0] / red[2]), (float)(red[1] / red[2]));
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            cmadd(e[c], omega, r[c]);
            cmadd(r[c], mk(-omega.re, -omega.im), t[c]);
        }
        const double r2n = red[3] - (red[0] * red[0] + red[1] * red[1]) / red[2];
        slow = !isfinite(r2n) || (r2n > thr2 && it % BL_WINDOW == 0 && r2n > GAIN * GAIN * window);
        if (!(r2n > thr2) || slow) break;
        if (it % BL_WINDOW == 0) window = r2n;
        // (only this thread reads its own operand record after the last barrier)
        if (act) lds_store(op, l, r);
        __syncthreads();
    }
    // x_e += ||r_e|| e in FP64
    if (act) {
        cx<double> x[12];
        if (BI) uload_spinor(fresh(eg), n2, lo, e);
        uload_spinor(xe, n2, lo, x);
#pragma unroll
        for (int c = 0; c < 12; ++c) x[c] = x[c] + mk(rn * (double)e[c].re, rn * (double)e[c].im);
        ustore_spinor(xe, n2, lo, x);
    }
    if (threadIdx.x == 0) {
        iters[k.key] += BI ? it : (it + 1) / 2;
        iters[gridDim.x + k.key] = slow;
    }
}

// ------------------------------------------------------------------ two or four lanes per site
// The iteration of k_blk_lds for launches that would leave SIMDs or lanes idle: there a step takes as long as one
// wavefront needs to issue it (3300 vector instructions, of four cycles each), so the work of a site is shared by
// two or four lanes.  Lane bit 0 is the spin s of the half spinors: h_s = psi_s + c psi_p with
// p = 2 + s (mu = 0, 3) or 3 - s (mu = 1, 2) needs nothing of the other half, and c^* W h_s goes back to spin p.  Lane bit 1
// (of four) is a pair of directions, (0, 1) or (3, 2) in this order, so that p is the same for both lanes of a slot
// and only the constant c differs.  Exchanges between neighbouring lanes add the sums and turn them into chiral
// halves (spins 0, 1 or 2, 3), on which a lane applies its clover block, the same in both lanes of bit 1.  The links
// of a lane in either parity stay in registers for the whole solve.
// One launch on 4^4 (128 sites a parity, two lanes), 8 RHS: 256 -> 187 us; on its 2^4 blocks (8 sites, four lanes), one
// colour: 53 -> 30 us.
constexpr int BQ_THREADS = 256;  // one wavefront per SIMD, so that the links fit its registers
constexpr int CU_COUNT = 256;

template <int N>  // v of the lane with bits N flipped (inside a quad)
__device__ __forceinline__ float quad_xor(float v) {
    constexpr int perm = (0 ^ N) | (1 ^ N) << 2 | (2 ^ N) << 4 | (3 ^ N) << 6;
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), perm, 0xf, 0xf, false));
}
template <int N>
__device__ __forceinline__ cx<float> quad_xor(cx<float> v) {
    return mk(quad_xor<N>(v.re), quad_xor<N>(v.im));
}

template <bool WRAP, int LANES>
__global__ __launch_bounds__(BQ_THREADS, LANES == 4 ? 2 : 1) void k_lds_lanes(Geom g, EoFields<float> F, const float4* Ainv, const double2* re,
                                                        double2* xe, const double* bb, const double* rr, double mass4,
                                                        double tol, double aim, double inner_floor, int maxit, int* iters, int colour,
                                                        int nrhs) {
    extern __shared__ float2 bq_lds[];  // the operand and the odd intermediate: records of four spins
    __shared__ double red_lds[2][8 * 16];
    constexpr int NS = 16 / LANES;  // directions of a lane
    constexpr double GAIN = WRAP ? BL_GAIN_WRAP : BL_GAIN;
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const double b2 = bb[k.key], r2 = rr[k.key];
    if (!(b2 > 0) || !(r2 > tol * tol * b2) || !isfinite(r2)) return;  // uniform over the workgroup
    const unsigned n2 = F.n2, HV = (unsigned)g.hvb, h0 = k.h0;
    const unsigned s = threadIdx.x & 1, dg = LANES == 4 ? (threadIdx.x >> 1) & 1 : 0u;
    const bool act = threadIdx.x / LANES < HV;
    const unsigned l = act ? threadIdx.x / LANES : HV, own = h0 + (act ? l : 0u);
    float2 *op = bq_lds, *tp = bq_lds + 12 * (HV + 1);
    for (unsigned q = threadIdx.x; q < 2 * 8 * 16; q += blockDim.x) red_lds[0][q] = 0;
    if (threadIdx.x < 24) (threadIdx.x < 12 ? op : tp)[12 * HV + threadIdx.x % 12] = make_float2(0.f, 0.f);
    // the slots of a lane: hops along 0, (3,) 1 (and 2), or along 3 and 2 with bit 1 set; the links of both parities, with
    // the sign of a time boundary
    auto direction = [&](int q) -> unsigned { return LANES == 4 ? (dg ? q ^ 6 : q) : q < 2 ? q : q < 4 ? q + 4 : q - 2; };
    cx<float> u[2][NS][9];
    unsigned nb[2][NS / 2];  // LDS records of the neighbours, two per register
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const unsigned d = direction(q);
            const int e = F.nbr[p][(size_t)d * n2 + own];
            const unsigned t = (e < 0 ? (unsigned)~e : (unsigned)e) - h0;
            const unsigned li = act && t < HV ? t : HV;
            nb[p][q >> 1] = (q & 1) ? nb[p][q >> 1] | li << 16 : li;
            const unsigned at = (q & 1) ? h0 + (li < HV ? li : 0u) : own;
            const char* base = F.W[(q & 1) ? 1 - p : p] + (size_t)(d >> 1) * packed_link_bytes<float>() * n2;
            const float sg = WRAP && e < 0 ? -1.f : 1.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 w = ((const float4*)base)[(size_t)j * n2 + at];
                u[p][q][2 * j] = mk(sg * w.x, sg * w.y);
                u[p][q][2 * j + 1] = mk(sg * w.z, sg * w.w);
            }
            const float2 w = ((const float2*)(base + (size_t)64 * n2))[at];
            u[p][q][8] = mk(sg * w.x, sg * w.y);
        }
    // c of a forward hop: 1 (mu = 0), i (mu = 1), sg (mu = 2), i sg (mu = 3)
    const float sg = s ? -1.f : 1.f;
    const cx<float> c0 = dg ? mk(0.f, sg) : mk(1.f, 0.f), c2 = dg ? mk(sg, 0.f) : mk(0.f, 1.f);
    // x += c z (four lanes), or its part for a c known to be real or imaginary, and x += c^* z
    auto add_c = [&](cx<float>& x, int q, cx<float> z, bool conj) {
        const float sign = (q & 1) ? -1.f : 1.f;
        if (LANES == 4) {
            const cx<float> cf = q < 2 ? c0 : c2, c = mk(sign * cf.re, sign * cf.im);
            if (conj)
                cjmadd(x, c, z);
            else
                cmadd(x, c, z);
        } else {
            const int mu = (int)direction(q) >> 1;
            const float c = sign * (mu >= 2 ? sg : 1.f) * (conj && (mu & 1) ? -1.f : 1.f);
            if (mu & 1)
                x = mk(fmad(-c, z.im, x.re), fmad(c, z.re, x.im));
            else
                x = mk(fmad(c, z.re, x.re), fmad(c, z.im, x.im));
        }
    };
    // y = the hops of parity p from L, this lane's chiral half
    auto hops = [&](int p, const float2* L, cx<float> y[6]) {
        cx<float> up[3], lo[2][3];
#pragma unroll
        for (int a = 0; a < 3; ++a) up[a] = lo[0][a] = lo[1][a] = mk(0.f, 0.f);
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const unsigned li = (q & 1) ? nb[p][q >> 1] >> 16 : nb[p][q >> 1] & 0xffffu;
            const float2 *r0 = L + 12 * li + 3 * s, *r1 = L + 12 * li + 3 * (q < NS / 2 ? 2 + s : 3 - s);
            cx<float> h[3], w[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float2 x = r0[a], z = r1[a];
                h[a] = mk(x.x, x.y);
                add_c(h[a], q, mk(z.x, z.y), false);
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                w[a] = mk(0.f, 0.f);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    if (q & 1)
                        cjmadd(w[a], u[p][q][3 * b + a], h[b]);
                    else
                        cmadd(w[a], u[p][q][3 * a + b], h[b]);
                }
                up[a] = up[a] + w[a];
                add_c(lo[q >= NS / 2][a], q, w[a], true);
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            // spin 2 + s from the first half of the slots here and the second half of the other spin; all directions
            cx<float> v = lo[0][a] + quad_xor<1>(lo[1][a]);
            if (LANES == 4) up[a] = up[a] + quad_xor<2>(up[a]), v = v + quad_xor<2>(v);
            // spins (s, 2 + s) -> (0, 1) for s = 0, (2, 3) for s = 1
            const cx<float> x = quad_xor<1>(s ? up[a] : v);
            y[a] = s ? x : up[a];
            y[3 + a] = s ? v : x;
        }
    };
    // the words with a chiral half's diagonal and off-diagonal reals are planes s, s + 1 and 3 + 7 s to 10 + 7 s
    const unsigned kd = byte_offset(own + s * n2, 16), ko = byte_offset(own + 7 * s * n2, 16);
    // (two lanes, one wavefront per SIMD: loaded before the hops, whose time hides them: 216 -> 187 us on 4^4)
    constexpr bool EARLY = LANES == 2;
    auto load_diag = [&](const float4* K, float w[40]) {
        Planes qd(fresh(K), n2), qo(fresh(K), n2, 3);
        const unsigned od = reissue(kd), oo = reissue(ko);
#pragma unroll
        for (int j = 0; j < 10; ++j) {
            const f4v x = j < 2 ? qd.load<f4v>(od) : qo.load<f4v>(oo);
            w[4 * j] = x[0], w[4 * j + 1] = x[1], w[4 * j + 2] = x[2], w[4 * j + 3] = x[3];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // y = (m4 + C) v + hsc y on the chiral half
    auto diag = [&](const float w[40], float m4, const cx<float> v[6], cx<float> y[6], float hsc) {
        float d[6], o[30];
#pragma unroll
        for (int j = 0; j < 6; ++j) d[j] = s ? w[j + 2] : w[j];
#pragma unroll
        for (int j = 0; j < 30; ++j) o[j] = s ? w[j + 10] : w[j + 8];
        diag_block<float>(d, o, m4, v, y, hsc);
    };
    auto store = [&](float2* L, const cx<float> v[6]) {
        if (act && !dg) {
#pragma unroll
            for (int a = 0; a < 6; ++a) L[12 * l + 6 * s + a] = make_float2(v[a].re, v[a].im);
        }
    };
    const float m4 = (float)mass4;
    const double rn = sqrt(r2), sc = 1.0 / rn;
    double eps = aim * tol * sqrt(b2) / rn;
    if (eps < inner_floor) eps = inner_floor;
    const size_t oh = (size_t)k.rhs * 12 * n2 + (size_t)(6 * s) * n2 + own;
    cx<float> e[6], r[6];
    int phase = 0;
    // (with four lanes every value counts twice in the sums: only their ratios matter)
    double red[4] = {0, 0, 0, 0};
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        const double2 x = re[oh + (size_t)a * n2];
        r[a] = act ? mk((float)(sc * x.x), (float)(sc * x.y)) : mk(0.f, 0.f);
        e[a] = mk(0.f, 0.f);
        red[0] += (double)(r[a].re * r[a].re + r[a].im * r[a].im);
    }
    store(op, r);
    __syncthreads();
    wg_sums<1>(red, red_lds[phase ^= 1]);
    const double thr2 = eps * eps * red[0];
    double window = red[0];
    int it = 0;
    bool slow = false;
    while (it < maxit) {
        cx<float> t[6], w[6];
        float kw[40];
        if (EARLY) load_diag(Ainv, kw);
        hops(1, op, t);
        if (!EARLY) load_diag(Ainv, kw);
#pragma unroll
        for (int a = 0; a < 6; ++a) w[a] = mk(0.f, 0.f);
        diag(kw, 0.f, t, w, 0.f);
        store(tp, w);
        if (EARLY) load_diag(F.K[0], kw);
        __syncthreads();
        hops(0, tp, t);
        if (!EARLY) load_diag(F.K[0], kw);
        diag(kw, m4, r, t, -0.25f);
        float v[4] = {0, 0, 0, 0};
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            v[0] += t[a].re * r[a].re + t[a].im * r[a].im;
            v[1] += t[a].re * r[a].im - t[a].im * r[a].re;
            v[2] += t[a].re * t[a].re + t[a].im * t[a].im;
            v[3] += r[a].re * r[a].re + r[a].im * r[a].im;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) red[q] = act ? (double)v[q] : 0.0;
        wg_sums<4>(red, red_lds[phase ^= 1]);
        ++it;
        slow = !(red[2] > 0);
        if (slow) break;
        const cx<float> omega = mk((float)(red[0] / red[2]), (float)(red[1] / red[2]));
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            cmadd(e[a], omega, r[a]);
            cmadd(r[a], mk(-omega.re, -omega.im), t[a]);
        }
        const double r2n = red[3] - (red[0] * red[0] + red[1] * red[1]) / red[2];
        slow = !isfinite(r2n) || (r2n > thr2 && it % BL_WINDOW == 0 && r2n > GAIN * GAIN * window);
        if (!(r2n > thr2) || slow) break;
        if (it % BL_WINDOW == 0) window = r2n;
        // (all reads of the operand were before the last barrier)
        store(op, r);
        __syncthreads();
    }
    if (act && !dg) {
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            const double2 x = xe[oh + (size_t)a * n2];
            xe[oh + (size_t)a * n2] = make_double2(x.x + rn * (double)e[a].re, x.y + rn * (double)e[a].im);
        }
    }
    if (threadIdx.x == 0) {
        iters[k.key] += (it + 1) / 2;
        iters[gridDim.x + k.key] = slow;
    }
}

static bool lds_fits(int hv, int lds_max_bytes) {
    return hv <= BL_MAX && (long long)2 * 6 * 16 * (hv + 1) + 2 * 8 * 16 * 8 <= lds_max_bytes;
}
bool blk_lds_fits(const Geom& g, int lds_max_bytes) { return g.eo && lds_fits(g.hvb, lds_max_bytes); }
bool eo_lds_fits(const Geom& g, int lds_max_bytes) { return g.eo && lds_fits(g.V / 2, lds_max_bytes); }

// Lanes per site.  More lanes issue more instructions for a site in all, and pay where they add no wavefronts (four
// lanes on at most 16 sites) or where SIMDs are free for them (two).  One colour, 8 RHS, to 1e-10, one / two / four
// lanes: 32x16^3, blocks of 8, 16, 32, 64 sites a parity 3.69 / 4.39 / 3.60, 2.24 / 2.59 / 2.16, 1.52 / 1.70 / 1.93,
// 1.33 / 1.82 / 2.01 ms; 8^4, blocks of 16, 32, 64, 128 sites 0.326 / 0.287 / 0.280, 0.322 / 0.282 / 0.278, 0.338 / 0.303 /
// 0.309, 0.389 / 0.345 / - ms.
static int lanes_per_site(int hv, long long groups, unsigned n2) {
    if (n2 >= 1u << 25) return 1;  // (the byte offsets over eight clover planes stay below 4 GiB)
    if (4 * hv <= 64) return 4;
    return 2 * hv <= BQ_THREADS && groups * ((hv + 63) / 64) <= 2 * CU_COUNT ? 2 : 1;
}
template <bool WRAP>
static void launch_lds(hipStream_t st, const Geom& g, const EoFields<float>& F, const float4* Ainv, const double2* re,
                       double2* xe, const double* bb, const double* rr, double mass4, double tol, double aim, double floor_eps,
                       int maxit, int* iters, int colour, int nrhs) {
    const int steps = maxit < (1 << 30) ? 2 * maxit : maxit;  // (a BiCGStab iteration, the unit of maxit, is two steps)
    const int lanes = lanes_per_site(g.hvb, (long long)g.NBc * nrhs, F.n2);
    const size_t lds = (size_t)2 * 6 * (g.hvb + 1) * sizeof(float4);  // (a record of zeros after each field)
    const int groups = g.NBc * nrhs, threads = (lanes * g.hvb + 63) / 64 * 64;
    if (lanes == 1) {
        k_blk_lds<WRAP, false><<<groups, threads, lds, st>>>(g, F, Ainv, re, xe, nullptr, nullptr, nullptr, bb, rr, mass4, tol,
                                                             aim, floor_eps, steps, iters, colour, nrhs);
        return;
    }
    auto k = k_lds_lanes<WRAP, 2>;
    if constexpr (!WRAP)  // (no lattice has that few sites)
        if (lanes == 4) k = k_lds_lanes<false, 4>;
    k<<<groups, threads, lds, st>>>(g, F, Ainv, re, xe, bb, rr, mass4, tol, aim, floor_eps, steps, iters, colour, nrhs);
}
void launch_blk_lds(Exec& e, const Geom& g, const EoFields<float>& F, const float4* Ainv, const double2* re,
                    double2* xe, const double* bb, const double* rr, double mass4, double tol, double aim,
                    int maxit, int* iters, int colour, int nrhs) {
    Timed t(e, 2, 0);
    launch_lds<false>(e.stream, g, F, Ainv, re, xe, bb, rr, mass4, tol, aim, MR_FLOOR32, maxit, iters, colour, nrhs);
}
void launch_blk_lds_bi(Exec& e, const Geom& g, const EoFields<float>& F, const float4* Ainv, const double2* re,
                       double2* xe, void* const w[7], const double* bb, const double* rr, double mass4, double tol,
                       int maxit, int* iters, int colour, int nrhs) {
    Timed t(e, 2, 0);
    const size_t lds = (size_t)2 * 6 * (g.hvb + 1) * sizeof(float4);
    k_blk_lds<false, true><<<g.NBc * nrhs, (g.hvb + 63) / 64 * 64, lds, e.stream>>>(
        g, F, Ainv, re, xe, (float4*)w[1], (float4*)w[2], (float4*)w[5], bb, rr, mass4, tol, BI_AIM, 2e-6, maxit, iters,
        colour, nrhs);
}
void launch_eo_lds(Exec& e, Geom g, const EoFields<float>& F, const float4* Ainv, const double2* re, double2* xe,
                   const double* bb, const double* rr, double mass4, double tol, double floor_eps, int maxit, int* iters,
                   int nrhs) {
    Timed t(e, DDWC_K_DSLASH32, 0);
    g.hvb = g.V / 2, g.NBc = 1;
    launch_lds<true>(e.stream, g, F, Ainv, re, xe, bb, rr, mass4, tol, mr_aim(tol, MR_AIM), floor_eps, maxit, iters, 0, nrhs);
}

// ------------------------------------------------------------------ FP64 passes through LDS
// The same two passes for block parities of at most BP_MAX sites, one site of either parity per thread, with the field
// that the hops gather from in LDS (FP64, records of BP_PITCH words): x_e, then A_oo^-1 H^k x_e in its place.
// Read from the caches, as by k_blk_prep and k_blk_resid, the gathers are half of what passes through a CU's load
// path, and the odd field comes back from memory, more blocks being in flight than the L2s hold.
// 48x24^3, 6^4 blocks, 12 RHS, one colour: residual 894 -> 666 us, preparation 760 -> 611 us; 32x16^3, 4^4 blocks, 8 RHS:
// 112 -> 88 and 107 -> 87 us.  A 6^4 block's workgroup is alone on its CU, so its loads and stores (0.3 ms at the rate
// of a copy) and its hops follow each other.
constexpr int BP_MAX = 768;    // 12 waves: 3 per SIMD at up to 168 VGPRs
constexpr int BP_PITCH = 13;   // 208 bytes: the eight lanes served together fall on distinct banks
struct PassSite {
    unsigned l, lg;    // LDS record (hv, the record of zeros, for a thread past the block); site in the block
    bool act;
};
__device__ __forceinline__ PassSite pass_site(unsigned hv) {
    PassSite p;
    p.act = threadIdx.x < hv;
    p.l = p.act ? threadIdx.x : hv;
    p.lg = p.act ? threadIdx.x : 0u;
    return p;
}
__device__ __forceinline__ void pass_store(double2* L, unsigned l, const cx<double> q[12]) {
#pragma unroll
    for (int c = 0; c < 12; ++c) L[l * BP_PITCH + c] = make_double2(q[c].re, q[c].im);
}
// in-block hops of the half site h0 + st.lg of parity P (as lds_hops; the next link is in flight during a hop)
template <int P>
__device__ __forceinline__ void pass_hops(const EoFields<double>& F, unsigned h0, unsigned hv, const PassSite& st, const double2* L,
                                          cx<double> acc[12]) {
    const unsigned n2 = F.n2;
    const BlkNbr<false> nb = blk_nbr<false>(F.nbr[P], n2, h0 + st.lg, h0, hv, st.act);
    Planes pf(fresh(F.U[P]), n2), pb(fresh(F.U[1 - P]), n2);
    const unsigned own = byte_offset(h0 + st.lg, 16);
    auto lu = [&](int d, cx<double> u[9]) {
        if (d & 1) {
            const unsigned t = nb[d];
            uload_link(pb, reissue(byte_offset(h0 + (t < hv ? t : st.lg), 16)), u);
        } else {
            uload_link(pf, reissue(own), u);
        }
    };
    cx<double> u[9], un[9], h[6];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = mk(0.0, 0.0);
    lu(0, u);
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        if (d + 1 < 8) lu(d + 1, un);
        __builtin_amdgcn_sched_barrier(0);
        {
            const double2* r = L + reissue(nb[d]) * BP_PITCH;
            cx<double> q[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) q[c] = mk(r[c].x, r[c].y);
            proj_dispatch<double>(d, q, h);
        }
        pin6(h);
        apply_dispatch<double>(d, u, h, acc);
        pin(acc);
#pragma unroll
        for (int k = 0; k < 9; ++k) u[k] = un[k];
    }
}
// y = (m4 + C) p + hsc y, the words of one chiral block in registers at a time
__device__ __forceinline__ void pass_diag(const double2* K, unsigned n2, unsigned off, double m4, const cx<double> p[12],
                                          cx<double> y[12], double hsc) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        double d[6], o[30];
        Planes qd(fresh(K), n2, 3 * blk), qo(fresh(K), n2, 6 + 15 * blk);
        const unsigned of = reissue(off);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const d2v v = qd.load<d2v>(of);
            d[2 * k] = v.x, d[2 * k + 1] = v.y;
        }
#pragma unroll
        for (int k = 0; k < 15; ++k) {
            const d2v v = qo.load<d2v>(of);
            o[2 * k] = v.x, o[2 * k + 1] = v.y;
        }
        diag_block<double>(d, o, m4, p + 6 * blk, y + 6 * blk, hsc);
        pin6(y + 6 * blk);
    }
}

__global__ __launch_bounds__(BP_MAX) void k_blk_prep_lds(Geom g, EoFields<double> F, const double2* Ainv, const double2* b,
                                                        double2* bpe, double2* re, double2* xe, double2* to, double* bb,
                                                        double* rr, int colour, int nrhs) {
    extern __shared__ double2 bp_lds[];
    __shared__ double lds[2 * 16];
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const unsigned n2 = F.n2, hv = (unsigned)g.hvb;
    const PassSite st = pass_site(hv);
    const size_t oh = (size_t)k.rhs * 12 * n2;
    b += (size_t)k.rhs * 12 * g.V;
    const unsigned h = k.h0 + st.lg, off = byte_offset(h, 16);
    if (threadIdx.x < 12) bp_lds[hv * BP_PITCH + threadIdx.x] = make_double2(0.0, 0.0);
    double red[2];
    {
        cx<double> v[12], w[12];
        uload_spinor(b, g.V, byte_offset(full_index(g, h, 1), 16), v);
        red[0] = st.act ? acc_nrm(v) : 0.0;
#pragma unroll
        for (int c = 0; c < 12; ++c) w[c] = mk(0.0, 0.0);
        pass_diag(Ainv, n2, off, 0.0, v, w, 0.0);
        if (st.act) {
            ustore_spinor(fresh(to + oh), n2, off, w);
            pass_store(bp_lds, st.l, w);
        }
    }
    __syncthreads();
    cx<double> v[12], y[12];
    pass_hops<0>(F, k.h0, hv, st, bp_lds, y);
    uload_spinor(fresh(b), g.V, byte_offset(full_index(g, h, 0), 16), v);
    red[0] += st.act ? acc_nrm(v) : 0.0;
#pragma unroll
    for (int c = 0; c < 12; ++c) y[c] = v[c] + 0.5 * y[c];
    red[1] = st.act ? acc_nrm(y) : 0.0;
    if (st.act) {
        ustore_spinor(fresh(bpe + oh), n2, off, y);
        ustore_spinor(fresh(re + oh), n2, off, y);
#pragma unroll
        for (int c = 0; c < 12; ++c) y[c] = mk(0.0, 0.0);
        ustore_spinor(fresh(xe + oh), n2, off, y);
    }
    block_sum<2>(red, lds);
    if (threadIdx.x == 0) {
        bb[k.key] = red[0];
        rr[k.key] = red[1];
    }
}

__global__ __launch_bounds__(BP_MAX) void k_blk_resid_lds(Geom g, EoFields<double> F, const double2* Ainv, const double2* bpe,
                                                         const double2* xe, double2* re, double2* to, double* rr,
                                                         double mass4, int colour, int nrhs) {
    extern __shared__ double2 bp_lds[];
    __shared__ double lds[16];
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const unsigned n2 = F.n2, hv = (unsigned)g.hvb;
    const PassSite st = pass_site(hv);
    const size_t oh = (size_t)k.rhs * 12 * n2;
    const unsigned off = byte_offset(k.h0 + st.lg, 16);
    if (threadIdx.x < 12) bp_lds[hv * BP_PITCH + threadIdx.x] = make_double2(0.0, 0.0);
    cx<double> v[12], w[12];
    uload_spinor(xe + oh, n2, off, v);
    if (st.act) pass_store(bp_lds, st.l, v);
    __syncthreads();
    // t_o = A_oo^-1 H^k x_e
    pass_hops<1>(F, k.h0, hv, st, bp_lds, v);
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = mk(0.0, 0.0);
    pass_diag(Ainv, n2, off, 0.0, v, w, 0.0);
    __syncthreads();
    if (st.act) {
        ustore_spinor(fresh(to + oh), n2, off, w);
        pass_store(bp_lds, st.l, w);
    }
    __syncthreads();
    // r_e = b'_e - (A_ee x_e - 1/4 H^k t_o)
    pass_hops<0>(F, k.h0, hv, st, bp_lds, w);
    uload_spinor(fresh(xe + oh), n2, reissue(off), v);
    pass_diag(F.K[0], n2, off, mass4, v, w, -0.25);
    uload_spinor(fresh(bpe + oh), n2, reissue(off), v);
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = v[c] - w[c];
    if (st.act) ustore_spinor(fresh(re + oh), n2, off, w);
    double red[1] = {st.act ? acc_nrm(w) : 0.0};
    block_sum<1>(red, lds);
    if (threadIdx.x == 0) rr[k.key] = red[0];
}

// ------------------------------------------------------------------ minimal residual in global memory
// The same iteration for blocks that do not fit k_blk_lds (8^4: 2048 sites of a parity) and for FP16
// storage: one workgroup per (block, RHS), a few sites per thread.  The odd intermediate, t = M_k r and the
// correction e are slabs; r is in LDS where it fits (8^4 in FP16: 107 KB), else a slab too.
//
// An in-block neighbour is the site's own half index shifted by half the stride of its direction
// (along x3: by 0 or 1, by the parity of l3), so the hops of a site are one 16-bit mask: bit d set where
// hop d stays in the block, bit 8 the parity of l3.  The masks of all blocks are the same and lie in LDS.
//
// What bounds it: vector-memory instructions.  BiCGStab on entry-major links issued about 286 a site and operator
// application in FP16 (nine 4-byte loads a link, eight table entries, eleven vector accesses), this 140.  Per launch:
// 8^4 in FP16, 64x32^3, 6 RHS, one colour 8110 -> 5554 us; in FP32, 32x16^3, 8 RHS 2640 -> 2060 us.
constexpr int BM_MAX = 1024;

// LDS records of a stored spinor: FP32 as k_blk_lds, FP16 three words per site and after them the scales.
__device__ __forceinline__ void rec_load(float4* L, unsigned, unsigned l, cx<float> q[12], float) { lds_load(L, l, q); }
__device__ __forceinline__ void rec_store(float4* L, unsigned, unsigned l, const cx<float> q[12], float) { lds_store(L, l, q); }
__device__ __forceinline__ void rec_load(float4* L, unsigned HV, unsigned l, cx<float> q[12], H16) {
    const h8v* p = (const h8v*)L + l * 3;
    const float sc = ((const float*)(L + HV * 3))[l];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const h8v w = p[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) q[4 * k + i] = mk(sc * (float)w[2 * i], sc * (float)w[2 * i + 1]);
    }
}
__device__ __forceinline__ void rec_store(float4* L, unsigned HV, unsigned l, const cx<float> q[12], H16) {
    h8v w[3];
    ((float*)(L + HV * 3))[l] = to_half(q, w);
#pragma unroll
    for (int k = 0; k < 3; ++k) ((h8v*)L)[l * 3 + k] = w[k];
}

template <class S, bool RLDS>
__global__ __launch_bounds__(BM_MAX) void k_blk_mr(Geom g, EoFields<S> F, const float4* Ainv, const double2* re,
                                                   double2* xe, typename Traits<S>::word* rg,
                                                   typename Traits<S>::word* tg, typename Traits<S>::word* wg, float4* eg,
                                                   const double* __restrict__ bb, const double* __restrict__ rr,
                                                   double mass4, double tol, double aim, double inner_floor, int maxit, int* iters,
                                                   int colour, int nrhs) {
    extern __shared__ float4 bm_lds[];
    __shared__ double red_lds[2][8 * 16];
    constexpr double GAIN = std::is_same<S, H16>::value ? BL_GAIN : BM_GAIN32;
    typedef typename std::conditional<std::is_same<S, H16>::value, f16, float>::type L;
    const S tag{};
    const BlkIdx k = blk_idx(g, colour, nrhs);
    const double b2 = bb[k.key], r2 = rr[k.key];
    if (!(b2 > 0) || !(r2 > tol * tol * b2) || !isfinite(r2)) return;  // uniform over the workgroup
    const unsigned n2 = F.n2, HV = (unsigned)g.hvb, h0 = k.h0;
    unsigned short* mask = (unsigned short*)bm_lds;  // [2][HV]
    float4* rl = bm_lds + (2 * HV * sizeof(unsigned short) + 15) / 16;
    for (unsigned q = threadIdx.x; q < 2 * HV; q += blockDim.x) {
        // coordinates inside the block of the q-th site (parity-major)
        const Site st = decode(g, (int)q);
        unsigned m = (unsigned)(st.l[3] & 1) << 8;
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
            m |= (unsigned)(st.l[mu] < g.b[mu] - 1) << (2 * mu) | (unsigned)(st.l[mu] > 0) << (2 * mu + 1);
        mask[q] = (unsigned short)m;
    }
    for (unsigned q = threadIdx.x; q < 2 * 8 * 16; q += blockDim.x) red_lds[0][q] = 0;
    const size_t oh = (size_t)k.rhs * 12 * n2, oR = (size_t)k.rhs * slab_words<S>(n2), oX = (size_t)k.rhs * 6 * n2;
    re += oh;
    xe += oh;
    rg += oR;
    tg += oR;
    wg += oR;
    eg += oX;
    const unsigned sh[3] = {(unsigned)g.lstr[0] / 2, (unsigned)g.lstr[1] / 2, (unsigned)g.lstr[2] / 2};
    // local half index of the neighbour in direction d of the site (l, mask m); itself for a hop that leaves
    auto target = [&](unsigned l, unsigned m, int d) {
        const unsigned up = (m >> 8) & 1;
        const unsigned t = d < 6 ? ((d & 1) ? l - sh[d >> 1] : l + sh[d >> 1]) : d == 6 ? l + up : l - 1 + up;
        return (m >> d) & 1 ? t : l;
    };
    auto none = [](int) { return false; };
    // acc = in-block hops of the site l of parity p from the field that lq reads by local half index
    auto hops = [&](int p, unsigned l, auto&& lq, cx<float> acc[12]) {
        const unsigned m = mask[p * HV + l];
        PackedLinks<L> pf(fresh(F.W[p]), n2), pb(fresh(F.W[1 - p]), n2);
        hops_pipelined<float, false>(
            acc, [&](int d, cx<float> q[12]) { lq(reissue(target(l, m, d)), q); },
            [&](int d, cx<float> u[9]) {
                if (d & 1)
                    pb.next(byte_offset(h0 + reissue(target(l, m, d)), 16), u);
                else
                    pf.next(byte_offset(h0 + reissue(l), 16), u);
            },
            none, [&](int d) { return ((m >> d) & 1) != 0; });
    };
    auto load_r = [&](unsigned l, cx<float> q[12]) {
        if constexpr (RLDS)
            rec_load(rl, HV, l, q, tag);
        else
            uload_spinor(fresh(rg), n2, byte_offset(h0 + l, 16), q);
    };
    auto store_r = [&](unsigned l, const cx<float> q[12]) {
        if constexpr (RLDS)
            rec_store(rl, HV, l, q, tag);
        else
            ustore_spinor(fresh(rg), n2, byte_offset(h0 + l, 16), q);
    };
    const float m4 = (float)mass4;
    const double rn = sqrt(r2), sc = 1.0 / rn;
    double eps = aim * tol * sqrt(b2) / rn;
    if (eps < inner_floor) eps = inner_floor;
    const int nl = (int)((HV + blockDim.x - 1) / blockDim.x);  // sites per thread
    int phase = 0;
    double red[4] = {0, 0, 0, 0};
#pragma unroll 1
    for (int j = 0; j < nl; ++j) {
        const unsigned li = j * blockDim.x + threadIdx.x, l = li < HV ? li : 0u;
        const unsigned lo = byte_offset(h0 + l, 16);
        cx<double> a[12];
        uload_spinor(fresh(re), n2, lo, a);
        cx<float> r[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) r[c] = mk((float)(sc * a[c].re), (float)(sc * a[c].im));
        if (li < HV) {
            const cx<float> z[12] = {};
            store_r(l, r);
            ustore_spinor(fresh(eg), n2, lo, z);
            red[0] += acc_nrm(r);
        }
    }
    __syncthreads();
    wg_sums<1>(red, red_lds[phase ^= 1]);
    const double thr2 = eps * eps * red[0];
    double window = red[0];
    int it = 0;
    bool slow = false;
    while (it < maxit) {
        // w = A_oo^-1 H^k_oe r
#pragma unroll 1
        for (int j = 0; j < nl; ++j) {
            const unsigned li = j * blockDim.x + threadIdx.x, l = li < HV ? li : 0u;
            cx<float> acc[12], y[12];
            hops(1, l, load_r, acc);
            const unsigned lo = byte_offset(h0 + l, 16);
            UDiag<float> K(fresh(Ainv), n2, lo);
            K.first();
#pragma unroll
            for (int c = 0; c < 12; ++c) y[c] = mk(0.f, 0.f);
            K.apply(0.f, acc, y, 0.f);
            if (li < HV) ustore_spinor(fresh(wg), n2, lo, y);
        }
        __syncthreads();
        // t = (4 + m + C) r - 1/4 H^k_eo w, (t, r), (t, t), (r, r)
        red[0] = red[1] = red[2] = red[3] = 0;
#pragma unroll 1
        for (int j = 0; j < nl; ++j) {
            const unsigned li = j * blockDim.x + threadIdx.x, l = li < HV ? li : 0u;
            cx<float> t[12], r[12];
            hops(0, l, [&](unsigned q, cx<float> v[12]) { uload_spinor(fresh(wg), n2, byte_offset(h0 + q, 16), v); }, t);
            const unsigned lo = byte_offset(h0 + l, 16);
            UDiag<float> K(fresh(F.K[0]), n2, lo);
            K.first();
            load_r(l, r);
            K.apply(m4, r, t, -0.25f);
            if (li < HV) {
                ustore_spinor(fresh(tg), n2, lo, t);
                acc_dot(t, r, red[0], red[1]);
                red[2] += acc_nrm(t);
                red[3] += acc_nrm(r);
            }
        }
        wg_sums<4>(red, red_lds[phase ^= 1]);
        ++it;
        slow = !(red[2] > 0);
        if (slow) break;
        const cx<float> omega = mk((float)(red[0] / red[2]), (float)(red[1] / red[2]));
        const double r2n = red[3] - (red[0] * red[0] + red[1] * red[1]) / red[2];
        // e += omega r, r -= omega t
#pragma unroll 1
        for (int j = 0; j < nl; ++j) {
            const unsigned li = j * blockDim.x + threadIdx.x, l = li < HV ? li : 0u;
            const unsigned lo = byte_offset(h0 + l, 16);
            cx<float> e[12], r[12], t[12];
            uload_spinor(fresh(eg), n2, lo, e);
            uload_spinor(fresh(tg), n2, lo, t);
            load_r(l, r);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                cmadd(e[c], omega, r[c]);
                cmadd(r[c], mk(-omega.re, -omega.im), t[c]);
            }
            if (li < HV) {
                ustore_spinor(fresh(eg), n2, lo, e);
                store_r(l, r);
            }
        }
        slow = !isfinite(r2n) || (r2n > thr2 && it % BL_WINDOW == 0 && r2n > GAIN * GAIN * window);
        if (!(r2n > thr2) || slow) break;
        if (it % BL_WINDOW == 0) window = r2n;
        __syncthreads();
    }
    // x_e += ||r_e|| e in FP64
#pragma unroll 1
    for (int j = 0; j < nl; ++j) {
        const unsigned li = j * blockDim.x + threadIdx.x, l = li < HV ? li : 0u;
        const unsigned lo = byte_offset(h0 + l, 16);
        cx<float> e[12];
        cx<double> x[12];
        uload_spinor(fresh(eg), n2, lo, e);
        uload_spinor(fresh(xe), n2, lo, x);
#pragma unroll
        for (int c = 0; c < 12; ++c) x[c] = x[c] + mk(rn * (double)e[c].re, rn * (double)e[c].im);
        if (li < HV) ustore_spinor(fresh(xe), n2, lo, x);
    }
    if (threadIdx.x == 0) {
        iters[k.key] += (it + 1) / 2;
        iters[gridDim.x + k.key] = slow;
    }
}

static size_t mr_mask_bytes(const Geom& g) { return ((size_t)2 * g.hvb * sizeof(unsigned short) + 15) / 16 * 16; }
// (at most 40448 sites of a parity with 160 KB: larger blocks run k_blk_inner, which uses no LDS for a block's sites)
bool blk_mr_fits(const Geom& g, int lds_max) { return g.eo && mr_mask_bytes(g) + 2 * 8 * 16 * 8 <= (size_t)lds_max; }
template <class S>
void launch_blk_mr(Exec& e, const Geom& g, const EoFields<S>& F, const float4* Ainv, const double2* re, double2* xe,
                   void* const w[7], const double* bb, const double* rr, double mass4, double tol, double aim, int maxit,
                   int* iters, int colour, int nrhs, int lds_max) {
    Timed t(e, 2, 0);
    typedef typename Traits<S>::word W;
    const int threads = block_threads_for(g, e.blk_threads, BM_MAX);
    const size_t masks = mr_mask_bytes(g);
    const size_t recs = (size_t)g.hvb * (std::is_same<S, H16>::value ? 52 : 96);
    const bool rlds = masks + recs + 2 * 8 * 16 * 8 <= (size_t)lds_max;
    const size_t lds = std::max(rlds ? masks + recs : masks, std::min((size_t)e.blk_lds << 10, (size_t)lds_max - 2 * 8 * 16 * 8));
    const double floor_eps = std::is_same<S, H16>::value ? 1e-3 : MR_FLOOR32;
    const int steps = maxit < (1 << 30) ? 2 * maxit : maxit;
    if (rlds)
        k_blk_mr<S, true><<<g.NBc * nrhs, threads, lds, e.stream>>>(g, F, Ainv, re, xe, (W*)w[0], (W*)w[4], (W*)w[6],
                                                                    (float4*)w[5], bb, rr, mass4, tol, aim, floor_eps, steps,
                                                                    iters, colour, nrhs);
    else
        k_blk_mr<S, false><<<g.NBc * nrhs, threads, lds, e.stream>>>(g, F, Ainv, re, xe, (W*)w[0], (W*)w[4], (W*)w[6],
                                                                     (float4*)w[5], bb, rr, mass4, tol, aim, floor_eps, steps,
                                                                     iters, colour, nrhs);
}
template void launch_blk_mr<float>(Exec&, const Geom&, const EoFields<float>&, const float4*, const double2*, double2*,
                                   void* const[7], const double*, const double*, double, double, double, int, int*, int,
                                   int, int);
template void launch_blk_mr<H16>(Exec&, const Geom&, const EoFields<H16>&, const float4*, const double2*, double2*,
                                 void* const[7], const double*, const double*, double, double, double, int, int*, int,
                                 int, int);

// LDS bytes of the FP64 passes through LDS, 0 for blocks that do not fit
static size_t pass_lds(const Geom& g, int lds_max) {
    const size_t b = (size_t)BP_PITCH * 16 * (g.hvb + 1);
    return g.hvb <= BP_MAX && b + 2 * 16 * 8 <= (size_t)lds_max ? b : 0;
}
void launch_blk_prep(Exec& e, const Geom& g, const EoFields<double>& F, const double2* Ainv, const double2* b,
                     double2* bpe, double2* re, double2* xe, double2* to, double* bb, double* rr, int colour, int nrhs,
                     int lds_max) {
    Timed t(e, 4, 0);  // FP64 defect-correction passes: "other"
    if (const size_t lds = pass_lds(g, lds_max)) {
        k_blk_prep_lds<<<g.NBc * nrhs, (g.hvb + 63) / 64 * 64, lds, e.stream>>>(g, F, Ainv, b, bpe, re, xe, to, bb, rr, colour,
                                                                               nrhs);
        return;
    }
    k_blk_prep<<<g.NBc * nrhs, block_eo_threads(g, e.blk_threads), 0, e.stream>>>(g, F, Ainv, b, bpe, re, xe, to, bb, rr, colour, nrhs);
}
void launch_blk_resid(Exec& e, const Geom& g, const EoFields<double>& F, const double2* Ainv, const double2* bpe,
                      const double2* xe, double2* re, double2* to, double* rr, double mass4, int colour, int nrhs,
                      int lds_max) {
    Timed t(e, 4, 0);  // FP64 defect-correction passes: "other"
    if (const size_t lds = pass_lds(g, lds_max)) {
        k_blk_resid_lds<<<g.NBc * nrhs, (g.hvb + 63) / 64 * 64, lds, e.stream>>>(g, F, Ainv, bpe, xe, re, to, rr, mass4, colour,
                                                                                nrhs);
        return;
    }
    k_blk_resid<<<g.NBc * nrhs, block_eo_threads(g, e.blk_threads), 0, e.stream>>>(g, F, Ainv, bpe, xe, re, to, rr, mass4, colour,
                                                                    nrhs);
}
void launch_blk_recon(Exec& e, const Geom& g, const double2* to, const double2* th, const double2* xe, double2* x,
                      int colour, int nrhs) {
    Timed t(e, 4, 0);  // FP64 defect-correction passes: "other"
    k_blk_recon<<<g.NBc * nrhs, block_eo_threads(g, e.blk_threads), 0, e.stream>>>(g, to, th, xe, x, colour, nrhs);
}
template <class S>
void launch_blk_inner(Exec& e, const Geom& g, const EoFields<S>& F, const typename Traits<S>::kword* Ainv,
                      const double2* re, double2* xe, void* const w[7], const double* bb, const double* rr,
                      double mass4, double tol, int maxit, int* iters, int colour, int nrhs) {
    Timed t(e, 2, 0);
    BlkInner<S> bw;
    typedef typename Traits<S>::word W;
    bw.r = (W*)w[0];
    bw.rh = (W*)w[1];
    bw.p = (W*)w[2];
    bw.v = (W*)w[3];
    bw.t = (W*)w[4];
    bw.e = (typename BlkInner<S>::XW*)w[5];
    bw.tmp = (W*)w[6];
    // the inner solve stops at this relative residual at the least (the storage's reach)
    const double floor_eps = std::is_same<S, double>::value ? 0.0 : std::is_same<S, H16>::value ? 1e-3 : 2e-6;
    // e.blk_lds KiB of dynamic LDS (unused by the kernel) caps the workgroups resident per CU, and so
    // the slabs in flight, which then stay in the last-level cache
    k_blk_inner<S><<<g.NBc * nrhs, block_threads_for(g, e.blk_threads, be_inner_max<S>()), (size_t)e.blk_lds << 10,
                     e.stream>>>(g, F, Ainv, re, xe, bw, bb, rr, mass4, tol,
                                                                       floor_eps, maxit, iters, colour, nrhs);
}
size_t blk_slab_bytes(int prec, unsigned n2) {
    if (prec == DDWC_FP64) return slab_words<double>(n2) * 16;
    if (prec == DDWC_MIXED16) return slab_words<H16>(n2) * 16;
    return slab_words<float>(n2) * 16;
}
template void launch_blk_inner<double>(Exec&, const Geom&, const EoFields<double>&, const double2*, const double2*,
                                       double2*, void* const[7], const double*, const double*, double, double, int,
                                       int*, int, int);
template void launch_blk_inner<float>(Exec&, const Geom&, const EoFields<float>&, const float4*, const double2*,
                                      double2*, void* const[7], const double*, const double*, double, double, int,
                                      int*, int, int);
template void launch_blk_inner<H16>(Exec&, const Geom&, const EoFields<H16>&, const float4*, const double2*,
                                    double2*, void* const[7], const double*, const double*, double, double, int,
                                    int*, int, int);

}  // namespace ddwc
