// Derivatives of the exponents with respect to the links: the force kernels.
//
// Every link derivative of the estimator reduces to terms Re <a, (dD/dU) b> for pairs of
// full-lattice FP64 fields (a, b) with one weight per RHS.  The gradient is returned in the
// convention G = dL/dRe U + i dL/dIm U for each 3x3 link matrix U (no unitarity
// constraint); for a term Re tr[U Z] it is Z^+.
//
// Hops (D = (4 + m) + C - H/2):  the link U = U_mu(x) enters
//     a(x)^+ (1 - g_mu) U b(x + mu) + a(x + mu)^+ (1 + g_mu) U^+ b(x),
// times the time-boundary sign, so that G += -1/2 s [sum_alpha a_alpha(x) ((1 - g_mu) b(x + mu))_alpha^+
//                                                 + b_alpha(x) ((1 + g_mu) a(x + mu))_alpha^+]
// (colour outer products, spin summed).
//
// Clover (chiral blocks C_k = (i c_sw / 2) sum_l s_l x E_l^k, E from the field strengths as in
// clover_build.h):  Re <a, C b> = sum_x sum_{mu<nu} Re tr[Fhat_mu nu K_mu nu] with
// K = (i c_sw / 2) (signed sums of L_l^k), (L_l^k)_{ba} = sum_{alpha beta in block k} (s_l)_{alpha beta}
// b_{beta b} conj(a_{alpha a}); with Fhat = (Q - Q^+)/8 this is Re tr[Q J], J = (K - K^+)/8.  The four leaves at a
// plaquette's corners are its cyclic shifts, each with its corner's J (plaquette_force in force.h).
#include "ddwc_internal.h"
#include "force.h"

namespace ddwc {

// in-place gamma_5 = diag(1, 1, -1, -1) on the spin index (chiral basis)
__global__ void k_gamma5(Geom g, double2* __restrict__ v, int nrhs) {
    const unsigned s = blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (s >= (unsigned)g.V) return;
    double2* f = v + (size_t)r * 12 * g.V;
#pragma unroll
    for (int c = 6; c < 12; ++c) {
        double2 w = f[(size_t)c * g.V + s];
        f[(size_t)c * g.V + s] = make_double2(-w.x, -w.y);
    }
}

void launch_gamma5(Exec& e, const Geom& g, double2* v, int nrhs) {
    Timed t(e, 4, 0);
    k_gamma5<<<dim3(tiles_of(g.V), nrhs), WG, 0, e.stream>>>(g, v, nrhs);
}

// G_mu(x) += hop part, one thread per (x, mu); the four wavefronts of a workgroup are the four directions of the same
// 64 sites, so that these share the loads of a(x) and b(x) in the CU's cache.  Bound by its gathers: 32x16^3, 8 RHS, 1410 us
// with 256-site workgroups of one direction, whole spinors and the registers of a 1024-thread workgroup (836 bytes of
// scratch a thread), 379 us with half spinors, this grouping and no scratch (0.4 GB compulsory: 80 us).
__global__ __launch_bounds__(256) void k_force_hop(Geom g, const int* __restrict__ nbr, const double2* __restrict__ a,
                                                   const double2* __restrict__ b, const double* __restrict__ w,
                                                   int nrhs, cx<double>* __restrict__ G) {
    const unsigned s = blockIdx.x * 64 + (threadIdx.x & 63);
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (s >= (unsigned)g.V) return;
    force_hop_site(g, nbr, a, b, w, nrhs, G, s, mu);
}

void launch_force_hop(Exec& e, const Geom& g, const int* nbr, const double2* a, const double2* b, const double* w,
                      int nrhs, cx<double>* G) {
    Timed t(e, 4, 0);
    k_force_hop<<<(g.V + 63) / 64, 256, 0, e.stream>>>(g, nbr, a, b, w, nrhs, G);
}

// Clover part in three kernels.  The leaves' sums are linear in the outer products of (a, b) at their corner, so these
// are accumulated first, over every pair of fields that a gradient has (Lacc [6][9][V]: chiral block k, Pauli index l at
// slot 3 k + l), and the links are gathered once at the end without atomics.  32x16^3, 8 RHS: 110 us a pair (0.4 GB of
// fields, 0.23 GB of sums) and 0.69 ms at the end, against 3.67 ms a pair when every pair scattered its 96 products
// a site into the links with atomics.
// One thread per (site, chiral block).
__global__ __launch_bounds__(128) void k_force_outer(Geom g, const double2* __restrict__ a, const double2* __restrict__ b,
                                                     const double* __restrict__ w, int nrhs, cx<double>* __restrict__ Lacc) {
    const unsigned y = blockIdx.x * blockDim.x + threadIdx.x;
    if (y >= (unsigned)g.V) return;
    const int k = blockIdx.y;
    M3 L[3];
    force_outer(a, b, w, nrhs, (unsigned)g.V, y, k, L);
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            cx<double>& o = Lacc[((size_t)(3 * k + l) * 9 + q) * g.V + y];
            o = o + L[l].a[q];
        }
}
// Lacc -> J of the six planes, in place (slot of force_slot); one thread per (site, Pauli index).
__global__ __launch_bounds__(128) void k_force_planes(Geom g, double csw, cx<double>* __restrict__ Lacc) {
    const unsigned y = blockIdx.x * blockDim.x + threadIdx.x;
    if (y >= (unsigned)g.V) return;
    const int l = blockIdx.y;
    M3 Ja, Jb;
    force_planes(ld(Lacc, g, l, (int)y), ld(Lacc, g, 3 + l, (int)y), l, csw, Ja, Jb);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        Lacc[((size_t)l * 9 + q) * g.V + y] = Ja.a[q];
        Lacc[((size_t)(3 + l) * 9 + q) * g.V + y] = Jb.a[q];
    }
}
// G_mu(x) += clover part, one thread per (x, mu).
__global__ __launch_bounds__(64) void k_force_clover(Geom g, const int* __restrict__ nbr, const cx<double>* __restrict__ U,
                                                     const cx<double>* __restrict__ J, cx<double>* __restrict__ G) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x, mu = blockIdx.y;
    if (x >= g.V) return;
    const M3 Z = force_clover_link(
        mu, x,
        [&](int d, int s) {
            const int e = nbr[(size_t)d * g.V + s];
            return e < 0 ? ~e : e;
        },
        [&](int m, int s) { return ld(U, g, m, s); }, [&](int slot, int s) { return ld(J, g, slot, s); });
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        cx<double>& o = G[((size_t)mu * 9 + k) * g.V + x];
        o = o + Z.a[k];
    }
}

void launch_force_outer(Exec& e, const Geom& g, const double2* a, const double2* b, const double* w, int nrhs,
                        cx<double>* Lacc) {
    Timed t(e, 4, 0);
    k_force_outer<<<dim3((g.V + 127) / 128, 2), 128, 0, e.stream>>>(g, a, b, w, nrhs, Lacc);
}
void launch_force_clover(Exec& e, const Geom& g, const int* nbr, const cx<double>* U, double csw, cx<double>* Lacc,
                         cx<double>* G) {
    Timed t(e, 4, 0);
    k_force_planes<<<dim3((g.V + 127) / 128, 3), 128, 0, e.stream>>>(g, csw, Lacc);
    k_force_clover<<<dim3((g.V + 63) / 64, 4), 64, 0, e.stream>>>(g, nbr, U, Lacc, G);
}

// internal [4][9][V] -> canonical [4][V][3][3]
__global__ void k_links_export(Geom g, const cx<double>* __restrict__ G, double2* __restrict__ can) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const int mu = blockIdx.y;
    if (s >= g.V) return;
    const Site S = decode(g, s);
    double2* dst = can + ((size_t)mu * g.V + canonical_index(g, S)) * 9;
    for (int k = 0; k < 9; ++k) {
        const cx<double> v = G[((size_t)mu * 9 + k) * g.V + s];
        dst[k] = make_double2(v.re, v.im);
    }
}

void launch_links_export(Exec& e, const Geom& g, const cx<double>* G, void* canon) {
    Timed t(e, 4, 0);
    k_links_export<<<dim3(tiles_of(g.V), 4), WG, 0, e.stream>>>(g, G, (double2*)canon);
}

}  // namespace ddwc
