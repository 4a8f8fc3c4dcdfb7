// Per-site logic of the link-derivative (force) kernels, shared with host-side checks.
// The formulas are stated in grad.hip.
#pragma once
#include "clover_build.h"

namespace ddwc {

DDWC_HD void ld12(const double2* f, unsigned V, unsigned s, cx<double> p[12]) {
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        const double2 w = f[(size_t)c * V + s];
        p[c] = mk(w.x, w.y);
    }
}

// Hop part of the gradient of sum_r w_r Re <a_r, D b_r> at link (x = s, MU), added to G.  The projectors satisfy
// (1 -+ g)^2 = 2 (1 -+ g) and the lower components of a projected spinor repeat the upper ones up to a phase, so
// the four-spin outer products are outer products of the two half spinors (half_proj).
template <int MU>
DDWC_HD void force_hop_site_t(const Geom& g, const int* nbr, const double2* a, const double2* b, const double* w,
                              int nrhs, cx<double>* G, unsigned s) {
    const int e = nbr[(size_t)(2 * MU) * g.V + s];
    const unsigned t = e < 0 ? (unsigned)~e : (unsigned)e;
    const double sg = e < 0 ? -1.0 : 1.0;
    cx<double> acc[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] = mk(0.0, 0.0);
    // acc += f h_left h_right^+, summed over the two half spins
    auto outer = [&](double f, const cx<double> hl[6], const cx<double> hr[6]) {
#pragma unroll
        for (int al = 0; al < 2; ++al)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const cx<double> x = f * hl[3 * al + i];
#pragma unroll
                for (int j = 0; j < 3; ++j) cjmadd(acc[3 * i + j], hr[3 * al + j], x);
            }
    };
    for (int r = 0; r < nrhs; ++r) {
        const double wr = w[r];
        if (wr == 0.0) continue;
        const double2* ar = a + (size_t)r * 12 * g.V;
        const double2* br = b + (size_t)r * 12 * g.V;
        cx<double> q[12], hl[6], hr[6];
        ld12(ar, g.V, s, q);
        half_proj<double, MU, +1>(q, hl);
        ld12(br, g.V, t, q);
        half_proj<double, MU, +1>(q, hr);  // a(x) ((1 - g_mu) b(x + mu))^+
        outer(-0.5 * sg * wr, hl, hr);
        ld12(br, g.V, s, q);
        half_proj<double, MU, -1>(q, hl);
        ld12(ar, g.V, t, q);
        half_proj<double, MU, -1>(q, hr);  // b(x) ((1 + g_mu) a(x + mu))^+
        outer(-0.5 * sg * wr, hl, hr);
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        cx<double>& o = G[((size_t)MU * 9 + k) * g.V + s];
        o = o + acc[k];
    }
}

DDWC_HD void force_hop_site(const Geom& g, const int* nbr, const double2* a, const double2* b, const double* w,
                            int nrhs, cx<double>* G, unsigned s, int mu) {
    switch (mu) {
        case 0: force_hop_site_t<0>(g, nbr, a, b, w, nrhs, G, s); break;
        case 1: force_hop_site_t<1>(g, nbr, a, b, w, nrhs, G, s); break;
        case 2: force_hop_site_t<2>(g, nbr, a, b, w, nrhs, G, s); break;
        default: force_hop_site_t<3>(g, nbr, a, b, w, nrhs, G, s); break;
    }
}

// Clover part.  Its ingredients at one site: L[l], the colour matrices of Pauli index l + 1 and chiral block k,
// (L_l)_{ba} = sum_{alpha beta} (s_l)_{alpha beta} b_{beta b} conj(a_{alpha a}), summed over the RHS with their weights.
DDWC_HD void force_outer(const double2* a, const double2* b, const double* w, int nrhs, unsigned V, unsigned y, int k,
                         M3 L[3]) {
    cx<double> t01[9], t10[9], td[9];  // b_1 conj(a_0), b_0 conj(a_1), b_0 conj(a_0) - b_1 conj(a_1)
#pragma unroll
    for (int q = 0; q < 9; ++q) t01[q] = t10[q] = td[q] = mk(0.0, 0.0);
    for (int r = 0; r < nrhs; ++r) {
        const double wr = w[r];
        if (wr == 0.0) continue;
        const double2* ar = a + ((size_t)r * 12 + 6 * k) * V + y;
        const double2* br = b + ((size_t)r * 12 + 6 * k) * V + y;
        cx<double> av[6], bv[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            const double2 p = ar[(size_t)c * V], q = br[(size_t)c * V];
            av[c] = mk(p.x, p.y);
            bv[c] = mk(wr * q.x, wr * q.y);
        }
#pragma unroll
        for (int bb = 0; bb < 3; ++bb)
#pragma unroll
            for (int aa = 0; aa < 3; ++aa) {
                const int q = 3 * bb + aa;
                cjmadd(t01[q], av[aa], bv[3 + bb]);
                cjmadd(t10[q], av[3 + aa], bv[bb]);
                cjmadd(td[q], av[aa], bv[bb]);
                cjmadd(td[q], av[3 + aa], -bv[3 + bb]);
            }
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        L[0].a[q] = t01[q] + t10[q];
        L[1].a[q] = times_mi(t01[q]) + times_i(t10[q]);
        L[2].a[q] = td[q];
    }
}

// The planes (0, l + 1) and (j, k) with l + 1 their Pauli index, l = 0 (2,3), 1 (1,3), 2 (1,2), from L0, L1 of the two chiral
// blocks: J = (K - K^+)/8, K = (i c_sw / 2) times the signed sum of clover_build.h.  Slot of a plane: l for (0, l + 1),
// 3 + l for the other.
DDWC_HD void force_planes(const M3& L0, const M3& L1, int l, double csw, M3& Ja, M3& Jb) {
    const cx<double> ic2 = mk(0.0, 0.5 * csw);
    const double sb = l == 1 ? 1.0 : -1.0;
    M3 Ka, Kb;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        Ka.a[q] = ic2 * (L0.a[q] - L1.a[q]);
        Kb.a[q] = ic2 * (sb * (L0.a[q] + L1.a[q]));
    }
    const M3 Da = dag(Ka), Db = dag(Kb);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        Ja.a[q] = 0.125 * (Ka.a[q] - Da.a[q]);
        Jb.a[q] = 0.125 * (Kb.a[q] - Db.a[q]);
    }
}
DDWC_HD int force_slot(int mu, int nu) { return mu == 0 ? nu - 1 : mu == 2 ? 3 : nu == 3 ? 4 : 5; }  // mu < nu

// A plaquette X0 X1 X2 X3 (matrices as they stand in the product, daggers taken) appears in the leaves of its four
// corners, which are cyclic shifts of it with the corner's J inserted: Re tr of X0 Ja X1 X2 X3 + X0 X1 Jb X2 X3 +
// X0 X1 X2 Jc X3 + X0 X1 X2 X3 Jd, J's in the order of the corners.  This is Z of Re tr[X0 Z].
template <class LX, class LJ>
DDWC_HD M3 plaquette_force(const LX& X, const LJ& J) {
    const M3 X1 = X(1);
    M3 T = add(mul(J(0), X1), mul(X1, J(1)));
    const M3 X2 = X(2), X3 = X(3);
    const M3 S = mul(X2, X3);
    T = mul(T, S);
    const M3 W = add(mul(X2, mul(J(2), X3)), mul(S, J(3)));
    return add(T, mul(X1, W));
}

// The link q (0 .. 3 in product order A B C^+ D^+, A = U_mu(z), B = U_nu(z + mu), C = U_mu(z + nu), D = U_nu(z)) of the
// plaquette (z, mu < nu): its contribution to the link's gradient.  at(c): the corner sites z, z + mu, z + mu + nu,
// z + nu; ldU(direction, site), ldJ(slot, site).
template <class AT, class LU, class LJ>
DDWC_HD M3 plaquette_link_force(int mu, int nu, int q, const AT& at, const LU& ldU, const LJ& ldJ) {
    const int slot = force_slot(mu, nu);
    auto link = [&](int k) {  // the k-th matrix of the product, cyclic
        switch (k & 3) {
            case 0: return ldU(mu, at(0));
            case 1: return ldU(nu, at(1));
            case 2: return dag(ldU(mu, at(3)));
            default: return dag(ldU(nu, at(0)));
        }
    };
    // the corner after the k-th matrix: A ends at z + mu (1), B at z + mu + nu (2), C^+ at z + nu (3), D^+ at z (0)
    const M3 Z = plaquette_force([&](int k) { return link(q + k); },
                                 [&](int k) { return ldJ(slot, at((q + k + 1) & 3)); });
    return q < 2 ? dag(Z) : Z;
}

// Clover part at link (x, mu): the plaquettes of its three planes on both sides.  nb(d, s): neighbour of s in
// direction d = 2 mu + (backward ? 1 : 0).
template <class NB, class LU, class LJ>
DDWC_HD M3 force_clover_link(int mu, int x, const NB& nb, const LU& ldU, const LJ& ldJ) {
    M3 G;
#pragma unroll
    for (int k = 0; k < 9; ++k) G.a[k] = mk(0.0, 0.0);
    const int xm = nb(2 * mu, x);
#pragma unroll 1
    for (int o = 0; o < 3; ++o) {
        const int nu = o + (o >= mu);
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {
            // z: the plaquette's corner; the link is the near edge (side 0: z = x) or the far one (z = x - nu)
            const int z = side ? nb(2 * nu + 1, x) : x;
            const int zm = side ? nb(2 * mu, z) : xm, zn = side ? x : nb(2 * nu, x), zmn = side ? xm : nb(2 * nu, xm);
            // in the plane (lo < hi) the corners in order are z, z + lo, z + lo + hi, z + hi
            const bool first = mu < nu;
            const int c1 = first ? zm : zn, c3 = first ? zn : zm;
            const int q = first ? (side ? 2 : 0) : (side ? 1 : 3);
            G = add(G, plaquette_link_force(first ? mu : nu, first ? nu : mu, q,
                                            [&](int c) { return c == 0 ? z : c == 1 ? c1 : c == 2 ? zmn : c3; }, ldU, ldJ));
        }
    }
    return G;
}

}  // namespace ddwc
