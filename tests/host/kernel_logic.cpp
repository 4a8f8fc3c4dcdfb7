// Host-side execution of the library's per-site device code (test harness only).
// The same __host__ __device__ functions the HIP kernels call (geometry, spin
// projection, clover packing and application) run here on the CPU over every site,
// so their logic can be compared with the FP64 oracle without a GPU.
#include <vector>

#include "../../paper_1211_1214_amd/csrc/clover_build.h"
#include "../../paper_1211_1214_amd/csrc/uniform_mem.h"

using namespace ddwc;

// All hops of site s, as the operator kernels take them: field in, forward links Uf at s, backward links Ub at the
// neighbour, table nbr (index spaces of n sites).
static void all_hops(unsigned n, unsigned s, const double2* in, const cx<double>* Uf, const cx<double>* Ub, const int* nbr,
                     cx<double> acc[12]) {
    auto entry = [&](int d) { return nbr[(size_t)d * n + s]; };
    auto target = [&](int d) { return d < 2 && entry(d) < 0 ? (unsigned)~entry(d) : (unsigned)entry(d); };
    hops_pipelined<double, true>(
        acc, [&](int d, cx<double> q[12]) { load_spinor(in, n, target(d), q); },
        [&](int d, cx<double> u[9]) { load_link((d & 1) ? Ub : Uf, n, d >> 1, (d & 1) ? target(d) : s, u); },
        [&](int d) { return entry(d) < 0; }, [](int) { return true; });
}

// mode: 0 full operator, 1 Dirichlet blocks of colour `colour` (other colour zero),
//       2 hops crossing block faces into colour `colour` (other colour zero).
extern "C" int host_apply(const int* lat, const int* blk, int tbc, double csw, const double* links_canon,
                          const double* in_canon, double kappa, int mode, int colour, double* out_canon,
                          double* clover_out) {
    Geom g = make_geom(lat, blk, tbc);
    const int V = g.V;
    std::vector<cx<double>> U((size_t)36 * V);
    std::vector<int> can(V);
    for (int s = 0; s < V; ++s) {
        Site S = decode(g, s);
        can[s] = canonical_index(g, S);
        for (int mu = 0; mu < 4; ++mu)
            for (int k = 0; k < 9; ++k) {
                const double* src = links_canon + 2 * (((size_t)mu * V + can[s]) * 9 + k);
                U[((size_t)mu * 9 + k) * V + s] = mk(src[0], src[1]);
            }
    }
    std::vector<int> nbr((size_t)8 * V);
    for (int s = 0; s < V; ++s) {
        const Site S = decode(g, s);
        for (int mu = 0; mu < 4; ++mu) {
            nbr[(size_t)(2 * mu) * V + s] = table_entry<+1>(g, s, S, mu);
            nbr[(size_t)(2 * mu + 1) * V + s] = table_entry<-1>(g, s, S, mu);
        }
    }
    std::vector<double2> K((size_t)36 * V), in((size_t)12 * V);
    for (int s = 0; s < V; ++s) {
        double a[72];
        clover_site(g, U.data(), csw, s, a);
        for (int k = 0; k < 36; ++k) K[(size_t)k * V + s] = make_double2(a[2 * k], a[2 * k + 1]);
        if (clover_out)
            for (int k = 0; k < 72; ++k) clover_out[(size_t)can[s] * 72 + k] = a[k];
        for (int c = 0; c < 12; ++c) {
            const double* src = in_canon + 2 * ((size_t)can[s] * 12 + c);
            in[(size_t)c * V + s] = make_double2(src[0], src[1]);
        }
    }
    const double mass4 = 4.0 + (1.0 / (2.0 * kappa) - 4.0);
    for (int s = 0; s < V; ++s) {
        cx<double> y[12];
        const int c_s = s / (V / 2);
        if (mode == 0) {
            cx<double> c[12];
            all_hops(V, s, in.data(), U.data(), U.data(), nbr.data(), y);
            load_spinor(in.data(), V, s, c);
            apply_diag<double>(K.data(), V, s, mass4, c, y, -0.5);
        } else if (mode == 1 && c_s == colour)
            site_operator<double, true, HOPS_INSIDE>(g, s, in.data(), U.data(), K.data(), nbr.data(), mass4, y, 8);
        else if (mode == 2 && c_s == colour)
            site_operator<double, false, HOPS_CROSSING>(g, s, in.data(), U.data(), nullptr, nbr.data(), 0.0, y, 8);
        else
            for (int c = 0; c < 12; ++c) y[c] = mk(0.0, 0.0);
        for (int c = 0; c < 12; ++c) {
            out_canon[2 * ((size_t)can[s] * 12 + c)] = y[c].re;
            out_canon[2 * ((size_t)can[s] * 12 + c) + 1] = y[c].im;
        }
    }
    return 0;
}

// Even-odd operator on the host with the library's own helpers: y_e = Mee x_e with
// Mee = A_ee - 1/4 H_eo A_oo^-1 H_oe, half fields built as the setup kernel builds them.
// Output in canonical layout, zero on odd sites.  Requires every block extent even.
#include "../../paper_1211_1214_amd/csrc/eo.h"
extern "C" int host_eo_apply(const int* lat, const int* blk, int tbc, double csw, const double* links_canon,
                             const double* in_canon, double kappa, double* out_canon) {
    Geom g = make_geom(lat, blk, tbc);
    if (!g.eo) return -1;
    const int V = g.V, n2 = V / 2;
    std::vector<cx<double>> U((size_t)36 * V);
    std::vector<int> can(V), nbr((size_t)8 * V);
    for (int s = 0; s < V; ++s) {
        const Site S = decode(g, s);
        can[s] = canonical_index(g, S);
        for (int mu = 0; mu < 4; ++mu) {
            for (int k = 0; k < 9; ++k) {
                const double* src = links_canon + 2 * (((size_t)mu * V + can[s]) * 9 + k);
                U[((size_t)mu * 9 + k) * V + s] = mk(src[0], src[1]);
            }
            nbr[(size_t)(2 * mu) * V + s] = table_entry<+1>(g, s, S, mu);
            nbr[(size_t)(2 * mu + 1) * V + s] = table_entry<-1>(g, s, S, mu);
        }
    }
    const double mass4 = 4.0 + (1.0 / (2.0 * kappa) - 4.0);
    std::vector<cx<double>> Uh((size_t)2 * 36 * n2);
    std::vector<double2> Kh((size_t)2 * 36 * n2), Ah((size_t)36 * n2), xe((size_t)12 * n2), xo((size_t)12 * n2, make_double2(0, 0));
    std::vector<int> nh((size_t)2 * 8 * n2);
    for (int s = 0; s < V; ++s) {
        int p;
        const unsigned i = half_index(g, s, p);
        if (full_index(g, i, p) != (unsigned)s) return -2;
        for (int mu = 0; mu < 4; ++mu)
            for (int k = 0; k < 9; ++k) Uh[(((size_t)p * 4 + mu) * 9 + k) * n2 + i] = U[((size_t)mu * 9 + k) * V + s];
        double a[72], b[72];
        clover_site(g, U.data(), csw, s, a);
        for (int k = 0; k < 36; ++k) Kh[((size_t)p * 36 + k) * n2 + i] = make_double2(a[2 * k], a[2 * k + 1]);
        if (p == 1) {
            clover_inverse_site(a, mass4, b);
            for (int k = 0; k < 36; ++k) Ah[(size_t)k * n2 + i] = make_double2(b[2 * k], b[2 * k + 1]);
        }
        for (int d = 0; d < 8; ++d) nh[((size_t)p * 8 + d) * n2 + i] = half_entry(g, nbr[(size_t)d * V + s]);
        if (p == 0)
            for (int c = 0; c < 12; ++c) {
                const double* src = in_canon + 2 * ((size_t)can[s] * 12 + c);
                xe[(size_t)c * n2 + i] = make_double2(src[0], src[1]);
            }
    }
    const cx<double>* U0 = Uh.data();
    const cx<double>* U1 = Uh.data() + (size_t)36 * n2;
    // t_o = A_oo^-1 H_oe x_e
    for (int i = 0; i < n2; ++i) {
        cx<double> acc[12], w[12];
        all_hops(n2, i, xe.data(), U1, U0, nh.data() + (size_t)8 * n2, acc);
        for (int c = 0; c < 12; ++c) w[c] = mk(0.0, 0.0);
        apply_diag<double>(Ah.data(), n2, i, 0.0, acc, w, 0.0);
        store_spinor(xo.data(), n2, i, w);
    }
    for (size_t k = 0; k < (size_t)24 * V; ++k) out_canon[k] = 0;
    // y_e = A_ee x_e - 1/4 H_eo t_o
    for (int i = 0; i < n2; ++i) {
        cx<double> acc[12], c[12];
        all_hops(n2, i, xo.data(), U0, U1, nh.data(), acc);
        load_spinor(xe.data(), n2, i, c);
        apply_diag<double>(Kh.data(), n2, i, mass4, c, acc, -0.25);
        const int s = can[full_index(g, i, 0)];
        for (int k = 0; k < 12; ++k) {
            out_canon[2 * ((size_t)s * 12 + k)] = acc[k].re;
            out_canon[2 * ((size_t)s * 12 + k) + 1] = acc[k].im;
        }
    }
    return 0;
}

// Link gradient of Re <a, D(U) b> (one RHS, weight 1) with the library's force code: hop part
// and clover part, in canonical layout [4][V][3][3] (re, im).
#include "../../paper_1211_1214_amd/csrc/force.h"
extern "C" int host_force(const int* lat, const int* blk, int tbc, double csw, const double* links_canon,
                          const double* a_canon, const double* b_canon, double* grad_canon) {
    Geom g = make_geom(lat, blk, tbc);
    const int V = g.V;
    std::vector<cx<double>> U((size_t)36 * V), G((size_t)36 * V, mk(0.0, 0.0));
    std::vector<int> can(V), nbr((size_t)8 * V);
    std::vector<double2> a((size_t)12 * V), b((size_t)12 * V);
    for (int s = 0; s < V; ++s) {
        const Site S = decode(g, s);
        can[s] = canonical_index(g, S);
        for (int mu = 0; mu < 4; ++mu) {
            for (int k = 0; k < 9; ++k) {
                const double* src = links_canon + 2 * (((size_t)mu * V + can[s]) * 9 + k);
                U[((size_t)mu * 9 + k) * V + s] = mk(src[0], src[1]);
            }
            nbr[(size_t)(2 * mu) * V + s] = table_entry<+1>(g, s, S, mu);
            nbr[(size_t)(2 * mu + 1) * V + s] = table_entry<-1>(g, s, S, mu);
        }
        for (int c = 0; c < 12; ++c) {
            a[(size_t)c * V + s] = make_double2(a_canon[2 * ((size_t)can[s] * 12 + c)], a_canon[2 * ((size_t)can[s] * 12 + c) + 1]);
            b[(size_t)c * V + s] = make_double2(b_canon[2 * ((size_t)can[s] * 12 + c)], b_canon[2 * ((size_t)can[s] * 12 + c) + 1]);
        }
    }
    const double w = 1.0;
    for (int s = 0; s < V; ++s)
        for (int mu = 0; mu < 4; ++mu) force_hop_site(g, nbr.data(), a.data(), b.data(), &w, 1, G.data(), s, mu);
    if (csw != 0.0) {  // (the three passes of the kernels: outer products, planes, links)
        std::vector<cx<double>> J((size_t)54 * V);
        for (int y = 0; y < V; ++y) {
            M3 L[2][3], P[6];
            for (int k = 0; k < 2; ++k) force_outer(a.data(), b.data(), &w, 1, (unsigned)V, (unsigned)y, k, L[k]);
            for (int l = 0; l < 3; ++l) force_planes(L[0][l], L[1][l], l, csw, P[l], P[3 + l]);
            for (int slot = 0; slot < 6; ++slot)
                for (int k = 0; k < 9; ++k) J[((size_t)slot * 9 + k) * V + y] = P[slot].a[k];
        }
        auto nb = [&](int d, int s) {
            const int e = nbr[(size_t)d * V + s];
            return e < 0 ? ~e : e;
        };
        for (int s = 0; s < V; ++s)
            for (int mu = 0; mu < 4; ++mu) {
                const M3 Z = force_clover_link(
                    mu, s, nb, [&](int m, int t) { return ld(U.data(), g, m, t); },
                    [&](int slot, int t) { return ld(J.data(), g, slot, t); });
                for (int k = 0; k < 9; ++k) {
                    cx<double>& o = G[((size_t)mu * 9 + k) * V + s];
                    o = o + Z.a[k];
                }
            }
    }
    for (int s = 0; s < V; ++s)
        for (int mu = 0; mu < 4; ++mu)
            for (int k = 0; k < 9; ++k) {
                const cx<double> v = G[((size_t)mu * 9 + k) * V + s];
                grad_canon[2 * (((size_t)mu * V + can[s]) * 9 + k)] = v.re;
                grad_canon[2 * (((size_t)mu * V + can[s]) * 9 + k) + 1] = v.im;
            }
    return 0;
}

// FP16 spinor storage: store then load one spinor (24 reals) through the library's code.
extern "C" int host_h16_roundtrip(const double* in, double* out, float* scale_out) {
    struct alignas(16) Buf {
        hw16 w[3];
        float scale[4];
    } buf;
    cx<float> p[12], q[12];
    for (int c = 0; c < 12; ++c) p[c] = mk((float)in[2 * c], (float)in[2 * c + 1]);
    store_spinor(buf.w, 1, 0, p);
    load_spinor((const hw16*)buf.w, 1, 0, q);
    for (int c = 0; c < 12; ++c) {
        out[2 * c] = q[c].re;
        out[2 * c + 1] = q[c].im;
    }
    *scale_out = buf.scale[0];
    return 0;
}

// Dispatch order of the tiles: the kernel's walk over columns and cells, and the same by sorting all tiles on the position
// of their first site.  Returns the number of tiles; -1 if a column does not start where the counts of those before say.
#include <algorithm>
#include <array>
#include "../../paper_1211_1214_amd/csrc/tile_order.h"
extern "C" int host_tile_order(const int* lat, const int* blk, int parities, int nrhs, int nt, const int* c, int* walked,
                               int* sorted) {
    const Geom g = make_geom(lat, blk, -1);
    TileOrder o{{c[0], c[1], c[2]}, parities, nrhs, 0};
    while (1 << o.shift < nt) ++o.shift;
    const int per_block = parities * g.hvb, nin = o.blocks();
    int at = 0, before = 0;
    for (int col = 0; col < o.columns(g); ++col) {
        if (at != before) return -1;
        for (int k = 0; k < g.L[0] * nin; ++k)
            for (int p = 0; p < parities; ++p) {
                int from, to;
                o.tiles(g, col, k, p, from, to);
                for (int t = from; t < to; ++t) walked[at++] = t;
            }
        for (int w = 0; w < g.nb[0] * nin; ++w) {
            const long long B = o.block(g, col, w / nin, w % nin);
            before += o.first((B + 1) * per_block) - o.first(B * per_block);
        }
    }
    const long long pairs = (long long)per_block * g.NB * nrhs;
    const int n = (int)((pairs + nt - 1) / nt);
    std::vector<std::array<int, 9>> keys(n);
    for (int t = 0; t < n; ++t) {
        const long long i = (long long)t * nt / nrhs;
        const int B = (int)(i / per_block), loc = (int)(i % per_block);
        // (half fields: site h of block B is taken as the even site there, which has its coordinates up to x3)
        const Site S = decode(g, B * g.Vb + loc);
        const int time = S.n[0] * g.b[0] + S.l[0];
        keys[t] = {S.n[1] / c[0], S.n[2] / c[1], S.n[3] / c[2], time, S.n[1] % c[0], S.n[2] % c[1], S.n[3] % c[2], t, 0};
    }
    std::sort(keys.begin(), keys.end());
    for (int t = 0; t < n; ++t) sorted[t] = keys[t][7];
    return at == n && at == before ? n : -1;
}
