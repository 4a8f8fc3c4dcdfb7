// Dispatch order of the tiles of the operator kernels: the tiles sorted into spatial columns of whole blocks that run
// through all of time, inside a column by time slice, inside a slice by block and inside a block's slice (a cell) by
// number.  A tile belongs to the cell of its first site.
#pragma once
#include "ddwc_device.h"

namespace ddwc {

struct TileOrder {
    int c[3];      // blocks of a column along x1, x2, x3 (each divides the lattice's)
    int parities;  // 1: half fields, 2: full fields (parity-major inside a block)
    int nrhs;      // (site, RHS) pairs are numbered site-major, RHS-minor
    int shift;     // 1 << shift pairs a tile

    DDWC_HD int blocks() const { return c[0] * c[1] * c[2]; }  // of a column's time slice
    DDWC_HD int columns(const Geom& g) const { return g.nb[1] / c[0] * (g.nb[2] / c[1]) * (g.nb[3] / c[2]); }
    // the first tile that starts at or after site i
    DDWC_HD int first(long long i) const { return (int)((i * nrhs + (1LL << shift) - 1) >> shift); }
    // the block of column col at block time n0, number `in` of its slice
    DDWC_HD int block(const Geom& g, int col, int n0, int in) const {
        int n[4] = {n0, 0, 0, 0};
        for (int m = 3; m >= 1; --m) {
            const int nc = g.nb[m] / c[m - 1];
            n[m] = col % nc * c[m - 1] + in % c[m - 1];
            col /= nc;
            in /= c[m - 1];
        }
        return block_base(g, n) / g.Vb;
    }
    // the tiles [from, to) of parity p's sites in cell k of column col (cells: time slices, blocks in a slice)
    DDWC_HD void tiles(const Geom& g, int col, int k, int p, int& from, int& to) const {
        const int time = k / blocks(), n0 = time / g.b[0], slice = g.hvb / g.b[0];
        const long long i = ((long long)block(g, col, n0, k - time * blocks()) * parities + p) * g.hvb +
                            (long long)(time - n0 * g.b[0]) * slice;
        from = first(i);
        to = first(i + slice);
    }
};

}  // namespace ddwc
