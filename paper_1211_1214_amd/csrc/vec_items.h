// Work-item mapping and partial sums shared by the site-parallel kernels.
//
// Workgroups are numbered tile-major / RHS-minor and remapped so that each of the 8 XCDs
// (which receive workgroups round-robin) sweeps one contiguous range: the RHS of a tile
// share its links and clover in that XCD's L2, and neighbouring tiles stay in one L2.
#pragma once
#include <type_traits>

#include "ddwc_internal.h"

namespace ddwc {

__device__ __forceinline__ int xcd_remap(int i, int n) {
    if ((n & 7) != 0) return i;
    return (i & 7) * (n >> 3) + (i >> 3);
}

struct TileRhs {
    int tile, rhs;
};

__device__ __forceinline__ TileRhs tile_rhs(int ntiles, int nrhs) {
    int L = xcd_remap(blockIdx.x, ntiles * nrhs);
    TileRhs t;
    t.tile = L / nrhs;
    t.rhs = L - t.tile * nrhs;
    return t;
}

// Partial sums are stored component-major: value k of (RHS r, tile w) at
// part[(k * nrhs + r) * ntiles + w], so that a reduction over the tiles reads each component it
// needs as one contiguous run.
template <int NV>
__device__ __forceinline__ void write_partials(double v[NV], double* part, int ntiles, int nrhs, TileRhs tr) {
    __shared__ double lds[NV * 16];
    block_sum<NV>(v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) part[((size_t)k * nrhs + tr.rhs) * ntiles + tr.tile] = v[k];
    }
}

// Work item of a multi-RHS vector kernel over n sites.  RHS-major fields [nrhs][NCW][n]:
// a workgroup holds WG consecutive sites of one RHS (tiles_of(n) tiles per RHS).
// RHS-innermost fields [NCW][n][nrhs] (RI): a workgroup holds WG consecutive (site, RHS)
// pairs, RHS fastest (tiles_of(n * nrhs) tiles in all).
struct VItem {
    unsigned i;   // site
    int r;        // right-hand side
    bool ok;      // inside the field
    int tile;
    unsigned g0;  // first pair of the workgroup (RI)
};

// NT: threads per workgroup of an RHS-innermost kernel (the RHS-major path always uses WG).
// order (may be null): the tile each dispatch slot processes, after the XCD remap.
template <bool RI, int NT = WG>
__device__ __forceinline__ VItem vitem(unsigned n, int nrhs, int ntiles, const int* __restrict__ order = nullptr) {
    VItem it;
    if (!RI) {
        const TileRhs tr = tile_rhs(ntiles, nrhs);
        it.tile = order ? order[tr.tile] : tr.tile;
        it.r = tr.rhs;
        it.i = it.tile * WG + threadIdx.x;
        it.ok = it.i < n;
        it.g0 = 0;
    } else {
        it.tile = xcd_remap(blockIdx.x, ntiles);
        if (order) it.tile = order[it.tile];
        it.g0 = (unsigned)it.tile * NT;
        const unsigned gi = it.g0 + threadIdx.x;
        it.ok = gi < n * (unsigned)nrhs;
        it.i = gi / (unsigned)nrhs;
        it.r = (int)(gi - it.i * (unsigned)nrhs);
    }
    return it;
}

// Component stride, element index and base offset (in words) of (site i, RHS r).
template <bool RI, class R>
struct VView {
    unsigned stride, idx;
    size_t base;
    __device__ __forceinline__ VView(unsigned n, int nrhs, unsigned i, int r) {
        if (RI) {
            stride = n * (unsigned)nrhs;
            idx = i * (unsigned)nrhs + r;
            base = 0;
        } else {
            stride = n;
            idx = i;
            base = (size_t)r * Traits<R>::NCW * n;
        }
    }
};

template <int NV, bool RI, int NT = WG, class T = double>
__device__ __forceinline__ void vpartials(double v[NV], double* part, int ntiles, const VItem& it, int nrhs) {
    if (RI) {
        seg_partials<NV, NT, T>(v, part, ntiles, it.tile, it.g0, nrhs);
    } else {
        TileRhs tr;
        tr.tile = it.tile;
        tr.rhs = it.r;
        write_partials<NV>(v, part, ntiles, nrhs, tr);
    }
}

// Staging of what the lanes of one site share (RHS-innermost FP32 and FP16 kernels with enough
// RHS): the own-site link records, the clover words and the neighbour-table entries of the sites
// a workgroup covers are copied into LDS with coalesced loads before the hop loop, which then
// reads them there: one copy per site instead of one vector-memory load per (site, RHS) lane.  They are
// read once, so they bypass the caches (non-temporal) that keep the neighbours' spinors.
// Fewer RHS cover more sites, and a workgroup's copy then leaves room for too few workgroups (solves of
// 4 / 5 / 6 RHS at 48x24^3, unstaged and staged: FP32 34.5, 42.2, 47.7 and -, -, 44.5 ms; FP16 28.4, -, 39.2 and 29.5, -,
// 36.6 ms; FP16 6 RHS at 32x16^3, whose fields stay in the last-level cache: 8.0 and 8.7 ms).
template <class S>
inline bool stage_ok(unsigned n, int nrhs) {
    if (std::is_same<S, double>::value) return false;
    return nrhs >= (std::is_same<S, H16>::value && n < (1u << 18) ? 8 : 6);
}
inline __host__ __device__ unsigned stg_sites(int nt, int nrhs) {  // sites that nt consecutive pairs can touch
    return (unsigned)((nt - 1) / nrhs + 2);
}

template <class S>
constexpr unsigned record_words() {  // 16-byte words of one own-site link record
    return 8 * 9 * sizeof(cx<typename Traits<S>::link>) / 16;
}
template <class S>
inline size_t stage_bytes(int nt, int nrhs) {
    return (size_t)stg_sites(nt, nrhs) * ((record_words<S>() + Traits<S>::NKW) * 16 + 8 * sizeof(int));
}

template <class S>
struct Staged {
    const cx<typename Traits<S>::link>* U;  // link records of sites l0, l0 + 1, ...
    const typename Traits<S>::kword* K;     // clover words [NKW][n] of the same sites
    const int* nbr;                         // neighbour-table entries [8][n] of the same sites
    unsigned l0, n;
};

// Copies the records, clover words and table entries of the sites of the workgroup's pairs;
// every thread of the workgroup must call it (it ends with a barrier).
template <class S, int NT = WG>
__device__ __forceinline__ Staged<S> stage_site_data(const VItem& it, unsigned n2, int nrhs,
                                                     const cx<typename Traits<S>::link>* __restrict__ Up,
                                                     const typename Traits<S>::kword* __restrict__ K,
                                                     const int* __restrict__ nbr) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static_assert(std::is_same<typename Traits<S>::kword, float4>::value, "clover words are float4");
    extern __shared__ __align__(16) char dyn[];
    v4* stg = (v4*)dyn;
    constexpr unsigned RW = record_words<S>(), NK = Traits<S>::NKW;
    const unsigned NS = stg_sites(NT, nrhs);
    const unsigned l0 = it.g0 / (unsigned)nrhs;
    unsigned l1 = (it.g0 + NT - 1) / (unsigned)nrhs + 1;
    if (l1 > n2) l1 = n2;
    const unsigned ns = l1 - l0;  // <= NS
    const v4* src = (const v4*)Up + (size_t)l0 * RW;
    for (unsigned k = threadIdx.x; k < ns * RW; k += NT) stg[k] = __builtin_nontemporal_load(src + k);
    v4* ck = stg + NS * RW;
    for (unsigned k = threadIdx.x; k < NK * ns; k += NT) {
        const unsigned w = k / ns, j = k - w * ns;
        ck[w * NS + j] = __builtin_nontemporal_load((const v4*)K + ((size_t)w * n2 + l0 + j));
    }
    int* cn = (int*)(ck + NK * NS);
    for (unsigned k = threadIdx.x; k < 8 * ns; k += NT) {
        const unsigned d = k / ns, j = k - d * ns;
        cn[d * NS + j] = nbr[(size_t)d * n2 + l0 + j];
    }
    __syncthreads();
    Staged<S> st;
    st.U = (const cx<typename Traits<S>::link>*)stg;
    st.K = (const typename Traits<S>::kword*)ck;
    st.nbr = cn;
    st.l0 = l0;
    st.n = NS;
    return st;
}

}  // namespace ddwc
