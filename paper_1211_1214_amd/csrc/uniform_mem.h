// Global accesses at (wave-uniform plane pointer, 32-bit byte offset per lane).
//
// The planes of a field (spinor words, link entries, clover words) share one per-lane offset and
// differ in their base, which is uniform.  Left alone, the compiler folds the per-lane offset into
// one 64-bit pointer and then adds each plane's distance to it in vector registers: one 64-bit
// vector add and two registers per load, and in a loop it hoists all of these sums out of it.  A
// Planes walks the planes of a field instead: its pointer is a scalar register pair that passes
// through an empty asm statement, so that every access is that pair plus the shared offset, and the
// step to the next plane is two scalar additions.
//
// The pointer MUST be uniform over the wave (kernel arguments, blockIdx); byte offsets stay below
// 4 GiB and come from byte_offset().
#pragma once
#include "ddwc_device.h"

namespace ddwc {

// i * size as a byte offset, opaque to the compiler (which would otherwise fold the shift into the
// 64-bit address, in vector registers).
__device__ __forceinline__ unsigned byte_offset(unsigned i, unsigned size) {
    unsigned o = i * size;
    asm("" : "+v"(o));
    return o;
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef double d2v __attribute__((ext_vector_type(2)));
template <class R>
struct VecOf;
template <>
struct VecOf<float> {
    typedef f4v word;  // spinor and clover word
    typedef f2v link;  // link entry
};
template <>
struct VecOf<double> {
    typedef d2v word;
    typedef d2v link;
};

struct Planes {
    typedef __attribute__((address_space(1))) char* gptr;
    gptr p;
    unsigned long long step;  // bytes from plane to plane
    // n elements of size bytes per plane, from plane k of base
    template <class T>
    __device__ __forceinline__ Planes(const T* base, unsigned n, unsigned k = 0)
        : p((gptr)(unsigned long long)base + (unsigned long long)n * sizeof(T) * k),
          step((unsigned long long)n * sizeof(T)) {}
    // the element at byte offset off of the next plane
    template <class V>
    __device__ __forceinline__ V load(unsigned off) {
        asm("" : "+s"(p));
        const V v = *(const __attribute__((address_space(1))) V*)(p + off);
        p += step;
        return v;
    }
    template <class V>
    __device__ __forceinline__ void store_nt(unsigned off, V v) {
        asm("" : "+s"(p));
        __builtin_nontemporal_store(v, (__attribute__((address_space(1))) V*)(p + off));
        p += step;
    }
    template <class V>
    __device__ __forceinline__ void store(unsigned off, V v) {
        asm("" : "+s"(p));
        *(__attribute__((address_space(1))) V*)(p + off) = v;
        p += step;
    }
};

// An opaque copy of a uniform pointer: what is computed from it is neither merged with what was
// computed from another copy nor moved out of a loop (either would keep the pointers of all planes
// alive).
template <class T>
__device__ __forceinline__ T* fresh(T* p) {
    unsigned long long q = (unsigned long long)p;
    asm volatile("" : "+s"(q));
    return (T*)q;
}

// Orders the computation of a spinor before every later fresh(), pin() and reissue(): instruction
// selection otherwise gathers the loads of a long straight-line body at its start and spills them.  (On the host, where
// hops_pipelined is checked too, there is nothing to order.)
template <class R>
DDWC_HD void pin6(cx<R> p[6]) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile(""
                 : "+v"(p[0].re), "+v"(p[0].im), "+v"(p[1].re), "+v"(p[1].im), "+v"(p[2].re), "+v"(p[2].im),
                   "+v"(p[3].re), "+v"(p[3].im), "+v"(p[4].re), "+v"(p[4].im), "+v"(p[5].re), "+v"(p[5].im));
#endif
}
template <class R>
DDWC_HD void pin(cx<R> p[12]) {
    pin6(p);
    pin6(p + 6);
}
DDWC_HD void sched_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
}
// The loads addressed with the returned offset are issued after the last pin().
__device__ __forceinline__ unsigned reissue(unsigned off) {
    asm volatile("" : "+v"(off));
    return off;
}

__device__ __forceinline__ void uload_spinor(const float4* f, unsigned n, unsigned off, cx<float> p[12]) {
    Planes q(f, n);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const f4v w = q.load<f4v>(off);
        p[2 * k] = mk(w.x, w.y);
        p[2 * k + 1] = mk(w.z, w.w);
    }
}
__device__ __forceinline__ void uload_spinor(const double2* f, unsigned n, unsigned off, cx<double> p[12]) {
    Planes q(f, n);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        const d2v w = q.load<d2v>(off);
        p[c] = mk(w.x, w.y);
    }
}
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
// FP16 storage: three word planes and a plane of scales (ddwc_device.h)
__device__ __forceinline__ void uload_spinor(const hw16* f, unsigned n, unsigned off, cx<float> p[12]) {
    Planes q(f, n);
    h8v w[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = q.load<h8v>(off);
    unsigned o4 = off >> 2;
    asm("" : "+v"(o4));
    const float sc = q.load<float>(o4);
#pragma unroll
    for (int k = 0; k < 12; ++k) p[k] = mk(sc * (float)w[k >> 2][2 * (k & 3)], sc * (float)w[k >> 2][2 * (k & 3) + 1]);
}
// p as FP16 halves of multiples of its largest component modulus (returned)
__device__ __forceinline__ float to_half(const cx<float> p[12], h8v w[3]) {
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < 12; ++c) m = fmaxf(m, fmaxf(fabsf(p[c].re), fabsf(p[c].im)));
    const float inv = m > 0.f ? 1.f / m : 0.f;
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        w[c >> 2][2 * (c & 3)] = (_Float16)(inv * p[c].re);
        w[c >> 2][2 * (c & 3) + 1] = (_Float16)(inv * p[c].im);
    }
    return m;
}
__device__ __forceinline__ void ustore_spinor(hw16* f, unsigned n, unsigned off, const cx<float> p[12]) {
    h8v w[3];
    const float m = to_half(p, w);
    Planes q(f, n);
#pragma unroll
    for (int k = 0; k < 3; ++k) q.store<h8v>(off, w[k]);
    unsigned o4 = off >> 2;
    asm("" : "+v"(o4));
    q.store<float>(o4, m);
}
__device__ __forceinline__ void ustore_spinor(float4* f, unsigned n, unsigned off, const cx<float> p[12]) {
    Planes q(f, n);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        q.store<f4v>(off, (f4v){p[2 * k].re, p[2 * k].im, p[2 * k + 1].re, p[2 * k + 1].im});
}
__device__ __forceinline__ void ustore_spinor(double2* f, unsigned n, unsigned off, const cx<double> p[12]) {
    Planes q(f, n);
#pragma unroll
    for (int c = 0; c < 12; ++c) q.store<d2v>(off, (d2v){p[c].re, p[c].im});
}

__device__ __forceinline__ void ustore_spinor_nt(float4* f, unsigned n, unsigned off, const cx<float> p[12]) {
    Planes q(f, n);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        q.store_nt<f4v>(off, (f4v){p[2 * k].re, p[2 * k].im, p[2 * k + 1].re, p[2 * k + 1].im});
}

// The next link of a walk over entry-major links [4][9][n] (nine planes), of the site at byte offset off.
template <class R>
__device__ __forceinline__ void uload_link(Planes& q, unsigned off, cx<R> u[9]) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const typename VecOf<R>::link w = q.load<typename VecOf<R>::link>(off);
        u[k] = mk(w.x, w.y);
    }
}

// Packed links: per direction planes of 16-byte words (FP32: four planes of two entries, FP16: two of four)
// and one plane of the last entry, n elements each: five (three) loads per link instead of nine.
template <class L>
struct PackedLinks {
    Planes::gptr p;
    unsigned long long n16;
    __device__ __forceinline__ PackedLinks(const char* U, unsigned n) : p((Planes::gptr)(unsigned long long)U), n16(16ull * n) {}
    // the link of the next direction of the site at byte offset off16 (its index times 16)
    __device__ __forceinline__ void next(unsigned off16, cx<float> u[9]) {
        constexpr int PW = 16 / sizeof(cx<L>), NW = 8 / PW;
        typedef L wv __attribute__((ext_vector_type(2 * PW)));
        typedef L ev __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            asm("" : "+s"(p));
            const wv w = *(const __attribute__((address_space(1))) wv*)(p + off16);
#pragma unroll
            for (int i = 0; i < PW; ++i) u[PW * k + i] = mk((float)w[2 * i], (float)w[2 * i + 1]);
            p += n16;
        }
        unsigned oe = off16 / PW;
        asm("" : "+v"(oe));
        asm("" : "+s"(p));
        const ev w = *(const __attribute__((address_space(1))) ev*)(p + oe);
        u[8] = mk((float)w.x, (float)w.y);
        p += n16 / PW;
    }
};

// The packed Hermitian 6x6 blocks K [NKW][n] of one site, loaded in two parts: the diagonals and the
// first block's off-diagonal reals, then the second block's (which start inside the last word of the
// first part in FP32).  y = (mass4 + C) p + hsc y as apply_diag.
template <class R>
struct UDiag {
    typedef typename VecOf<R>::word V;
    static constexpr int PW = sizeof(V) / sizeof(R);         // reals per word
    static constexpr int W0 = (42 + PW - 1) / PW, W1 = 72 / PW;
    Planes q;
    unsigned off;
    R w[72];
    __device__ __forceinline__ UDiag(const typename Traits<R>::word* K, unsigned n, unsigned o) : q(K, n), off(o) {}
    __device__ __forceinline__ void words(int k0, int k1) {
#pragma unroll
        for (int k = k0; k < k1; ++k) {
            const V v = q.template load<V>(off);
#pragma unroll
            for (int i = 0; i < PW; ++i) w[PW * k + i] = v[i];
        }
    }
    __device__ __forceinline__ void first() { words(0, W0); }
    __device__ __forceinline__ void apply(R mass4, const cx<R> p[12], cx<R> y[12], R hsc) {
        diag_block<R>(w, w + 12, mass4, p, y, hsc);
        words(W0, W1);
        diag_block<R>(w + 6, w + 42, mass4, p + 6, y + 6, hsc);
    }
};

// acc = sum over the eight hops of (1 -+ g_mu) W psi(neighbour), with the neighbour's spinor from lq(d, q) and
// the link from lu(d, u), called at compile-time d in order; flip(d) (d = 0, 1: the hops in time) says
// whether the hop crosses an antiperiodic boundary, and take(d) whether it belongs to the sum.
// The spinor of hop d + 1 is loaded into the registers of the spinor of hop d as soon as that is projected, so that
// it is in flight during the products of hop d at no cost in registers, and (NEXT_LINK) the next link
// beside the current one.
template <class R, bool NEXT_LINK, class LQ, class LU, class Flip, class Take>
DDWC_HD void hops_pipelined(cx<R> acc[12], LQ&& lq, LU&& lu, Flip&& flip, Take&& take) {
    cx<R> q[12], u[9], un[9], h[6];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = mk(R(0), R(0));
    lq(0, q);
    lu(0, u);
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        if (NEXT_LINK && d + 1 < 8) lu(d + 1, un);
        sched_barrier();
        proj_dispatch<R>(d, q, h);
        if (d < 2 && flip(d)) {
#pragma unroll
            for (int c = 0; c < 6; ++c) h[c] = -h[c];
        }
        pin6(h);
        if (d + 1 < 8) lq(d + 1, q);
        sched_barrier();
        if (take(d)) apply_dispatch<R>(d, u, h, acc);
        pin(acc);
        if (NEXT_LINK) {
#pragma unroll
            for (int k = 0; k < 9; ++k) u[k] = un[k];
        } else if (d + 1 < 8) {
            lu(d + 1, u);
        }
    }
}

}  // namespace ddwc
