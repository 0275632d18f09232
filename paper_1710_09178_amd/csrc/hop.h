// Link storage formats and stencil geometry of the hopping operators, shared by
// the Dslash kernels (dslash.hip) and the resident solver (resident.hip).
//   LinkD18  FP64, 9 complex entries            (144 B/link)
//   LinkD12  FP64, rows 0-1, row 2 rebuilt       (96 B/link)
//   LinkS18  FP32, 9 complex entries             (72 B/link)
//   LinkH12  FP16, rows 0-1, row 2 rebuilt       (24 B/link)
#pragma once

#include <hip/hip_fp16.h>

#include "common.h"

namespace stag {

namespace {

// conj(a b - c d); in FP64 with the multiply-adds spelt out, so that the kernels
// that read links through this header, and each of their kinds of load, round
// alike (the batched operator rebuilds its rows with the compiler's contraction)
__device__ __forceinline__ double2 minor_conj(double2 a, double2 b, double2 c, double2 d) {
    const double x = fma(c.y, d.y, fma(-c.x, d.x, fma(-a.y, b.y, a.x * b.x)));
    const double y = fma(-c.y, d.x, fma(-c.x, d.y, fma(a.y, b.x, a.x * b.y)));
    return make_double2(x, -y);
}
__device__ __forceinline__ float2 minor_conj(float2 a, float2 b, float2 c, float2 d) {
    return cconj(csub(cmul(a, b), cmul(c, d)));
}
template <class C>
__device__ __forceinline__ void rebuild_row2(C (&m)[9]) {
    m[6] = minor_conj(m[1], m[5], m[2], m[4]);
    m[7] = minor_conj(m[2], m[3], m[0], m[5]);
    m[8] = minor_conj(m[0], m[4], m[1], m[3]);
}

// FP64 link entry; NT: a non-temporal load, for link fields larger than the
// Infinity Cache, most of which every Dslash streams from HBM: they then do not
// evict the vectors the neighbours share.
template <bool NT>
__device__ __forceinline__ double2 link_entry(const double2* p) {
    if constexpr (NT) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        const d2v t = __builtin_nontemporal_load((const d2v*)p);
        return make_double2(t.x, t.y);
    } else {
        return *p;
    }
}

template <bool NT>
struct LinkD18T {
    using C = double2;
    using R = double;
    const double2* __restrict__ u;
    int turn = 0;  // NT: output sites at either end of a launch whose links are loaded plainly
    __device__ __forceinline__ void load(const Geom& g, int par, int mu, int cb, C (&m)[9]) const {
        const double2* p = u + link_off(g, par, mu, 0) + cb;
#pragma unroll
        for (int e = 0; e < 9; ++e) m[e] = link_entry<NT>(p + (size_t)e * g.vh);
    }
};
using LinkD18 = LinkD18T<false>;

template <bool NT>
struct LinkD12T {
    using C = double2;
    using R = double;
    const double2* __restrict__ u;
    int turn = 0;  // NT: output sites at either end of a launch whose links are loaded plainly
    __device__ __forceinline__ void load(const Geom& g, int par, int mu, int cb, C (&m)[9]) const {
        const double2* p = u + link12_off(g, par, mu, 0) + cb;
#pragma unroll
        for (int e = 0; e < 6; ++e) m[e] = link_entry<NT>(p + (size_t)e * g.vh);
        rebuild_row2(m);
    }
};
using LinkD12 = LinkD12T<false>;

struct LinkS18 {
    using C = float2;
    using R = float;
    const float2* __restrict__ u;
    __device__ __forceinline__ void load(const Geom& g, int par, int mu, int cb, C (&m)[9]) const {
        const float2* p = u + link_off(g, par, mu, 0) + cb;
#pragma unroll
        for (int e = 0; e < 9; ++e) m[e] = p[(size_t)e * g.vh];
    }
};

struct LinkH12 {
    using C = float2;
    using R = float;
    const __half2* __restrict__ u;
    __device__ __forceinline__ void load(const Geom& g, int par, int mu, int cb, C (&m)[9]) const {
        const __half2* p = u + link12_off(g, par, mu, 0) + cb;
#pragma unroll
        for (int e = 0; e < 6; ++e) m[e] = __half22float2(p[(size_t)e * g.vh]);
        rebuild_row2(m);
    }
};

__device__ __forceinline__ void hop_geometry(const Geom& g, int mu, int x, int y, int z, int t, int& cbf,
                                             int& cbb, bool& nf, bool& nb) {
    // nf / nb: the forward / backward term carries a minus sign
    if (mu == 0) {
        const int xp = (x + 1 == g.nx) ? 0 : x + 1;
        const int xm = (x == 0) ? g.nx - 1 : x - 1;
        cbf = cb_index(g, xp, y, z, t);
        cbb = cb_index(g, xm, y, z, t);
        nf = nb = false;
    } else if (mu == 1) {
        const int yp = (y + 1 == g.ny) ? 0 : y + 1;
        const int ym = (y == 0) ? g.ny - 1 : y - 1;
        cbf = cb_index(g, x, yp, z, t);
        cbb = cb_index(g, x, ym, z, t);
        nf = nb = (x & 1);
    } else if (mu == 2) {
        const int zp = (z + 1 == g.nz) ? 0 : z + 1;
        const int zm = (z == 0) ? g.nz - 1 : z - 1;
        cbf = cb_index(g, x, y, zp, t);
        cbb = cb_index(g, x, y, zm, t);
        nf = nb = ((x + y) & 1);
    } else {
        const int tp = (t + 1 == g.nt) ? 0 : t + 1;
        const int tm = (t == 0) ? g.nt - 1 : t - 1;
        cbf = cb_index(g, x, y, z, tp);
        cbb = cb_index(g, x, y, z, tm);
        const bool eta = ((x + y + z) & 1);
        nf = eta ^ (t == g.nt - 1);  // antiperiodic time boundary
        nb = eta ^ (t == 0);
    }
}

// Neighbours at distance 3 and the signs of the three-link paths to them.
// eta_mu does not depend on x_mu, so a path carries eta_mu(x) once; each of
// its links that leaves the last time slice adds a factor -1: the forward
// path from t crosses floor((t+3)/Nt) times, the backward path (from t-3 to
// t) 3 - floor((t-3+3Nt)/Nt) times, for any even Nt >= 2.
__device__ __forceinline__ int wrap_p3(int v, int n) {
    v += 3;
    v -= (v >= n) ? n : 0;
    v -= (v >= n) ? n : 0;
    return v;
}
__device__ __forceinline__ int wrap_m3(int v, int n) {
    v -= 3;
    v += (v < 0) ? n : 0;
    v += (v < 0) ? n : 0;
    return v;
}
__device__ __forceinline__ void hop3_geometry(const Geom& g, int mu, int x, int y, int z, int t, int& cbf,
                                              int& cbb, bool& nf, bool& nb) {
    if (mu == 0) {
        cbf = cb_index(g, wrap_p3(x, g.nx), y, z, t);
        cbb = cb_index(g, wrap_m3(x, g.nx), y, z, t);
        nf = nb = false;
    } else if (mu == 1) {
        cbf = cb_index(g, x, wrap_p3(y, g.ny), z, t);
        cbb = cb_index(g, x, wrap_m3(y, g.ny), z, t);
        nf = nb = (x & 1);
    } else if (mu == 2) {
        cbf = cb_index(g, x, y, wrap_p3(z, g.nz), t);
        cbb = cb_index(g, x, y, wrap_m3(z, g.nz), t);
        nf = nb = ((x + y) & 1);
    } else {
        cbf = cb_index(g, x, y, z, wrap_p3(t, g.nt));
        cbb = cb_index(g, x, y, z, wrap_m3(t, g.nt));
        const bool eta = ((x + y + z) & 1);
        nf = eta ^ (((t + 3) / g.nt) & 1);
        nb = eta ^ ((3 - (t - 3 + 3 * g.nt) / g.nt) & 1);
    }
}

}  // namespace

}  // namespace stag
