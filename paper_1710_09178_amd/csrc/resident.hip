// The resident multi-shift CG: one cooperative launch per solve (Sec. 4).
//
// On a lattice of a few hundred 64-site tiles a CG iteration made of launches
// is a chain of launch gaps and cold memory round trips (16^3x8: 12.9 us per
// iteration, of which the 38 MB of links would take 4 us), so here one grid of
// co-resident blocks runs the whole solve.  Block t owns the 64 even and the 64
// odd sites of tile t.  A lane applies one hop at one site, of D_oe and of D_eo,
// and keeps those two links in registers from the first iteration to the last.
// Exchanges inside the wave add the hops of a site and leave its colours c in
// lane rows c, which own these elements of every vector.  What a lane needs
// from other blocks travels through memory, from its own block through LDS:
//
//   iteration j, p_j known at the own sites and at the neighbours read
//     w = D_oe p_j          own odd sites, published
//     Ap = mt p_j - D_eo w  own even sites, published; block sums of |r_j|^2,
//                           <p,Ap>, <r,Ap>, <Ap,Ap> published
//     the sums of all blocks, added in a fixed order (by groups of 16 blocks,
//     so that a block polls 512 bytes and not 8 KB), give every block
//     the same alpha and beta; r and p are then stepped at the own sites and,
//     from the published Ap, at the neighbours read, with the same fused
//     multiply-adds (cg_r_next, cg_p_next), hence to the same bits.
//
// Publishing.  Every published 64-bit word lives in a buffer that held an empty
// word (kResEmptyHi, kResEmptyLo) before; a reader polls the words it needs until
// none is empty.  Stores and loads are device-scope accesses (sc1: past the
// XCDs' L2s), one or two aligned 64-bit words each; since a word is its own flag,
// no order between different words is needed, no fence and no cache writeback.
// A value whose high half happens to be kResEmptyHi (a NaN, in FP64 one that no
// arithmetic produces) gets another NaN's.
//
// Reuse.  w has two buffers (by j mod 2), Ap and the sums three (j mod 3).
// When a block has the total sums of j - 1, every block has consumed w_{j-1},
// Ap_{j-2} and the sums of j - 2 (it publishes its sums of j - 1 after that),
// so the block then empties its own words of those.  It waits
// for these stores before it publishes its sums of j, and nobody polls the
// buffers again (for j + 1) before having the totals of j, which need those: a
// stale word is never taken for a new one.
//
// Every wait ends: a poll that lasts a.wait gives up and raises
// st->aborted, which all other polls watch; the block leaves at the end of the
// iteration and the host repeats the solve with the launch loop.  The grid is
// launched cooperatively, so all its blocks are resident or none is.
//
// Shifted systems: per window of `lag` steps as in the other loops, by the
// lanes that own an (even site, colour) pair.  A window's residuals and scalars
// stay in LDS (two buffers) while the next window runs, and its shifts are
// updated a group per iteration while the neighbours' w is under way; x_s and
// p_s stay in this XCD's L2 (only their owner touches them).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "hop.h"
#include "msfused.h"
#include "resident.h"

namespace stag {

namespace {

typedef unsigned long long u64;
typedef unsigned u2v __attribute__((ext_vector_type(2)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));
// As a double and as two floats a signalling NaN, told apart by its high half.
constexpr unsigned kResEmptyHi = 0x7FF4C3A5u, kResEmptyLo = 0xD2E1B697u;

// The exchange area as a buffer resource: a lane offset and a uniform offset, in
// bytes, per access; sc1 (device scope) on every load and store.
struct Xch {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Xch(void* p, unsigned bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000)) {}
    static constexpr int kScope = 16;  // sc1
    __device__ __forceinline__ u2v get2(unsigned off, unsigned at) const {
        return __builtin_amdgcn_raw_buffer_load_b64(r, off, at, kScope);
    }
    __device__ __forceinline__ u4v get4(unsigned off, unsigned at) const {
        return __builtin_amdgcn_raw_buffer_load_b128(r, off, at, kScope);
    }
    __device__ __forceinline__ void put2(unsigned off, unsigned at, u2v v) const {
        __builtin_amdgcn_raw_buffer_store_b64(v, r, off, at, kScope);
    }
    __device__ __forceinline__ void put4(unsigned off, unsigned at, u4v v) const {
        __builtin_amdgcn_raw_buffer_store_b128(v, r, off, at, kScope);
    }
};
// zero exactly for an empty word (the only ones with this high half)
__device__ __forceinline__ unsigned xseen(unsigned hi) { return hi ^ kResEmptyHi; }
__device__ __forceinline__ unsigned xhigh(unsigned hi) { return hi == kResEmptyHi ? 0x7FFCC3A5u : hi; }
__device__ __forceinline__ u2v xword(double v) {
    return u2v{(unsigned)__double2loint(v), xhigh((unsigned)__double2hiint(v))};
}
__device__ __forceinline__ double xdouble(u2v w) { return __hiloint2double((int)w.y, (int)w.x); }

// one vector element: a 16-byte word pair (FP64) or one 64-bit word (FP32)
template <class V>
struct XElem;
template <>
struct XElem<double2> {
    using T = u4v;
    static constexpr unsigned kBytes = 16;
    static __device__ __forceinline__ void put(const Xch& x, unsigned off, unsigned at, double2 v) {
        const u2v a = xword(v.x), b = xword(v.y);
        x.put4(off, at, u4v{a.x, a.y, b.x, b.y});
    }
    static __device__ __forceinline__ void clear(const Xch& x, unsigned off, unsigned at) {
        x.put4(off, at, u4v{kResEmptyLo, kResEmptyHi, kResEmptyLo, kResEmptyHi});
    }
    static __device__ __forceinline__ T load(const Xch& x, unsigned off, unsigned at) { return x.get4(off, at); }
    static __device__ __forceinline__ unsigned seen(T w) { return min(xseen(w.y), xseen(w.w)); }
    static __device__ __forceinline__ double2 get(T w) {
        return make_double2(xdouble(u2v{w.x, w.y}), xdouble(u2v{w.z, w.w}));
    }
};
template <>
struct XElem<float2> {
    using T = u2v;
    static constexpr unsigned kBytes = 8;
    static __device__ __forceinline__ void put(const Xch& x, unsigned off, unsigned at, float2 v) {
        x.put2(off, at, u2v{__float_as_uint(v.x), xhigh(__float_as_uint(v.y))});
    }
    static __device__ __forceinline__ void clear(const Xch& x, unsigned off, unsigned at) {
        x.put2(off, at, u2v{kResEmptyLo, kResEmptyHi});
    }
    static __device__ __forceinline__ T load(const Xch& x, unsigned off, unsigned at) { return x.get2(off, at); }
    static __device__ __forceinline__ unsigned seen(T w) { return xseen(w.y); }
    static __device__ __forceinline__ float2 get(T w) {
        return make_float2(__uint_as_float(w.x), __uint_as_float(w.y));
    }
};
__device__ __forceinline__ double2 pick(bool c, double2 a, double2 b) {
    return make_double2(c ? a.x : b.x, c ? a.y : b.y);
}
__device__ __forceinline__ float2 pick(bool c, float2 a, float2 b) {
    return make_float2(c ? a.x : b.x, c ? a.y : b.y);
}

// Called between unsuccessful polls: true when the wait has to be given up.
struct Patience {
    int* aborted;
    u64 limit;  // ticks of the 100 MHz wall clock; 0: no second poll
    u64 t0 = 0;
    int spins = 0;
    __device__ __forceinline__ bool gone() {
        if (++spins % 64 && limit) return false;
        if (__hip_atomic_load(aborted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return true;
        const u64 t = wall_clock64();
        if (spins <= 64) t0 = t;
        if (t - t0 < limit) return false;
        __hip_atomic_store(aborted, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
};

// Block barrier for LDS data alone: published words and flushed shifts stay in
// flight (__syncthreads would wait until they have reached memory).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- lane exchanges: rows are the four groups of 16 lanes of a wave
__device__ __forceinline__ void swap_halves(unsigned& a, unsigned& b) {  // lanes 32-63 of a <-> lanes 0-31 of b
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap_rows(unsigned& a, unsigned& b) {  // rows 1, 3 of a <-> rows 0, 2 of b
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
template <bool HALVES>
__device__ __forceinline__ void exchange(double& a, double& b) {
    unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
    unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
    if (HALVES) {
        swap_halves(al, bl);
        swap_halves(ah, bh);
    } else {
        swap_rows(al, bl);
        swap_rows(ah, bh);
    }
    a = __hiloint2double((int)ah, (int)al);
    b = __hiloint2double((int)bh, (int)bl);
}
template <bool HALVES>
__device__ __forceinline__ void exchange(float& a, float& b) {
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    if (HALVES)
        swap_halves(x, y);
    else
        swap_rows(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
// The sum over the four rows of v[c] for every lane column, left in row c
// (c < 3; row 3 repeats colour 1).
template <class T>
__device__ __forceinline__ T sum_rows3(T v0, T v1, T v2) {
    T u = v1;
    exchange<true>(v0, v2);
    exchange<true>(v1, u);
    T s = v0 + v2, t = v1 + u;
    exchange<false>(s, t);
    return s + t;
}
// The sum over the 16 lanes of a row, in every lane of it.
template <int CTRL>
__device__ __forceinline__ double add_ror(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double add_ror8(double v) { return add_ror<0x128>(v); }
__device__ __forceinline__ float add_ror8(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true));
}
template <int K>
__device__ __forceinline__ void sum_row(double (&v)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = add_ror<0x128>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = add_ror<0x124>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = add_ror<0x122>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = add_ror<0x121>(v[k]);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

struct ResStep {  // scalars of one shift in one step; a frozen shift has {0, 1, 0}
    double as, bs, zn;
};

// Eight waves of 8 sites each: lane 16 mu + 8 b + i does the forward (b = 0) or
// backward hop of direction mu at site i of its wave.  Two waves per SIMD leave
// a lane 256 registers, of which FP64 uses 226: two tiles per CU (128 registers)
// spill 165 of them and then lose to the launch loop (16^4: 23.6 against 23.2 us
// per iteration), and so do the 16 hops per site of the improved operator
// (16^3x8, 12-real links: 21.3 against 19.1 us).  Both hops of a direction in
// one lane, with four waves, take 8.0 us per iteration where this takes 7.0
// (16^3x8, 20 poles).
//
// FP32 leaves the registers of a second block per CU, and with it lattices of up
// to 512 tiles: 128 are enough for the single system of a refinement (SHIFTS
// false: no window, no ring), while the window's code spills 69, outside the
// wait for w.  Mixed solve of 12 poles, one launch per solve against the loops:
// 20^3x8 5.3 against 8.1 ms, 16^3x12 6.7 against 10.2 ms, 16^3x8 4.1 against
// 8.0 ms.  A third block per CU (80 registers, 90 spilled) takes 18.8 us per
// iteration where the loop takes 22 (24^3x6), and 15% more than two on the
// lattices that two hold: not used.  Where one block per CU holds the grid, so
// that its window's code keeps its registers, FP32 trajectories at 16^3x8 take
// 27.9 ms instead of 34.1 (20 steps; FP64 32.5).  WAVES: per SIMD.
template <class Link, bool SHIFTS, int WAVES>
__global__ __launch_bounds__(kResThreads, WAVES) void k_resident(Geom g, Link L, ResidentArgs<typename Link::C> a) {
    using C = typename Link::C;
    using R = typename Link::R;
    using X = XElem<C>;
    constexpr int SB = kResTile, NW = kResThreads / 64;
    __shared__ C ring[SHIFTS ? 2 : 1][SHIFTS ? kLagMax : 1][3 * SB];
    __shared__ C wl[3 * SB], al[3 * SB];
    __shared__ double red[4][4 * NW];
    __shared__ double2* xs[kMaxPoles];
    __shared__ double sh_alpha, sh_beta;
    __shared__ int list[2][kMaxPoles], nlist[2], sh_stop, sh_base_on, sh_bad;
    extern __shared__ double dyn[];
    ResStep* const hist = reinterpret_cast<ResStep*>(dyn);  // [2][lag][n]

    const int tid = threadIdx.x, lane = tid & 63, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = (lane >> 3) & 1;
    const int nb = gridDim.x, vh = g.vh, n = a.n, base = a.base, lag = a.lag;
    const int tile = xcd_tile_slab(blockIdx.x, nb, g, SB);
    const int li = wave * (SB / NW) + (lane & (SB / NW - 1));  // the lane's site in the tile
    const bool ok = tile * SB + li < vh;
    const int cb = ok ? tile * SB + li : vh - 1;   // (lanes past the end repeat the last site, and own nothing)
    const bool elem = row < 3 && ok;               // works on element (colour row, site cb) of both parities
    const bool own = elem && !half;                // ... and is the one that stores it
    const unsigned oi = min(row, 2) * vh + cb;     // element of a half vector
    const unsigned ob = oi * sizeof(double2);      // its byte offset, FP64
    const int oo = row * SB + li;                  // the same in the tile's LDS copies
    MsState* st = a.st;
    Patience pat{&st->aborted, a.wait};

    // exchange area (bytes): two odd vectors, three even ones, and three times
    // the sums of blocks and [copy] of groups, a record of its own cache line
    // each (words of several writers in one line arrive one by one)
    const unsigned plane = X::kBytes * vh, vb = 3 * plane;
    const int ngroups = (nb + 15) / 16, group = blockIdx.x / 16;
    const unsigned xw = 0, xa = 2 * vb, xd = (5 * vb + 127) & ~127u, db = kResRecord * (nb + kResCopies * ngroups);
    const Xch xch(a.xch, xd + 3 * db);
    const bool leader = blockIdx.x % 16 == 0;
    const bool direct = nb <= kResDirect;          // every block reads the block sums itself
    const unsigned ow = row * plane + X::kBytes * cb;  // the own element

    // ---- the links of this lane (signs folded in, backward ones as -U^dag), so
    // that its hop is M v(neighbour), and the neighbours
    C M1[9], M0[9];
    int n1, n0;
    {
        auto load = [&](int par, C(&M)[9], int& nn) {
            int x, y, z, t, f, b;
            bool nf, nbk;
            cb_coords(g, par, cb, x, y, z, t);
            hop_geometry(g, row, x, y, z, t, f, b, nf, nbk);
            C u[9];
            L.load(g, half ? 1 - par : par, row, half ? b : cb, u);
            const R s = (half ? !nbk : nf) ? R(-1) : R(1);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const C m = pick(half, cconj(u[3 * (e % 3) + e / 3]), u[e]);
                M[e] = C{s * m.x, s * m.y};
            }
            nn = half ? b : f;
        };
        load(1, M1, n1);
        load(0, M0, n0);
    }

    // ---- vectors: own element and the even neighbours of the lane's odd site
    double2 o_x = {0.0, 0.0};
    C o_r, o_p, rn[3], pn[3];
    const bool fresh = a.b != nullptr;
    if (fresh) {
        o_r = o_p = from_d2<C>(a.b[oi]);
#pragma unroll
        for (int c = 0; c < 3; ++c) rn[c] = pn[c] = from_d2<C>(a.b[c * vh + n1]);
    } else {
        o_r = a.r[oi];
        o_p = a.p[oi];
        o_x = a.x.template at<double2>(base)[oi];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            rn[c] = a.r[c * vh + n1];
            pn[c] = a.p[c * vh + n1];
        }
    }

    // ---- scalars, in wave 0: lane k holds shift k
    const MsIter& s0 = st->it[0];
    double zeta = 1.0, zeta_old = 1.0, shift = 0.0;
    int active = 0, ipp = 0;
    if (lane < n) {
        zeta = s0.zeta[lane];
        zeta_old = s0.zeta_old[lane];
        shift = st->shift[lane];
        active = s0.active[lane];
        ipp = s0.iters_per_pole[lane];
    }
    double alpha_old = s0.alpha_old, beta_old = s0.beta_old, bb = s0.bb, rr = 0.0;
    int iter = s0.iter, act = active, nonfinite = 0;
    const bool bb_given = st->bb_given || iter > 0;
    if (tid == 0) sh_bad = 0;
    if (tid < n) xs[tid] = a.x.template at<double2>(tid);
    C* const ps = a.ps.template at<C>(0);  // p_s: n vectors one after the other
    bool bad = false;

    // ---- window flush: groups of G shifts of a finished window, GL for each of
    // the two lanes of an element
    constexpr int G = kFlushGroup, GL = G / 2;
    int buf = 0, pend = 0;  // the window being filled, its steps so far
    bool first = fresh;     // the filling window is the solve's first
    int todo = 0, per = 0;  // groups left of the finished window, groups per iteration
    bool todo_first = false;
    double2 pk[GL], xk[GL];
    auto shifts_of = [&](int wb) { return __builtin_amdgcn_readfirstlane(nlist[wb]); };
    auto flush_entry = [&](int g0, int j) { return g0 + 2 * j + half; };
    auto flush_load = [&](int wb, bool start, int g0) {
        const int last = shifts_of(wb) - 1;
#pragma unroll
        for (int j = 0; j < GL; ++j) {
            const int q = list[wb][min(flush_entry(g0, j), last)];
            if (start) {
                pk[j] = to_d2(from_d2<C>(a.b[oi]));
                xk[j] = make_double2(0.0, 0.0);
            } else {
                pk[j] = to_d2(ps[(unsigned)q * 3u * vh + oi]);
                xk[j] = *(double2*)((char*)xs[q] + ob);
            }
        }
    };
    auto flush_apply = [&](int wb, int steps, int g0) {
        const int count = shifts_of(wb);
        int q[GL];
#pragma unroll
        for (int j = 0; j < GL; ++j) q[j] = list[wb][min(flush_entry(g0, j), count - 1)];
        const ResStep* h = hist + wb * lag * n;
        const C* rw = &ring[wb][0][oo];
#pragma unroll 2
        for (int t = 0; t < steps; ++t, h += n, rw += 3 * SB) {
            const double2 r = to_d2(*rw);
#pragma unroll
            for (int j = 0; j < GL; ++j) {
                const ResStep s = h[q[j]];
                xk[j] = make_double2(xk[j].x + s.as * pk[j].x, xk[j].y + s.as * pk[j].y);
                pk[j] = to_d2(from_d2<C>(make_double2(s.zn * r.x + s.bs * pk[j].x, s.zn * r.y + s.bs * pk[j].y)));
            }
        }
#pragma unroll
        for (int j = 0; j < GL; ++j)
            if (flush_entry(g0, j) < count) {
                *(double2*)((char*)xs[q[j]] + ob) = xk[j];
                ps[(unsigned)q[j] * 3u * vh + oi] = from_d2<C>(pk[j]);
            }
    };

    // the hop of this lane, added over the site's lanes: colour `row` of site cb
    auto hops = [&](const C(&M)[9], const C(&v)[3]) {
        C d[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            d[r] = cmul(M[3 * r], v[0]);
            d[r] = cadd(d[r], cmul(M[3 * r + 1], v[1]));
            d[r] = cadd(d[r], cmul(M[3 * r + 2], v[2]));
        }
        return C{add_ror8(sum_rows3(d[0].x, d[1].x, d[2].x)), add_ror8(sum_rows3(d[0].y, d[1].y, d[2].y))};
    };
    // A neighbour's three colours of a published vector; one of this tile comes
    // from its LDS copy `mine`.
    typename X::T qv[3];
    auto remote = [&](int nn) { return (unsigned)(nn - tile * SB) >= (unsigned)SB; };
    auto ask = [&](unsigned at, int nn) {
        asm volatile("" ::: "memory");  // (a load of its own each time)
        if (remote(nn))
#pragma unroll
            for (int c = 0; c < 3; ++c) qv[c] = X::load(xch, X::kBytes * nn, at + c * plane);
    };
    auto finish = [&](unsigned at, int nn, const C* mine, C(&out)[3]) {
        for (;;) {
            const unsigned m = min(min(X::seen(qv[0]), X::seen(qv[1])), X::seen(qv[2]));
            if (!__any(remote(nn) && m == 0)) break;
            if (pat.gone()) {
                bad = true;
                break;
            }
            ask(at, nn);
        }
        pat.spins = 0;
        const int ln = (nn - tile * SB) & (SB - 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) out[c] = pick(remote(nn), X::get(qv[c]), mine[c * SB + ln]);
    };
    // By one wave: the sums over `count` records, 32 at a time; lanes 4 i + k
    // receive sum k.
    auto add_up = [&](unsigned at, int count) {
        double t = 0.0;
        for (int i0 = 0; i0 < count; i0 += 32) {
            const int i = i0 + (lane >> 2);
            const unsigned o0 = kResRecord * min(i, count - 1) + 8 * (lane & 3);
            const unsigned o1 = kResRecord * min(i + 16, count - 1) + 8 * (lane & 3);
            u2v q0, q1;
            for (;;) {
                asm volatile("" ::: "memory");
                q0 = xch.get2(o0, at);
                q1 = xch.get2(o1, at);
                if (!__any(min(xseen(q0.y), xseen(q1.y)) == 0)) break;
                if (pat.gone()) {
                    bad = true;
                    break;
                }
            }
            pat.spins = 0;
            t += i < count ? xdouble(q0) : 0.0;
            t += i + 16 < count ? xdouble(q1) : 0.0;
        }
        t = add_ror8(t);
        t = add_ror<0x124>(t);
        double u = t;
        exchange<true>(t, u);
        t += u;
        u = t;
        exchange<false>(t, u);
        return t + u;
    };

    int stop = 0;
    double alpha = 0.0, beta = 0.0;
    for (int step = 0;; ++step) {
        // (the group of shifts applied below: its loads run beside the hops)
        const bool one = SHIFTS && todo > 0 && elem;
        if (one) flush_load(buf ^ 1, todo_first, (todo - 1) * G);
        // ---- w = D_oe p
        const unsigned wv = xw + (step & 1) * vb;
        const C w = hops(M1, pn);
        if (own) {
            X::put(xch, ow, wv, w);
            wl[oo] = w;
        }
        // ---- the shifted scalars of the step taken above
        if (step > 0) {
            if (wave == 0) {
                double zn = zeta, as = 0.0, bs = 1.0, zr = 0.0;
                if (lane == base) {
                    zn = 1.0;
                } else if (active) {
                    zn = zeta * zeta_old * alpha_old /
                         (alpha * beta_old * (zeta_old - zeta) + zeta_old * alpha_old * (1.0 + shift * alpha));
                    const double q = zn / zeta;
                    as = alpha * q;
                    bs = beta * q * q;
                    zr = zn;
                }
                if (SHIFTS && lane < n) hist[(buf * lag + pend) * n + lane] = ResStep{as, bs, zr};
                if (SHIFTS && pend == 0) {
                    const int mine = lane < n && lane != base && (active || first);
                    const u64 m = __ballot(mine != 0);
                    if (mine) list[buf][__popcll(m & ((1ull << lane) - 1ull))] = lane;
                    if (lane == 0) nlist[buf] = __popcll(m);
                }
                zeta_old = zeta;
                zeta = zn;
                alpha_old = alpha;
                beta_old = beta;
            }
            if (SHIFTS) ++pend;
        }
        lds_barrier();
        ask(wv, n0);
        // words that every block has consumed (see Reuse)
        if (own) {
            X::clear(xch, ow, xw + ((step + 1) & 1) * vb);
            X::clear(xch, ow, xa + ((step + 1) % 3) * vb);
        }
        if (wave == 0) {
            const unsigned d = xd + ((step + 1) % 3) * db;
            const u2v empty = {kResEmptyLo, kResEmptyHi};
            if (lane < 4) xch.put2(8 * lane, d + kResRecord * blockIdx.x, empty);
            if (leader && lane < 4 * kResCopies)
                xch.put2(kResRecord * (lane >> 2) * ngroups + 8 * (lane & 3), d + kResRecord * (nb + group), empty);
        }
        if (one) flush_apply(buf ^ 1, lag, (todo - 1) * G);
        if (todo > 0) --todo;
        for (int k = 1; SHIFTS && k < per && todo > 0; ++k, --todo)
            if (elem) {
                flush_load(buf ^ 1, todo_first, (todo - 1) * G);
                flush_apply(buf ^ 1, lag, (todo - 1) * G);
            }
        if (SHIFTS && pend == lag) {  // a window is full; the one before it is done (lag iterations, per groups each)
            todo = (shifts_of(buf) + G - 1) / G;
            per = (todo + lag - 1) / lag;
            todo_first = first;
            first = false;
            buf ^= 1;
            pend = 0;
        }
        // ---- Ap = mt p - D_eo w
        C v[3];
        finish(wv, n0, wl, v);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the emptied words have arrived
        const C u = hops(M0, v);
        const unsigned av = xa + (step % 3) * vb;
        const R m = (R)a.mt;
        const C o_a = C{m * o_p.x - u.x, m * o_p.y - u.y};
        double d[4] = {0.0, 0.0, 0.0, 0.0};
        if (own) {
            X::put(xch, ow, av, o_a);
            al[oo] = o_a;
            const double2 rd = to_d2(o_r), pd = to_d2(o_p), ad = to_d2(o_a);
            d[0] = rd.x * rd.x + rd.y * rd.y;
            d[1] = pd.x * ad.x + pd.y * ad.y;
            d[2] = rd.x * ad.x + rd.y * ad.y;
            d[3] = ad.x * ad.x + ad.y * ad.y;
        }
        sum_row<4>(d);
        if ((lane & 15) == 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) red[k][wave * 4 + row] = d[k];
        lds_barrier();
        // ---- the sums of all blocks, and the neighbours' Ap.  Wave 0 publishes
        // the block's sums, adds up the groups' (on small grids the blocks') and
        // takes the step's decisions; wave 1 of a group's first block adds up
        // and publishes the group's.
        const unsigned l1 = xd + (step % 3) * db, l2 = l1 + kResRecord * nb;
        if (wave == 0) {
            double s[1] = {red[row][lane & 15] + red[row][16 + (lane & 15)]};
            sum_row<1>(s);
            if ((lane & 15) == 0) xch.put2(8 * row, l1 + kResRecord * blockIdx.x, xword(s[0]));
        }
        ask(av, n1);
        if (wave == 1 && leader && !direct) {
            const double s = add_up(l1 + kResRecord * 16 * group, min(16, nb - 16 * group));
            if (lane < 4 * kResCopies)
                xch.put2(kResRecord * (lane >> 2) * ngroups + 8 * (lane & 3), l2 + kResRecord * group, xword(s));
        }
        if (wave == 0) {
            const double s = direct ? add_up(l1, nb)
                                    : add_up(l2 + kResRecord * (blockIdx.x % kResCopies) * ngroups, ngroups);
            // alpha, beta and the stop (the rules of the launch loops)
            rr = lane_value(s, 0);
            const double pAp = lane_value(s, 1), rAp = lane_value(s, 2), ApAp = lane_value(s, 3);
            if (!bb_given && step == 0) bb = rr;
            nonfinite = !isfinite(rr);
            alpha = beta = 0.0;
            if (!nonfinite) {
                const double inv = 1.0 / rr;  // beside the division below, not after it
                alpha = rr / pAp;
                double rr1 = rr - 2.0 * alpha * rAp + alpha * alpha * ApAp;
                if (rr1 < 0.0) rr1 = 0.0;
                beta = rr1 * inv;
            }
            act = active && !(zeta * zeta * rr <= st->tol2 * bb);
            const u64 any = __ballot(act != 0);
            if (any && !(isfinite(alpha) && isfinite(beta))) nonfinite = 1;
            const int halt = nonfinite || !any || iter >= st->maxiter;
            if (lane == 0) {
                sh_alpha = alpha;
                sh_beta = beta;
                sh_stop = halt;
                sh_base_on = (int)(any >> base) & 1;
            }
        }
        finish(av, n1, al, v);
        if (bad) sh_bad = 1;
        lds_barrier();
        if (sh_bad) return;
        stop = __builtin_amdgcn_readfirstlane(sh_stop);
        if (stop) break;
        alpha = sh_alpha;
        beta = sh_beta;
        ipp = act ? iter + 1 : (active ? iter : ipp);
        active = act;
        ++iter;
        // ---- r, p at the neighbours and at the own site
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            rn[c] = cg_r_next(rn[c], v[c], alpha);
            pn[c] = cg_p_next(rn[c], pn[c], beta);
        }
        const double2 pd = to_d2(o_p);
        if (sh_base_on) o_x = make_double2(fma(alpha, pd.x, o_x.x), fma(alpha, pd.y, o_x.y));
        o_r = cg_r_next(o_r, o_a, alpha);
        o_p = cg_p_next(o_r, o_p, beta);
        if (SHIFTS && own) ring[buf][pend][oo] = o_r;
        if (step + 1 == a.max_steps) break;
    }
    // ---- the rest of the finished window, the steps of the last one, the results
    lds_barrier();  // (the ring, for the other lane of an element)
    if (SHIFTS && elem) {
        for (; todo > 0; --todo) {
            flush_load(buf ^ 1, todo_first, (todo - 1) * G);
            flush_apply(buf ^ 1, lag, (todo - 1) * G);
        }
        if (pend > 0)
            for (int g0 = 0; g0 < shifts_of(buf); g0 += G) {
                flush_load(buf, first, g0);
                flush_apply(buf, pend, g0);
            }
    }
    if (own) {
        if (SHIFTS && first && pend == 0)  // stopped before the first step
            for (int k = 0; k < n; ++k) xs[k][oi] = make_double2(0.0, 0.0);
        xs[base][oi] = o_x;
        if (!fresh) {
            a.r[oi] = o_r;
            a.p[oi] = o_p;
        }
    }
    if (blockIdx.x == 0 && wave == 0) {
        MsIter& o = stop ? st->fin : st->it[0];
        if (lane < n) {
            o.active[lane] = act;
            o.iters_per_pole[lane] = stop && active ? iter : ipp;
            o.zeta[lane] = zeta;
            o.zeta_old[lane] = zeta_old;
        }
        if (lane == 0) {
            o.alpha_old = stop ? alpha_old : alpha;
            o.beta_old = stop ? beta_old : beta;
            o.bb = bb;
            o.rr = rr;
            o.iter = iter;
            o.nonfinite = nonfinite;
            if (stop) st->done[0] = st->done[1] = 1;
        }
    }
}

__global__ void k_fill_empty(u4v* __restrict__ p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = u4v{kResEmptyLo, kResEmptyHi, kResEmptyLo, kResEmptyHi};
}

// Blocks of this kernel that the current device holds at once, asked until the
// device has answered; 0 where it does not say.
constexpr size_t kResHistMax = (size_t)2 * kLagMax * kMaxPoles * sizeof(ResStep);
constexpr int kResDevices = 64;
template <class Link, bool SHIFTS, int WAVES>
int capacity() {
    static std::atomic<int> known[kResDevices];  // capacity + 1
    int dev = -1, blocks = 0, cus = 0, coop = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kResDevices) return 0;
    const int k = known[dev].load(std::memory_order_relaxed);
    if (k) return k - 1;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, (const void*)k_resident<Link, SHIFTS, WAVES>,
                                                     kResThreads, SHIFTS ? kResHistMax : 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;  // (asked again by the next solve)
    }
    known[dev].store(blocks * cus + 1, std::memory_order_relaxed);
    return blocks * cus;
}

// fn(link accessor) for the storage format of the operator
template <class Fn>
void with_link(const LinkSet& ls, double2, Fn fn) {
    if (ls.fmt64 == STAG_LINKS_F64_12)
        fn(LinkD12{ls.d12});
    else
        fn(LinkD18{ls.d18});
}
template <class Fn>
void with_link(const LinkSet& ls, float2, Fn fn) {
    if (ls.fmt32 == STAG_LINKS_F16_12)
        fn(LinkH12{(const __half2*)ls.h12});
    else
        fn(LinkS18{ls.s18});
}

// Single systems that continue from given vectors (b = NULL) in FP32 have a
// kernel of their own; others take the general one.
template <class V>
bool single(const ResidentArgs<V>& a) {
    return sizeof(V) == sizeof(float2) && a.n == 1 && !a.b;
}
// The kernel for nb blocks, NULL where they do not fit: two waves per SIMD, or
// four (a second block per CU) for FP32 where two do not hold the grid.  The
// single system has the registers for four anyway.
template <class Link, bool SHIFTS>
const void* kernel_for(int nb) {
    constexpr bool fp32 = sizeof(typename Link::C) == sizeof(float2);
    if (nb > kResMax) return nullptr;
    if constexpr (SHIFTS || !fp32)
        if (nb <= capacity<Link, SHIFTS, 2>()) return (const void*)k_resident<Link, SHIFTS, 2>;
    if constexpr (fp32)
        if (nb <= capacity<Link, SHIFTS, 4>()) return (const void*)k_resident<Link, SHIFTS, 4>;
    return nullptr;
}
template <bool SHIFTS, class V>
bool fits(const Geom& g, const LinkSet& ls) {
    bool ok = false;
    with_link(ls, V{}, [&](auto L) { ok = kernel_for<decltype(L), SHIFTS>(resident_blocks(g)) != nullptr; });
    return ok;
}

}  // namespace

bool resident_fits(const Geom& g, const LinkSet& ls, bool fp64, bool refine) {
    if (ls.naik) return false;
    if (refine) return fits<false, float2>(g, ls);
    return fp64 ? fits<true, double2>(g, ls) : fits<true, float2>(g, ls);
}

template <class V>
hipError_t launch_resident(const Geom& g, const LinkSet& ls, const ResidentArgs<V>& a, hipStream_t s) {
    const size_t n = resident_bytes(g) / 16;
    k_fill_empty<<<(int)std::min<size_t>((n + 255) / 256, 2048), 256, 0, s>>>((u4v*)a.xch, n);
    hipError_t err = hipErrorInvalidValue;
    with_link(ls, V{}, [&](auto L) {
        Geom gg = g;
        ResidentArgs<V> aa = a;
        void* args[] = {&gg, &L, &aa};
        const void* kernel = kernel_for<decltype(L), true>(resident_blocks(g));
        size_t dyn = (size_t)2 * a.lag * a.n * sizeof(ResStep);
        if constexpr (sizeof(V) == sizeof(float2))
            if (single(a)) {
                kernel = kernel_for<decltype(L), false>(resident_blocks(g));
                dyn = 0;
            }
        if (!kernel) return;
        err = hipLaunchCooperativeKernel(kernel, dim3(resident_blocks(g)), dim3(kResThreads), args, dyn, s);
    });
    return err;
}
template hipError_t launch_resident<double2>(const Geom&, const LinkSet&, const ResidentArgs<double2>&, hipStream_t);
template hipError_t launch_resident<float2>(const Geom&, const LinkSet&, const ResidentArgs<float2>&, hipStream_t);

}  // namespace stag
