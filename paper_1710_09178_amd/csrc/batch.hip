// Batched multi-shift CG kernels: every launch covers all tiles of all
// lattices of the batch, and each Dslash thread applies the links it loads to
// every right-hand side of its lattice (links read once per nrhs vectors).
// Scalars are per system (lattice, right-hand side); reductions are per tile
// and are summed over the lattice's tiles by the consuming kernel.
#include <type_traits>

#include "batch.h"

namespace stag {

namespace {

template <class V>
struct BPrec;
template <>
struct BPrec<double2> {
    using R = double;
};
template <>
struct BPrec<float2> {
    using R = float;
};

// a link entry; NT: non-temporal (link fields larger than the Infinity Cache)
template <bool NT>
__device__ __forceinline__ double2 bload(const double2* p) {
    if constexpr (NT) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        const d2v t = __builtin_nontemporal_load((const d2v*)p);
        return make_double2(t.x, t.y);
    } else {
        return *p;
    }
}
template <bool NT>
__device__ __forceinline__ float2 bload(const float2* p) {
    if constexpr (NT) {
        typedef float f2v __attribute__((ext_vector_type(2)));
        const f2v t = __builtin_nontemporal_load((const f2v*)p);
        return make_float2(t.x, t.y);
    } else {
        return *p;
    }
}

// An SU(3) matrix's row 2 from rows 0 and 1: conj(row 0 x row 1).  With it
// the operators read 12 of a link's 18 reals (rows 0-1; the storage keeps
// all 9 entries as separate planes, so row 2's planes are simply not read).
template <class V>
__device__ __forceinline__ void brebuild_row2(V (&m)[9]) {
    m[6] = cconj(csub(cmul(m[1], m[5]), cmul(m[2], m[4])));
    m[7] = cconj(csub(cmul(m[2], m[3]), cmul(m[0], m[5])));
    m[8] = cconj(csub(cmul(m[0], m[4]), cmul(m[1], m[3])));
}

__device__ __forceinline__ void bhop_geometry(const Geom& g, int mu, int x, int y, int z, int t, int& cbf, int& cbb,
                                              bool& nf, bool& nb) {
    if (mu == 0) {
        cbf = cb_index(g, (x + 1 == g.nx) ? 0 : x + 1, y, z, t);
        cbb = cb_index(g, (x == 0) ? g.nx - 1 : x - 1, y, z, t);
        nf = nb = false;
    } else if (mu == 1) {
        cbf = cb_index(g, x, (y + 1 == g.ny) ? 0 : y + 1, z, t);
        cbb = cb_index(g, x, (y == 0) ? g.ny - 1 : y - 1, z, t);
        nf = nb = (x & 1);
    } else if (mu == 2) {
        cbf = cb_index(g, x, y, (z + 1 == g.nz) ? 0 : z + 1, t);
        cbb = cb_index(g, x, y, (z == 0) ? g.nz - 1 : z - 1, t);
        nf = nb = ((x + y) & 1);
    } else {
        cbf = cb_index(g, x, y, z, (t + 1 == g.nt) ? 0 : t + 1);
        cbb = cb_index(g, x, y, z, (t == 0) ? g.nt - 1 : t - 1);
        const bool eta = ((x + y + z) & 1);
        nf = eta ^ (t == g.nt - 1);
        nb = eta ^ (t == 0);
    }
}

// Epilogues of the operator, one call per entry (right-hand side rh, colour,
// site) at index i of a batched vector; K sums per right-hand side go to
// part[tile][kMaxRhs][K].
template <class V>
struct BEpiStore {
    static constexpr int K = 0;
    double* part;  // (unused)
    V* out;
    __device__ __forceinline__ void item(const BInst&, int, size_t i, V v, double*) const { out[i] = v; }
};

// Ap = (4 m_i^2 + sigma_0) p - v and per-rhs partials of <p,Ap>, <r,Ap>, <Ap,Ap>
template <class V>
struct BEpiCG {
    static constexpr int K = 3;
    double* part;
    V* Ap;
    const V* p;
    const V* r;
    const double* sigma0_term;  // [inst] 4 m_i^2 + sigma_0
    __device__ __forceinline__ void item(const BInst&, int inst, size_t i, V v, double* acc) const {
        const V pv = p[i], rv = r[i];
        using Rl = typename BPrec<V>::R;
        const Rl m = (Rl)sigma0_term[inst];
        const V a = V{m * pv.x - v.x, m * pv.y - v.y};
        Ap[i] = a;
        const double2 pd = to_d2(pv), rd = to_d2(rv), ad = to_d2(a);
        acc[0] += pd.x * ad.x + pd.y * ad.y;
        acc[1] += rd.x * ad.x + rd.y * ad.y;
        acc[2] += ad.x * ad.x + ad.y * ad.y;
    }
};

// r = b - (A_i + pole) x with per-rhs |r|^2 partials; r stored when rout != null
struct BEpiResid {
    static constexpr int K = 1;
    double* part;
    const double2* x;
    const double2* b;
    double2* rout;
    double pole;
    __device__ __forceinline__ void item(const BInst& I, int, size_t i, double2 v, double* acc) const {
        const double coef = I.four_m2 + pole;
        const double2 xv = x[i], bv = b[i];
        const double rx = bv.x - (coef * xv.x - v.x), ry = bv.y - (coef * xv.y - v.y);
        if (rout) rout[i] = make_double2(rx, ry);
        acc[0] += rx * rx + ry * ry;
    }
};

// Sums of a block whose threads take entries of any right-hand side.
template <class Epi>
struct BlockSums {
    static constexpr int N = Epi::K * kMaxRhs;
    double acc[N > 0 ? N : 1];
    __device__ __forceinline__ BlockSums() {
#pragma unroll
        for (int k = 0; k < N; ++k) acc[k] = 0.0;
    }
    template <class V>
    __device__ __forceinline__ void item(const Epi& epi, const BInst& I, int inst, int rh, size_t i, V v) {
        double d[Epi::K + 1] = {};
        epi.item(I, inst, i, v, d);
#pragma unroll
        for (int q = 0; q < kMaxRhs; ++q)  // selects: no dynamic register indexing
#pragma unroll
            for (int k = 0; k < Epi::K; ++k) acc[q * Epi::K + k] += (q == rh) ? d[k] : 0.0;
    }
    __device__ __forceinline__ void finish(const Epi& epi, int tile) {
        if constexpr (N > 0) {
            __shared__ double lds[4 * N];
            block_sum<N>(acc, lds);
            if (threadIdx.x == 0)
#pragma unroll
                for (int k = 0; k < N; ++k) epi.part[(size_t)tile * N + k] = acc[k];
        }
    }
};

// One block per tile: TPS threads per site split the 4 directions; every
// thread applies its links to all right-hand sides of the lattice.  At 9 lattices
// of 70,848 sites together and 4 right-hand sides the four-thread form cannot
// do without 109 MB (storing) and 136 MB (CG epilogue) and misses the L2 for 155
// and 184 MB, at 6 TB/s: 24 and 27 us (26 and 33 us before the tiles
// of a lattice were put in neighbour order and the waves finished a right-hand
// side each).  156 registers: three waves per SIMD; a fourth (128 registers, 12
// spilled) gains nothing.
template <int TPS, class V, class Epi, bool NT, bool L12>
__global__ __launch_bounds__(kBlock, TPS == 4 ? 3 : 2) void k_bdslash(BatchDev bd, const V* __restrict__ links, const V* __restrict__ in,
                                                    int out_par, Epi epi, const int* __restrict__ inst_done) {
    constexpr int SB = kBlock / TPS;
    constexpr int DPT = 4 / TPS;
    using Rl = typename BPrec<V>::R;
    const int ti = out_par ? (int)blockIdx.x : turned(blockIdx.x, gridDim.x);
    const BTile tl = bd.tiles[ti];
    if (inst_done && inst_done[tl.inst]) return;
    const BInst I = bd.inst[tl.inst];
    const Geom& g = I.g;
    const int R = bd.nrhs;
    constexpr bool kWaveRhs = TPS == 4;  // wave r of four finishes right-hand side r
    __shared__ V part[(kWaveRhs ? (TPS - 1) : TPS) * kMaxRhs * 3 * SB];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slice = wave % TPS, sgrp = wave / TPS;
    const int j = sgrp * 64 + lane;
    const int cb = tl.cb0 + j;
    V acc[kMaxRhs][3];
#pragma unroll
    for (int r = 0; r < kMaxRhs; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[r][c] = V{0, 0};
    const V* lk = links + blink_base(I);
    if (cb < g.vh) {
        int x, y, z, t;
        cb_coords(g, out_par, cb, x, y, z, t);
#pragma unroll
        for (int d = 0; d < DPT; ++d) {
            const int mu = slice * DPT + d;
            int cbf, cbb;
            bool nf, nb;
            bhop_geometry(g, mu, x, y, z, t, cbf, cbb, nf, nb);
            const V* uf = lk + link_off(g, out_par, mu, 0) + cb;
            const V* ub = lk + link_off(g, 1 - out_par, mu, 0) + cbb;
            constexpr int NE = L12 ? 6 : 9;
            // one matrix at a time, for its registers
            {
                V U[9];
#pragma unroll
                for (int e = 0; e < NE; ++e) U[e] = bload<NT>(uf + (size_t)e * g.vh);
                if constexpr (L12) brebuild_row2(U);
                const Rl sf = nf ? Rl(-1) : Rl(1);
#pragma unroll
                for (int r = 0; r < kMaxRhs; ++r) {
                    if (r >= R) break;
                    V pf[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) pf[c] = in[bvec_off(I, R, r, c) + cbf];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        V f = cmul(U[3 * a], pf[0]);
                        f = cadd(f, cmul(U[3 * a + 1], pf[1]));
                        f = cadd(f, cmul(U[3 * a + 2], pf[2]));
                        acc[r][a].x += sf * f.x;
                        acc[r][a].y += sf * f.y;
                    }
                }
            }
            {
                V W[9];
#pragma unroll
                for (int e = 0; e < NE; ++e) W[e] = bload<NT>(ub + (size_t)e * g.vh);
                if constexpr (L12) brebuild_row2(W);
                const Rl sb = nb ? Rl(-1) : Rl(1);
#pragma unroll
                for (int r = 0; r < kMaxRhs; ++r) {
                    if (r >= R) break;
                    V pb[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) pb[c] = in[bvec_off(I, R, r, c) + cbb];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        V bb = cmulc(W[a], pb[0]);
                        bb = cadd(bb, cmulc(W[3 + a], pb[1]));
                        bb = cadd(bb, cmulc(W[6 + a], pb[2]));
                        acc[r][a].x -= sb * bb.x;
                        acc[r][a].y -= sb * bb.y;
                    }
                }
            }
        }
    }
    if constexpr (kWaveRhs) {
        // The wave of right-hand side r keeps its own slice of it and adds the
        // other three: a quarter less LDS (36.9 KB), and its sums need no
        // other wave.
        static_assert(kMaxRhs == 4, "one wave per right-hand side");
#pragma unroll
        for (int r = 0; r < kMaxRhs; ++r)
            if (r != slice && r < R)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    part[((r * 3 + (slice < r ? slice : slice - 1)) * 3 + c) * SB + lane] = acc[r][c];
        __syncthreads();
        if (slice >= R) return;
        double racc[Epi::K + 1] = {};
        if (cb < g.vh) {
            V own[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                own[c] = acc[0][c];
#pragma unroll
                for (int r = 1; r < kMaxRhs; ++r)
                    if (slice == r) own[c] = acc[r][c];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                V v = own[c];
                V o[3];
#pragma unroll
                for (int s = 0; s < 3; ++s) o[s] = part[((slice * 3 + s) * 3 + c) * SB + lane];
                // slices in order
                const V a0 = slice == 0 ? v : o[0];
                const V a1 = slice == 0 ? o[0] : slice == 1 ? v : o[1];
                const V a2 = slice <= 1 ? o[1] : slice == 2 ? v : o[2];
                const V a3 = slice == 3 ? v : o[2];
                v = cadd(cadd(cadd(a0, a1), a2), a3);
                epi.item(I, tl.inst, bvec_off(I, R, slice, c) + cb, v, racc);
            }
        }
        if constexpr (Epi::K > 0) {
            double v[Epi::K];
#pragma unroll
            for (int k = 0; k < Epi::K; ++k) v[k] = racc[k];
            wave_sum<Epi::K>(v);
            if (lane == 0)
#pragma unroll
                for (int k = 0; k < Epi::K; ++k)
                    epi.part[((size_t)ti * kMaxRhs + slice) * Epi::K + k] = v[k];
        }
    } else {
#pragma unroll
        for (int r = 0; r < kMaxRhs; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                if (r < R) part[((slice * kMaxRhs + r) * 3 + c) * SB + j] = acc[r][c];
        __syncthreads();
        BlockSums<Epi> sums;
        for (int it = threadIdx.x; it < R * 3 * SB; it += kBlock) {
            const int plane = it / SB, rh = plane / 3, c = plane % 3, jj = it % SB;
            const int site = tl.cb0 + jj;
            if (site >= g.vh) continue;
            V v = part[((0 * kMaxRhs + rh) * 3 + c) * SB + jj];
#pragma unroll
            for (int s = 1; s < TPS; ++s) v = cadd(v, part[((s * kMaxRhs + rh) * 3 + c) * SB + jj]);
            sums.item(epi, I, tl.inst, rh, bvec_off(I, R, rh, c) + site, v);
        }
        sums.finish(epi, ti);
    }
}

// Eight lanes per output site, one hop each: lane h takes direction h / 2,
// the forward hop U_mu(x) p(x+mu) for even h and the backward hop
// U_mu(x-mu)^dag p(x-mu) for odd h (its matrix is loaded transposed and
// conjugated, so both kinds run the same arithmetic).  Each lane holds one
// link matrix, the eight partial colour vectors of a site meet by lane
// exchanges (no LDS), and every right-hand side is finished right after its
// exchange: its three (rhs, colour) outputs go to lanes (3 rhs + colour) mod 8.
template <class V, class Epi>
__global__ __launch_bounds__(kBlock) void k_bdslash8(BatchDev bd, const V* __restrict__ links,
                                                     const V* __restrict__ in, int out_par, Epi epi,
                                                     const int* __restrict__ inst_done) {
    using Rl = typename BPrec<V>::R;
    const int ti = out_par ? (int)blockIdx.x : turned(blockIdx.x, gridDim.x);
    const BTile tl = bd.tiles[ti];
    if (inst_done && inst_done[tl.inst]) return;
    const BInst I = bd.inst[tl.inst];
    const Geom& g = I.g;
    const int R = bd.nrhs;
    const int h = threadIdx.x & 7, mu = h >> 1;
    const bool bwd = h & 1;
    const int cb = tl.cb0 + (int)(threadIdx.x >> 3);
    const bool on = cb < g.vh;
    V U[9];
    int nbr = 0;
    Rl sg = 0;
    if (on) {
        int x, y, z, t;
        cb_coords(g, out_par, cb, x, y, z, t);
        int cbf, cbb;
        bool nf, nb;
        bhop_geometry(g, mu, x, y, z, t, cbf, cbb, nf, nb);
        const V* lk = links + blink_base(I);
        const V* u = bwd ? lk + link_off(g, 1 - out_par, mu, 0) + cbb : lk + link_off(g, out_par, mu, 0) + cb;
        const Rl cj = bwd ? Rl(-1) : Rl(1);
        V M[9];
        if (bd.link12) {
#pragma unroll
            for (int e = 0; e < 6; ++e) M[e] = u[(size_t)e * g.vh];
            brebuild_row2(M);
        } else {
#pragma unroll
            for (int e = 0; e < 9; ++e) M[e] = u[(size_t)e * g.vh];
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const int src = bwd ? 3 * (e % 3) + e / 3 : e;
            U[e] = V{M[src].x, cj * M[src].y};
        }
        nbr = bwd ? cbb : cbf;
        sg = bwd ? (nb ? Rl(1) : Rl(-1)) : (nf ? Rl(-1) : Rl(1));
    } else {
#pragma unroll
        for (int e = 0; e < 9; ++e) U[e] = V{0, 0};
    }
    BlockSums<Epi> sums;
#pragma unroll
    for (int r = 0; r < kMaxRhs; ++r) {
        if (r >= R) break;
        V pv[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) pv[c] = on ? in[bvec_off(I, R, r, c) + nbr] : V{0, 0};
        V a[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            V f = cmul(U[3 * c], pv[0]);
            f = cadd(f, cmul(U[3 * c + 1], pv[1]));
            f = cadd(f, cmul(U[3 * c + 2], pv[2]));
            a[c] = V{sg * f.x, sg * f.y};
        }
#pragma unroll
        for (int m = 1; m < 8; m <<= 1)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                a[c].x += __shfl_xor(a[c].x, m, 64);
                a[c].y += __shfl_xor(a[c].y, m, 64);
            }
        if (on)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                if ((3 * r + c) % 8 == h) sums.item(epi, I, tl.inst, r, bvec_off(I, R, r, c) + cb, a[c]);
    }
    sums.finish(epi, ti);
}

template <class V, class Epi>
void bdslash_tps(const BatchDev& bd, int tps, const V* links, const V* in, int out_par, const Epi& epi,
                 const int* inst_done, hipStream_t s) {
    if (tps == 8) {
        k_bdslash8<V, Epi><<<bd.ntiles, kBlock, 0, s>>>(bd, links, in, out_par, epi, inst_done);
        return;
    }
    auto go = [&](auto nt, auto l12) {
        constexpr bool NT = decltype(nt)::value, L12 = decltype(l12)::value;
        switch (tps) {
            case 1:
                k_bdslash<1, V, Epi, NT, L12><<<bd.ntiles, kBlock, 0, s>>>(bd, links, in, out_par, epi, inst_done);
                break;
            case 2:
                k_bdslash<2, V, Epi, NT, L12><<<bd.ntiles, kBlock, 0, s>>>(bd, links, in, out_par, epi, inst_done);
                break;
            default:
                k_bdslash<4, V, Epi, NT, L12><<<bd.ntiles, kBlock, 0, s>>>(bd, links, in, out_par, epi, inst_done);
                break;
        }
    };
    if (bd.link_nt) {
        if (bd.link12)
            go(std::true_type{}, std::true_type{});
        else
            go(std::true_type{}, std::false_type{});
    } else {
        if (bd.link12)
            go(std::false_type{}, std::true_type{});
        else
            go(std::false_type{}, std::false_type{});
    }
}

// r = p = p_k = b, x_k = 0, per-rhs partials of |b|^2
template <class V>
__global__ __launch_bounds__(kBlock) void k_bms_init(BatchDev bd, const double2* __restrict__ b, V* __restrict__ r,
                                                     V* __restrict__ p, VecPtrs x, VecPtrs ps,
                                                     BState st, double* __restrict__ qout) {
    const BTile tl = bd.tiles[blockIdx.x];
    const BInst I = bd.inst[tl.inst];
    const int R = bd.nrhs, SB = bd.tile_sites;
    const int n = st.n, base = st.base;
    double acc[kMaxRhs] = {0.0, 0.0, 0.0, 0.0};
    for (int it = threadIdx.x; it < R * 3 * SB; it += kBlock) {
        const int rh = it / (3 * SB), c = (it / SB) % 3, jj = it % SB;
        const int site = tl.cb0 + jj;
        if (site >= I.g.vh) continue;
        const size_t i = bvec_off(I, R, rh, c) + site;
        const double2 bv = b[i];
        const V bl = from_d2<V>(bv);
        r[i] = bl;
        p[i] = bl;
        for (int k = 0; k < n; ++k) {
            x.at<double2>(k)[i] = make_double2(0.0, 0.0);
            if (k != base || st.lag > 1) ps.at<V>(k)[i] = bl;
        }
#pragma unroll
        for (int q = 0; q < kMaxRhs; ++q)
            if (q == rh) acc[q] += bv.x * bv.x + bv.y * bv.y;
    }
    __shared__ double lds[4 * kMaxRhs];
    block_sum<kMaxRhs>(acc, lds);
    if (threadIdx.x == 0)
        for (int q = 0; q < kMaxRhs; ++q) qout[(size_t)blockIdx.x * kMaxRhs + q] = acc[q];
}

// Scalars of system s from this iteration's sums, by one wave with one shift
// per lane.  The shifted updates are deferred over windows of st.lag iterations
// as in the single-lattice solver: the scalars of each iteration stay in the
// system's [lag][n] window tables w_*, and the window's last iteration (or the
// stopping one) applies them in order.  Also writes the system's state for the
// next iteration (or the final one).
static_assert(kMaxPoles <= 64, "one lane per shift");
struct ShiftState {  // what a lane reads of the previous iteration's state
    double z, zo, shift, bb, a_old, b_old;
    int was, ipp, iter;
    __device__ __forceinline__ ShiftState(const BState& st, const MsIter& S, int k) {
        const bool on = k < st.n;
        z = on ? S.zeta[k] : 0.0;
        zo = on ? S.zeta_old[k] : 0.0;
        shift = on ? st.shift[k] : 0.0;
        was = on ? S.active[k] : 0;
        ipp = on ? S.iters_per_pole[k] : 0;
        bb = S.bb;
        a_old = S.alpha_old;
        b_old = S.beta_old;
        iter = S.iter;
    }
};
__device__ __forceinline__ void bsystem_scalars(const BState& st, int s, int par, const ShiftState& S, double rr,
                                                double pAp, double rAp, double ApAp, BScal& o, double* w_as,
                                                double* w_bs, double* w_zn, int* w_act) {
    const int n = st.n, base = st.base, L = st.lag;
    const int k = threadIdx.x & 63;
    const bool on = k < n;
    const int iter = S.iter;
    const int slot = iter % L;
    const double bb = (iter == 0 && !st.bb_given) ? rr : S.bb;
    const double a_old = S.a_old, b_old = S.b_old, z = S.z, zo = S.zo, shift = S.shift;
    const int was = S.was, ipp = S.ipp;
    const int act = was && !(z * z * rr <= st.tol2 * bb);
    const unsigned long long acts = __ballot(act);
    int nonfinite = !isfinite(rr);
    int stop = nonfinite || !acts || iter >= st.maxiter;
    double alpha = 0.0, beta = 0.0;
    if (!stop) {
        alpha = rr / pAp;
        double rr1 = rr - 2.0 * alpha * rAp + alpha * alpha * ApAp;
        if (rr1 < 0.0) rr1 = 0.0;
        beta = rr1 / rr;
        if (!isfinite(alpha) || !isfinite(beta)) {
            nonfinite = 1;
            stop = 1;
        }
    }
    double zn = z, as = 0.0, bs = 0.0;
    if (!stop) {
        if (k == base) {
            zn = 1.0;
            as = alpha;
            bs = beta;
        } else if (act) {
            zn = z * zo * a_old / (alpha * b_old * (zo - z) + zo * a_old * (1.0 + shift * alpha));
            const double q = zn / z;
            as = alpha * q;
            bs = beta * q * q;
        }
    }
    const int npend = stop ? slot : slot + 1;
    const int flush = npend > 0 && (stop || slot == L - 1);
    int first = act;  // active at the window's first iteration
    if (on) {
        if (slot > 0) first = w_act[k];
        w_as[slot * n + k] = as;
        w_bs[slot * n + k] = bs;
        w_zn[slot * n + k] = zn;
        w_act[slot * n + k] = act;
        MsIter& N = stop ? st.fin[s] : st.it[par ^ 1][s];
        N.active[k] = act;
        N.iters_per_pole[k] = (act && !stop) ? iter + 1 : (was ? iter : ipp);
        N.zeta[k] = zn;
        N.zeta_old[k] = stop ? zo : z;
    }
    const unsigned long long list = __ballot(flush && first && (k != base || L > 1));
    if ((list >> k) & 1) o.list[__popcll(list & ((1ull << k) - 1))] = k;
    if (k == 0) {
        o.alpha = alpha;
        o.beta = beta;
        o.stop = stop;
        o.flush = flush;
        o.npend = npend;
        o.slot = slot;
        o.base_on = L == 1 && !stop && ((acts >> base) & 1);
        o.nact = __popcll(list);
        MsIter& N = stop ? st.fin[s] : st.it[par ^ 1][s];
        N.alpha_old = stop ? a_old : alpha;
        N.beta_old = stop ? b_old : beta;
        N.bb = bb;
        N.rr = rr;
        N.iter = stop ? iter : iter + 1;
        N.nonfinite = nonfinite;
        if (stop) {
            st.sys_done[(size_t)(par ^ 1) * st.n_inst * st.nrhs + s] = 1;
            st.t_done[s] = wall_clock64();
        }
    }
}

// One block per instance: the sums over the instance's tiles and the scalars
// of its systems, evaluated once per iteration instead of in every tile of the
// step.  Reads the stop flags of parity par and writes those of par ^ 1.  One
// wave per right-hand side, whose sums and shifts need no other wave.  Bound by
// a chain of dependent reads (flags, table,
// partials, tables written): 6 us for 9 lattices x 4 right-hand sides x 12
// shifts, every iteration (28 us, and 15 more at the end of a window, with one
// thread per system and the window's scalars copied from a second table).
__global__ __launch_bounds__(64 * kMaxRhs) void k_bms_scalars(BatchDev bd, BState st, const double* __restrict__ dpart,
                                                              const double* __restrict__ qin, int par) {
    const int inst = blockIdx.x;
    const int R = bd.nrhs;
    const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int* done_in = st.inst_done + par * st.n_inst;
    int* done_out = st.inst_done + (par ^ 1) * st.n_inst;
    const BInst& I = bd.inst[inst];
    const int t0 = I.tile0, t1 = t0 + I.ntiles;
    if (done_in[inst]) {
        if (threadIdx.x == 0) done_out[inst] = 1;
        return;
    }
    __shared__ int sh_stop[kMaxRhs];
    const int s = inst * R + q;
    if (q < R) {
        BScal& o = st.scal[s];
        // stopped before this launch; a stop in this launch is written to the other parity
        if (st.sys_done[(size_t)par * st.n_inst * R + s]) {
            if (lane == 0) {
                st.sys_done[(size_t)(par ^ 1) * st.n_inst * R + s] = 1;
                o.stop = 1;
                o.flush = 0;
                o.nact = 0;
                o.base_on = 0;
                sh_stop[q] = 1;
            }
        } else {
            const ShiftState S(st, st.it[par][s], lane);
            double v[4] = {0.0, 0.0, 0.0, 0.0};  // rr and the three dots of the operator
            for (int t = t0 + lane; t < t1; t += 64) {
                v[0] += qin[(size_t)t * kMaxRhs + q];
#pragma unroll
                for (int d = 0; d < 3; ++d) v[1 + d] += dpart[(size_t)t * 3 * kMaxRhs + 3 * q + d];
            }
            wave_sum<4>(v);
            double* wt = st.w_tab + (size_t)s * 3 * kWinTab;
            bsystem_scalars(st, s, par, S, v[0], v[1], v[2], v[3], o, wt, wt + kWinTab, wt + 2 * kWinTab,
                            st.w_act + (size_t)s * kWinTab);
            if (lane == 0) sh_stop[q] = o.stop;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int all = 1;
        for (int r = 0; r < R; ++r) all &= sh_stop[r];
        if (all) done_out[inst] = 1;
    }
}

// r, p and, at the end of a window, the shifted systems of one tile.  A wave
// takes entries of one right-hand side only (four, two or one waves each for
// one, two or more of them), so that the scalars, the list of shifts, their
// vectors' addresses and the window's coefficients are the same for its lanes
// and come by scalar loads.  Bound by its vectors: for 9 lattices of
// 70,848 sites together, 4 right-hand sides and 12 shifts, 12 us an iteration
// (68 MB) and 125 us with the shifts (830 MB, 6.6 TB/s); 22 and 190 us with
// entries of any right-hand side in a wave and the coefficients in LDS.
template <class V>
__global__ __launch_bounds__(kBlock) void k_bms_step(BatchDev bd, V* __restrict__ ring, const V* __restrict__ Ap,
                                                     V* __restrict__ p, VecPtrs x, VecPtrs ps, BState st,
                                                     const BScal* __restrict__ scal,
                                                     const double* __restrict__ w_tab, const int* __restrict__ w_act,
                                                     double* __restrict__ qout, int par) {
    const BTile tl = bd.tiles[blockIdx.x];
    if (st.inst_done[par * st.n_inst + tl.inst]) return;
    const BInst I = bd.inst[tl.inst];
    const int R = bd.nrhs, SB = bd.tile_sites, n = st.n, L = st.lag, base = st.base;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nw = R == 1 ? 4 : R == 2 ? 2 : 1;  // waves per right-hand side
    const int rh = wave / nw;
    __shared__ double lds[kBlock / 64];
    double acc[1] = {0.0};
    if (rh < R) {
        const size_t sy = (size_t)tl.inst * R + rh;
        const BScal& S = scal[sy];
        const int nitem = 3 * SB, first = (wave % nw) * 64 + lane, stride = nw * 64;
        const int lgSB = 31 - __clz(SB);  // SB is a power of two
        const size_t off = bvec_off(I, R, rh, 0);
        // the base system's r and p (and its x where the window is one iteration;
        // longer windows update it with the others, which saves reading and
        // writing it each time): kItems entries per lane with their loads in
        // flight together
        constexpr int kItems = 3;
        if (!S.stop) {
            const double alpha = S.alpha, beta = S.beta;
            const V* r_in = ring + (size_t)S.slot * st.ring_stride;
            V* r_out = ring + (size_t)((S.slot + 1) % L) * st.ring_stride;
            for (int it0 = first; it0 < nitem; it0 += kItems * stride) {
                V r0[kItems], a[kItems], pv[kItems];
                double2 xv[kItems];
                size_t idx[kItems];
                bool on[kItems];
#pragma unroll
                for (int u = 0; u < kItems; ++u) {
                    const int it = it0 + u * stride;
                    const int c = it >> lgSB, site = tl.cb0 + (it & (SB - 1));
                    on[u] = it < nitem && site < I.g.vh;
                    idx[u] = off + (size_t)c * I.g.vh + site;
                    if (on[u]) {
                        r0[u] = r_in[idx[u]];
                        a[u] = Ap[idx[u]];
                        pv[u] = p[idx[u]];
                        if (S.base_on) xv[u] = x.at<double2>(base)[idx[u]];
                    }
                }
#pragma unroll
                for (int u = 0; u < kItems; ++u) {
                    if (!on[u]) continue;
                    double2 rv = to_d2(r0[u]);
                    const double2 av = to_d2(a[u]), pd = to_d2(pv[u]);
                    rv.x -= alpha * av.x;
                    rv.y -= alpha * av.y;
                    const V rl = from_d2<V>(rv);
                    r_out[idx[u]] = rl;
                    rv = to_d2(rl);
                    acc[0] += rv.x * rv.x + rv.y * rv.y;
                    if (S.base_on)
                        x.at<double2>(base)[idx[u]] = make_double2(xv[u].x + alpha * pd.x, xv[u].y + alpha * pd.y);
                    p[idx[u]] = from_d2<V>(make_double2(rv.x + beta * pd.x, rv.y + beta * pd.y));
                }
            }
        }
        // the shifted systems at the end of their window (residuals of the window
        // are in the ring: a lane reads back the ones that it wrote above)
        const int nact = S.flush ? S.nact : 0, npend = S.npend;
        const double* w_as = w_tab + sy * 3 * kWinTab;
        const double* w_bs = w_as + kWinTab;
        const double* w_zn = w_bs + kWinTab;
        const int* act = w_act + sy * kWinTab;
        for (int it = first; nact > 0 && it < nitem; it += stride) {
            const int c = it >> lgSB, site = tl.cb0 + (it & (SB - 1));
            if (site >= I.g.vh) continue;
            const size_t i = off + (size_t)c * I.g.vh + site;
            double2 rw[kLagMax];
#pragma unroll
            for (int t = 0; t < kLagMax; ++t) {
                if (t >= npend) break;
                rw[t] = to_d2(ring[(size_t)((t + 1) % L) * st.ring_stride + i]);
            }
            constexpr int G = 4;
            for (int g0 = 0; g0 < nact; g0 += G) {
                double2 pk[G], xk[G];
#pragma unroll
                for (int jq = 0; jq < G; ++jq)
                    if (g0 + jq < nact) {
                        const int k = S.list[g0 + jq];
                        pk[jq] = to_d2(ps.at<V>(k)[i]);
                        xk[jq] = x.at<double2>(k)[i];
                    }
#pragma unroll
                for (int t = 0; t < kLagMax; ++t) {
                    if (t >= npend) break;
#pragma unroll
                    for (int jq = 0; jq < G; ++jq)
                        if (g0 + jq < nact) {
                            const int k = S.list[g0 + jq];
                            if (act[t * n + k]) {
                                const double aq = w_as[t * n + k], bq = w_bs[t * n + k], zq = w_zn[t * n + k];
                                xk[jq] = make_double2(xk[jq].x + aq * pk[jq].x, xk[jq].y + aq * pk[jq].y);
                                pk[jq] = to_d2(from_d2<V>(make_double2(zq * rw[t].x + bq * pk[jq].x,
                                                                       zq * rw[t].y + bq * pk[jq].y)));
                            }
                        }
                }
#pragma unroll
                for (int jq = 0; jq < G; ++jq)
                    if (g0 + jq < nact) {
                        const int k = S.list[g0 + jq];
                        x.at<double2>(k)[i] = xk[jq];
                        ps.at<V>(k)[i] = from_d2<V>(pk[jq]);
                    }
            }
        }
    }
    wave_sum<1>(acc);
    if (lane == 0) lds[wave] = acc[0];
    __syncthreads();
    if ((int)threadIdx.x < R) {
        double v = 0.0;
        for (int w = 0; w < nw; ++w) v += lds[threadIdx.x * nw + w];
        qout[(size_t)blockIdx.x * kMaxRhs + threadIdx.x] = v;
    }
}

// one block per system: its (tile, rhs) partials over the instance's tiles
__global__ __launch_bounds__(kBlock) void k_bsys_sum(BatchDev bd, const double* __restrict__ part,
                                                     double* __restrict__ out) {
    const int s = blockIdx.x;
    const int R = bd.nrhs;
    const BInst I = bd.inst[s / R];
    const int q = s % R;
    double t[1] = {0.0};
    for (int k = threadIdx.x; k < I.ntiles; k += kBlock) t[0] += part[(size_t)(I.tile0 + k) * kMaxRhs + q];
    __shared__ double lds[4];
    block_sum<1>(t, lds);
    if (threadIdx.x == 0) out[s] = t[0];
}

// canonical packed [inst][rhs][site][colour] <-> internal [inst][rhs][colour][site]
__global__ void k_bvec_import(BatchDev bd, const double2* __restrict__ canon, double2* __restrict__ vec) {
    const BTile tl = bd.tiles[blockIdx.x];
    const BInst I = bd.inst[tl.inst];
    const int R = bd.nrhs, SB = bd.tile_sites;
    for (int it = threadIdx.x; it < R * SB; it += blockDim.x) {
        const int rh = it / SB, site = tl.cb0 + it % SB;
        if (site >= I.g.vh) continue;
        const size_t cbase = (size_t)3 * ((size_t)R * I.off + (size_t)rh * I.g.vh + site);
#pragma unroll
        for (int c = 0; c < 3; ++c) vec[bvec_off(I, R, rh, c) + site] = canon[cbase + c];
    }
}

__global__ void k_bvec_export(BatchDev bd, const double2* __restrict__ vec, double2* __restrict__ canon) {
    const BTile tl = bd.tiles[blockIdx.x];
    const BInst I = bd.inst[tl.inst];
    const int R = bd.nrhs, SB = bd.tile_sites;
    for (int it = threadIdx.x; it < R * SB; it += blockDim.x) {
        const int rh = it / SB, site = tl.cb0 + it % SB;
        if (site >= I.g.vh) continue;
        const size_t cbase = (size_t)3 * ((size_t)R * I.off + (size_t)rh * I.g.vh + site);
#pragma unroll
        for (int c = 0; c < 3; ++c) canon[cbase + c] = vec[bvec_off(I, R, rh, c) + site];
    }
}

__global__ void k_blinks_to_f32(const double2* __restrict__ d, float2* __restrict__ f, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const double2 v = d[i];
        f[i] = make_float2((float)v.x, (float)v.y);
    }
}

__global__ void k_bstate_init(BState st, int from_fin) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const int nsys = st.n_inst * st.nrhs;
    if (s >= nsys) return;
    MsIter& S = st.it[0][s];
    for (int k = 0; k < st.n; ++k) {
        S.zeta[k] = S.zeta_old[k] = 1.0;
        S.active[k] = 1;
        S.iters_per_pole[k] = 0;
    }
    S.alpha_old = 1.0;
    S.beta_old = 0.0;
    S.bb = from_fin ? st.fin[s].bb : 0.0;
    S.rr = 0.0;
    S.iter = 0;
    S.nonfinite = 0;
    st.sys_done[s] = 0;
    st.sys_done[nsys + s] = 0;
    st.t_done[s] = 0;
    if (s % st.nrhs == 0) {
        st.inst_done[s / st.nrhs] = 0;
        st.inst_done[st.n_inst + s / st.nrhs] = 0;
    }
}

__global__ void k_baxpy(size_t n, double2* __restrict__ x, const double2* __restrict__ e) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const double2 a = x[i], b = e[i];
        x[i] = make_double2(a.x + b.x, a.y + b.y);
    }
}

__global__ void k_timestamp(unsigned long long* t) {
    if (threadIdx.x == 0 && blockIdx.x == 0) t[0] = wall_clock64();
}

}  // namespace

template <class V>
void launch_bdslash(const BatchDev& bd, int tps, const void* links, const V* in, V* out, int out_par,
                    const int* inst_done, hipStream_t s) {
    bdslash_tps<V>(bd, tps, (const V*)links, in, out_par, BEpiStore<V>{nullptr, out}, inst_done, s);
}
template void launch_bdslash<double2>(const BatchDev&, int, const void*, const double2*, double2*, int, const int*,
                                      hipStream_t);
template void launch_bdslash<float2>(const BatchDev&, int, const void*, const float2*, float2*, int, const int*,
                                     hipStream_t);

template <class V>
void launch_bdslash_cg(const BatchDev& bd, int tps, const void* links, const V* w_o, const V* p, const V* r, V* Ap,
                       BState st, const int* inst_done, double* dpart, hipStream_t s) {
    bdslash_tps<V>(bd, tps, (const V*)links, w_o, 0, BEpiCG<V>{dpart, Ap, p, r, st.sigma0_term}, inst_done, s);
}
template void launch_bdslash_cg<double2>(const BatchDev&, int, const void*, const double2*, const double2*,
                                         const double2*, double2*, BState, const int*, double*, hipStream_t);
template void launch_bdslash_cg<float2>(const BatchDev&, int, const void*, const float2*, const float2*, const float2*,
                                        float2*, BState, const int*, double*, hipStream_t);

void launch_bdslash_resid(const BatchDev& bd, int tps, const double2* links, const double2* w_o, const double2* x,
                          const double2* b, double pole, double* part, double2* rout, hipStream_t s) {
    bdslash_tps<double2>(bd, tps, links, w_o, 0, BEpiResid{part, x, b, rout, pole}, nullptr, s);
}

template <class V>
void launch_bms_init(const BatchDev& bd, const double2* b, V* r, V* p, VecPtrs x, VecPtrs ps, BState st,
                     double* qout, hipStream_t s) {
    k_bms_init<V><<<bd.ntiles, kBlock, 0, s>>>(bd, b, r, p, x, ps, st, qout);
}
template void launch_bms_init<double2>(const BatchDev&, const double2*, double2*, double2*, VecPtrs, VecPtrs,
                                       BState, double*, hipStream_t);
template void launch_bms_init<float2>(const BatchDev&, const double2*, float2*, float2*, VecPtrs, VecPtrs,
                                      BState, double*, hipStream_t);

template <class V>
void launch_bms_step(const BatchDev& bd, V* r, const V* Ap, V* p, VecPtrs x, VecPtrs ps, BState st,
                     const double* dpart, const double* qin, double* qout, int par, hipStream_t s) {
    (void)dpart;
    (void)qin;
    k_bms_step<V><<<bd.ntiles, kBlock, 0, s>>>(bd, r, Ap, p, x, ps, st, st.scal, st.w_tab, st.w_act, qout, par);
}
template void launch_bms_step<double2>(const BatchDev&, double2*, const double2*, double2*, VecPtrs, VecPtrs, BState,
                                       const double*, const double*, double*, int, hipStream_t);
template void launch_bms_step<float2>(const BatchDev&, float2*, const float2*, float2*, VecPtrs, VecPtrs, BState,
                                      const double*, const double*, double*, int, hipStream_t);

void launch_bms_scalars(const BatchDev& bd, BState st, const double* dpart, const double* qin, int par,
                        hipStream_t s) {
    k_bms_scalars<<<st.n_inst, kBlock, 0, s>>>(bd, st, dpart, qin, par);
}

void launch_bsys_sum(const BatchDev& bd, int n_inst, const double* part, double* out, hipStream_t s) {
    const int n = n_inst * bd.nrhs;
    k_bsys_sum<<<n, kBlock, 0, s>>>(bd, part, out);
}

void launch_bvec_import(const BatchDev& bd, const double2* canon, double2* vec, hipStream_t s) {
    k_bvec_import<<<bd.ntiles, kBlock, 0, s>>>(bd, canon, vec);
}
void launch_bvec_export(const BatchDev& bd, const double2* vec, double2* canon, hipStream_t s) {
    k_bvec_export<<<bd.ntiles, kBlock, 0, s>>>(bd, vec, canon);
}
void launch_blinks_to_f32(const double2* d, float2* f, size_t n, hipStream_t s) {
    int nb = (int)((n + 255) / 256);
    if (nb > 8192) nb = 8192;
    k_blinks_to_f32<<<nb, 256, 0, s>>>(d, f, n);
}
void launch_b_timestamp(unsigned long long* t, hipStream_t s) { k_timestamp<<<1, 64, 0, s>>>(t); }

void launch_bstate_init(BState st, int from_fin, hipStream_t s) {
    const int n = st.n_inst * st.nrhs;
    k_bstate_init<<<(n + 255) / 256, 256, 0, s>>>(st, from_fin);
}

void launch_baxpy(size_t n, double2* x, const double2* e, hipStream_t s) {
    int nb = (int)((n + 255) / 256);
    if (nb > 8192) nb = 8192;
    k_baxpy<<<nb, 256, 0, s>>>(n, x, e);
}

}  // namespace stag
