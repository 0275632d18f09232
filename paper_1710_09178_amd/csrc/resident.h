// The resident multi-shift CG (Sec. 4): a whole solve in one cooperative launch
// that keeps the links in registers.  Kernel and protocol: resident.hip.
#pragma once

#include "dslash.h"

namespace stag {

constexpr int kResTile = 64;     // even (and odd) sites of one block
constexpr int kResThreads = 512;
constexpr int kResCopies = 8;    // copies of the group sums, read by the blocks of one XCD each
constexpr int kResRecord = 128;  // bytes from one record of sums to the next
constexpr int kResMax = 1024;    // blocks at most
constexpr int kResDirect = 32;   // grids up to this add the block sums without groups
inline int resident_blocks(const Geom& g) { return (g.vh + kResTile - 1) / kResTile; }
// Exchange area of a lattice: two odd and three even half vectors (FP64 size), and
// three times the sums of blocks and of groups of 16 blocks.
inline size_t resident_bytes(const Geom& g) {
    const size_t nb = resident_blocks(g);
    return 5 * (size_t)48 * g.vh + 128 + 3 * kResRecord * (nb + kResCopies * ((nb + 15) / 16));
}

template <class V>
struct ResidentArgs {
    const double2* b;     // source of a new solve (x = 0, r = p = p_s = b), or NULL:
    V *r, *p;             // ... continue from r, p, x_base and st->it[0], and leave them there
    VecPtrs x, ps;        // ps: consecutive half vectors
    MsState* st;          // st->fin, st->done at the stop; st->aborted when a wait timed out
    void* xch;            // resident_bytes(g)
    int n, base, lag, max_steps;
    double mt;            // 4m^2 + sigma_0
    unsigned long long wait;  // ticks of the 100 MHz wall clock before a wait is given up
};

// Can this lattice and operator run in one co-resident grid on the current device?
// (refine: the FP32 CG of a single system, continued from given vectors)
bool resident_fits(const Geom& g, const LinkSet& ls, bool fp64, bool refine = false);
// Fills the exchange area and enqueues the solver; V = double2 (operator
// format fmt64) or float2 (format fmt32).
template <class V>
hipError_t launch_resident(const Geom& g, const LinkSet& ls, const ResidentArgs<V>& a, hipStream_t s);

}  // namespace stag
