// When to try again a path that failed for reasons that may pass: a launch that
// was refused, memory that could not be had, a wait that took too long because
// another process held the GPU.  Host code without HIP.
#pragma once

namespace stag {

// After a failure the path is left out of the next kFirst uses, after another one
// without a success between them of twice as many, up to kMost, and a try has
// kShare of the first one's patience.  A wait of a second, the only failure
// that costs anything, then takes 1 s once and 31 ms in at least kFirst uses; the
// path that stands in takes up to twice the time of the one left out, so that
// leaving it out for good costs more within a few thousand uses.
class Backoff {
    static constexpr int kFirst = 16, kMost = 1024, kShare = 32;
    int left = 0, next = kFirst;

   public:
    // Is the path to be tried in this use?
    bool use() {
        if (left == 0) return true;
        --left;
        return false;
    }
    void failed() {
        left = next;
        next = 2 * next < kMost ? 2 * next : kMost;
    }
    void worked() { next = kFirst; }
    unsigned long long patience(unsigned long long full) const { return next == kFirst ? full : full / kShare; }
};

}  // namespace stag
