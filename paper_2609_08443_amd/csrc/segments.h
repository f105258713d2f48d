// Ragged scheduling without a work-list launch: a workgroup finds the segments of
// its own token range from the offsets.
//
// The (head, token) pairs form one head-major index space of length H*T, cut into
// equal ranges of C, as for the work list (worklist.hip).  A (user, head) pair whose
// tokens span several ranges leaves one partial a range: slot r from the segment
// that begins with range r (only one does), slot n_ranges + h B + b from the pair's
// first segment when it begins inside a range.  The merge derives a pair's slots
// from its offsets in the same way; there are n_ranges + H B of them.
//
// Offsets are device data the host never reads: every value is clamped to [0, T]
// and every step of the walk moves forward, so malformed offsets give wrong
// values but neither an access out of range nor an endless loop.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sa {

__device__ inline int64_t seg_clamp(int64_t x, int64_t T) { return x < 0 ? 0 : (x > T ? T : x); }

// first user whose tokens end after t (B when there is none)
__device__ inline int64_t first_user_after(const int64_t* off, int64_t B, int64_t T, int64_t t) {
    int64_t lo = 0, hi = B;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (seg_clamp(off[mid + 1], T) > t) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// the same from user b on, in steps that double: a run of n users without tokens costs
// about 2 log2 n reads (one at a time, 4,000 of them between two users took 1.1 ms)
__device__ inline int64_t next_user_after(const int64_t* off, int64_t b, int64_t B, int64_t T, int64_t t) {
    int64_t lo = b, hi = b, step = 1;
    while (hi < B && seg_clamp(off[hi + 1], T) <= t) {
        lo = hi + 1;
        hi = lo + step;
        step *= 2;
    }
    if (hi > B) hi = B;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (seg_clamp(off[mid + 1], T) > t) hi = mid; else lo = mid + 1;
    }
    return lo;
}

struct Segment {
    int32_t b, h;       // user and head
    int32_t t0, t1;     // tokens [t0, t1)
    int64_t slot;       // partial slot, used when split
    bool split;         // the user's tokens of this head span several ranges
};

class SegmentWalk {
  public:
    __device__ inline SegmentWalk(const int64_t* off, int64_t B, int64_t T, int32_t H, int64_t C, int64_t n_ranges, int64_t range)
        : off_(off), B_(B), T_(T), C_(C), n_ranges_(n_ranges), range_(range) {
        const int64_t HT = (int64_t)H * T;
        g_ = range * C;
        end_ = g_ + C < HT ? g_ + C : HT;
        h_ = g_ < T || T <= 0 ? 0 : (int32_t)(g_ / T);
        b_ = first_user_after(off, B, T, g_ - (int64_t)h_ * T);
    }
    // the next non-empty segment, or false at the end of the range
    __device__ inline bool next(Segment& s) {
        while (g_ < end_) {
            if (b_ >= B_) {   // past the last user of this head
                ++h_;
                g_ = (int64_t)h_ * T_;
                b_ = 0;
                continue;
            }
            const int64_t base = (int64_t)h_ * T_;
            const int64_t lo = seg_clamp(off_[b_], T_), hi = seg_clamp(off_[b_ + 1], T_);
            const int64_t t = g_ - base;
            const int64_t t0 = t > lo ? t : lo;
            const int64_t lim = end_ - base;
            const int64_t t1 = hi < lim ? hi : lim;
            const int32_t b = (int32_t)b_++;
            if (__builtin_expect(t1 <= t0, 0)) {
                if (lo >= lim) g_ = end_;   // begins after this range
                else b_ = next_user_after(off_, b_, B_, T_, t);
                continue;
            }
            s.b = b;
            s.h = h_;
            s.t0 = (int32_t)t0;
            s.t1 = (int32_t)t1;
            s.split = base + lo < range_ * C_ || base + hi > (range_ + 1) * C_;
            s.slot = base + t0 == range_ * C_ ? range_ : n_ranges_ + h_ * B_ + b;
            g_ = base + t1;
            return true;
        }
        return false;
    }

  private:
    const int64_t* off_;
    int64_t B_, T_, C_, n_ranges_, range_, g_, end_, b_;
    int32_t h_;
};

// Partial slots of user b of B, head h, with tokens [lo, hi): slot(i) for
// i = 0 .. count - 1, in token order; count = 0 for an empty user.
struct PairSlots {
    int64_t count, first, rest;   // slot(0), and slot(i) = rest + i from there on
    __device__ inline PairSlots(int64_t lo, int64_t hi, int64_t b, int64_t h, int64_t B, int64_t T, int64_t C,
                                int64_t n_ranges)
        : count(0), first(0), rest(0) {
        if (hi <= lo) return;
        const int64_t g0 = h * T + lo, g1 = h * T + hi - 1;
        rest = g0 / C;
        count = g1 / C - rest + 1;
        first = g0 == rest * C ? rest : n_ranges + h * B + b;
    }
    __device__ inline int64_t slot(int64_t i) const { return i == 0 ? first : rest + i; }
};

}  // namespace sa
