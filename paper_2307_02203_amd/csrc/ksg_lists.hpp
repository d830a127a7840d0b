// Layout of the neighbour search's lists and the bounds of a walk over them (ksg.hip), in
// plain C++ so that a host program can run the same arithmetic.
//
// A pair's lists are the x order's two, then the y order's two, each list between kPad
// sentinels:
//   [pad | list 0: n0 | pad | pad | list 1: n1 = N - n0 | pad] = list_entries(N)
// entries per order; list 0 holds the samples of the lower n0 ranks of the other order, 0 <
// n0 < N.  A walk reads blocks of kPad entries outwards, a side at a time, and
// goes on while the farthest one of its block is nearer than the k-th distance, which is at
// most kUnset.  The blocks of a side are kPad apart, so exactly one of them has its farthest
// entry in the outermost sentinels of its side; a code in [0, 2^23] is at least kUnset away
// from those, so the walk ends there at the latest, with every read inside the region, for
// any place that walk_place or walk_other returns and whatever the entries between hold.
#pragma once
#include <stdint.h>

namespace ndf {

constexpr int kPad = 4;             // sentinel samples on each side of a list
constexpr int kFar = 1 << 29;       // sentinel code: its distance to any sample exceeds kUnset
constexpr int kUnset = (1 << 24) - 32;  // k-th distance before k samples are seen: above any
                                    // code difference (<= 2^23), below any sentinel distance,
                                    // and the greatest list distance of a walk start
constexpr int kTopCode = 1 << 23;   // codes lie in [0, kTopCode]
static_assert(kFar - kTopCode >= kUnset, "a sentinel ends a walk");

// The rank at which an order's samples are split, from its sorted codes a[0 .. N): N / 2, or
// where a long run of equal codes (kLongRun: a sixteenth of the samples) lies across it, the
// nearer end of the run (but not an end of the order).  A run cut in two leaves a few of its
// samples in the list of the other codes, where each walks through all of them (20,000
// vertices, us: 1000 members of two values, k = 8, 528 cut and 298 whole; 90 % zeros, k = 4,
// 902 and 503; 2048 members of four values 1265 and 822).  Short runs stay cut: the search
// took 7 % of a pair of 1000 members and 100 values.  From 1 to N - 1 whatever a holds.
constexpr int kLongRun = 16;
template <typename Codes>
__host__ __device__ inline int split_rank(const Codes &a, int N) {
    const int h = N / 2, c = a[h], q = N / kLongRun;
    if (a[h - 1] < c || (a[h - 1 - q] < c && a[h + q] > c)) return h;
    int lo = 0, hi = h;  // first rank of code c or more
    while (lo < hi) {
        const int m = (lo + hi) / 2;
        if (a[m] < c)
            lo = m + 1;
        else
            hi = m;
    }
    int end = h + 1, top = N;  // first rank above code c
    while (end < top) {
        const int m = (end + top) / 2;
        if (a[m] > c)
            top = m;
        else
            end = m + 1;
    }
    if (lo == 0) return end < N ? end : h;
    return end == N || h - lo <= end - h ? lo : end;
}

__host__ __device__ constexpr int list_entries(int N) { return N + 4 * kPad; }
__host__ __device__ constexpr int clamp_int(int v, int lo, int hi) {
    return v < lo ? lo : v > hi ? hi : v;
}

// Places count entries from the first list's first.  Place of the sample of rank r in its
// order's lists, q1 of the ranks below r being in list 1 (clamped into the list, so that
// even unprepared orders stay in bounds).
__host__ __device__ inline int list_place(bool up, int r, int q1, int n0, int n1) {
    return up ? n0 + 2 * kPad + (q1 < n1 - 1 ? q1 : n1 - 1) : clamp_int(r - q1, 0, n0 - 1);
}
// A sample's place in one list plus the place where it would stand in the order's other
// list, r samples of the order being below it; `first`: the order's first entry.
__host__ __device__ constexpr int place_sum(int first, int n0, int r) {
    return 2 * first + n0 + 2 * kPad + r;
}

// Pad `pad` (0..3: left and right of list 0, left and right of list 1) of an order that
// starts at entry `first`: its first entry, and the sentinels' code.
__host__ __device__ inline int pad_place(int pad, int first, int n0, int n1) {
    return first + (pad == 0   ? 0
                    : pad == 1 ? kPad + n0
                    : pad == 2 ? n0 + 2 * kPad
                               : n0 + 3 * kPad + n1);
}
__host__ __device__ inline int pad_code(int pad) { return pad & 1 ? kFar : -kFar; }

// The place a walk starts at (its own sample's) and the one it goes on at in the other
// list: no-ops on prepared orders.  In an order that is no permutation a sample without an
// entry leaves what its word held before, which must not lead out of the lists (a negative
// place is a large unsigned one).
__host__ __device__ constexpr uint32_t min_u32(uint32_t a, uint32_t b) { return a < b ? a : b; }
__host__ __device__ constexpr int walk_place(uint32_t at, int entries) {
    return (int)min_u32(at, (uint32_t)(2 * entries - 2 * kPad - 1));
}
__host__ __device__ constexpr int walk_other(int at, int entries) {
    return (int)min_u32((uint32_t)at, (uint32_t)(2 * entries - 2 * kPad));
}
// The walked code of a walk's own sample: a no-op on a sample's entry, else in the range
// from which every sentinel is far.
__host__ __device__ constexpr int walk_code(int c) { return clamp_int(c, 0, kTopCode); }

// The member at an entry of a stored order: a no-op on prepared orders, else in bounds.
__host__ __device__ constexpr int order_member(uint16_t m, int N) { return m < N ? m : N - 1; }

// A walk start as one word: place (13 bits) and the distance to the other list in units of
// 32, rounded down (a list visited for nothing changes no result).
__host__ __device__ constexpr uint32_t pack_start(int place, int gap) {
    return (uint32_t)place | (uint32_t)(gap > 0 ? gap : 0) >> 5 << 13;
}
__host__ __device__ constexpr uint32_t start_place(uint32_t s) { return s & 0x1fff; }
__host__ __device__ constexpr int start_gap(uint32_t s) { return (int)(s >> 13 << 5); }

}  // namespace ndf
