// Direct KSG mutual-information dependence (Sec. 3.2, Eq. 2; nearest-neighbour
// estimator of Kraskov, Stoegbauer and Grassberger, their first algorithm).
//
// For one (reference a, query b) pair the N samples are (x_m, y_m) =
// (code[a][m], code[b][m]), integer codes from ndf_prepare.  For every sample
//   eps_m = k-th smallest max(|x_m - x_j|, |y_m - y_j|) over j != m,
//   nx_m  = #{j != m : |x_m - x_j| < eps_m},  ny_m likewise in y,
// and I = psi(k) + psi(N) - <psi(nx+1) + psi(ny+1)>, which with
// psi(n) = H_{n-1} - gamma is H_{k-1} + H_{N-1} - <H_nx + H_ny>.
//
// GPU design (one workgroup per pair, four samples per thread, everything in LDS; a
// pair of up to 256 members is one wave, of up to 2048 eight):
//  * the samples are known in two orders, by x and by y; both come from the
//    per-vertex sorted member orders that ndf_prepare stores (ties by member
//    index), so no query sorts anything; without stored orders every column is
//    sorted on the fly, which gives the same results;
//  * for the neighbour search each order is split in two lists: the x order into the
//    samples below and above the median y rank, the y order likewise by x rank (at the end
//    of a run of equal codes where the median lies in one);
//  * the k nearest neighbours of a sample are found by walking outwards from its
//    own position in its list of one order, stopping on each side once the
//    distance along that coordinate reaches the current k-th distance (under the
//    max-norm no later sample can be closer); only a sample nearer to the other list
//    (in the coordinate that splits them) than its k-th distance walks that list too.
//    Each sample walks the order in which its nearest codes are spread widest, i.e.
//    where the strip the walk must cover holds the fewest samples; any choice gives
//    the same exact result;
//  * the marginal counts are two lower bounds each, over the sorted x codes and
//    over the sorted y codes; a bucket table of each order (built per pair in
//    LDS) narrows every search to the few samples of one code bucket;
//  * all distances and counts are exact int32, so the counts equal a brute-force
//    evaluation bit for bit; the harmonic sum is FP64.
#include <type_traits>

#include "ksg_lists.hpp"
#include "order.hpp"

namespace ndf {

constexpr int kKsgWaves = 4;  // of the sorting kernels
constexpr int kKsgThreads = 64 * kKsgWaves;

__device__ __forceinline__ int pow2_ceil(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// Ascending bitonic sort of P (power of two) keys in LDS by the workgroup.
template <typename T>
__device__ void block_bitonic_sort(T *a, int P) {
    const int tid = threadIdx.x;
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = tid; t < P / 2; t += kKsgThreads) {
                const int i = 2 * t - (t & (stride - 1));
                const int j = i + stride;
                const bool up = (i & size) == 0;
                T u = a[i], w = a[j];
                if ((u > w) == up) {
                    a[i] = w;
                    a[j] = u;
                }
            }
            __syncthreads();
        }
    }
}

// H[n] = 1 + 1/2 + ... + 1/n, summed in order in FP64 (a thread that summed it on the
// GPU took 60 us for 1000 members in front of every call).
constexpr int kKsgMaxN = 2048;
struct Harmonic {
    double v[kKsgMaxN + 1];
    constexpr Harmonic() : v() {
        double h = 0.0;
        v[0] = 0.0;
        for (int i = 1; i <= kKsgMaxN; ++i) {
            h += 1.0 / (double)i;
            v[i] = h;
        }
    }
};
static __device__ const Harmonic kHarmonic{};

// Shape of the pair kernels with W waves: four samples per thread, up to 256 W members.
// Bucket tables of the marginal searches: T[b] = number of sorted codes below
// b << kShift for b = 0 .. kTab - 1 (codes lie in [0, 2^23], so the last entry is N).
// A lower bound of v then only searches [T[b], T[b + 1]] with b = v >> kShift: a
// handful of samples instead of all N.  The bucket width follows the sample count
// (at 1000 members half and twice the width cost 5 and 1.6 %).
constexpr int kPer = 4;  // samples per thread
template <int W>
struct Pair {
    static constexpr int kT = 64 * W;                       // threads
    static constexpr int kMax = kPer * kT;                  // members
    static constexpr int kChunks = kMax / 64;
    static constexpr int kShift = 16 - (W >= 8 ? 3 : W >= 4 ? 2 : W >= 2 ? 1 : 0);
    static constexpr int kTab = ((1 << 23) >> kShift) + 2;  // W = 4: 514 entries
};

template <int W>
__device__ __forceinline__ int tab_bucket(int v) {
    return min(max(v, 0), 1 << 23) >> Pair<W>::kShift;  // at most kTab - 2
}

// Table construction in three steps with a workgroup barrier between them:
// every entry N (all threads) ...
template <int W>
__device__ __forceinline__ void tab_fill(uint16_t *T, int N) {
    for (int i = threadIdx.x; i < Pair<W>::kTab; i += Pair<W>::kT) T[i] = (uint16_t)N;
}
// ... the first position of every non-empty bucket of the sorted a[0..N) (all
// threads) ...
template <int W>
__device__ __forceinline__ void tab_scatter(const int *a, uint16_t *T, int N) {
    for (int j = threadIdx.x; j < N; j += Pair<W>::kT) {
        const int b = tab_bucket<W>(a[j]);
        if (j == 0 || tab_bucket<W>(a[j - 1]) != b) T[b] = (uint16_t)j;
    }
}
// ... and a suffix minimum by one wave, so that an empty bucket takes the first
// position of the next non-empty one (lane l owns entries kP l .. kP l + kP - 1).
template <int W>
__device__ __forceinline__ void tab_scan(uint16_t *T) {
    constexpr int kTab = Pair<W>::kTab, kP = (kTab + 63) / 64;
    const int lane = threadIdx.x & 63;
    int v[kP];
    int run = 0xffff;
#pragma unroll
    for (int i = kP - 1; i >= 0; --i) {
        const int idx = lane * kP + i;
        if (idx < kTab) run = min(run, (int)T[idx]);
        v[i] = run;
    }
    int s = run;  // minimum over the chunks of this lane and all later ones
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_down(s, d);
        if (lane + d < 64) s = min(s, t);
    }
    int carry = __shfl_down(s, 1);
    if (lane == 63) carry = 0xffff;
#pragma unroll
    for (int i = 0; i < kP; ++i) {
        const int idx = lane * kP + i;
        if (idx < kTab) T[idx] = (uint16_t)min(v[i], carry);
    }
}

// Marginal counts of one sample (x, y) with k-th distance eps > 0: entries of the
// sorted x codes xs and of the sorted y codes ys strictly inside (v - eps, v + eps),
// minus the sample itself.  Each of the four lower bounds starts from its bucket
// range [T[b], T[b + 1]]; the searches advance in lockstep from the widest range's
// step, so their LDS reads are in flight together.  A probe stops at its range's end
// (the entry before the end may lie at index -1, which is readable and moves nothing).
template <int W>
__device__ __forceinline__ void marginal_counts(const int *xs, const int *ys, const uint16_t *Tx,
                                                const uint16_t *Ty, int x, int y, int eps, int &nx,
                                                int &ny) {
    const int val[4] = {x + eps, x - eps + 1, y + eps, y - eps + 1};
    int pos[4], hi[4], span = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint16_t *T = (i < 2 ? Tx : Ty) + tab_bucket<W>(val[i]);
        pos[i] = T[0];
        hi[i] = T[1];
        span = max(span, hi[i] - pos[i]);
    }
    for (int st = span > 0 ? 1 << (31 - __clz(span)) : 0; st > 0; st >>= 1) {
        int t[4], c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            t[i] = min(pos[i] + st, hi[i]);
            c[i] = (i < 2 ? xs : ys)[t[i] - 1];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) pos[i] = c[i] < val[i] ? t[i] : pos[i];
    }
    nx = pos[0] - pos[1] - 1;
    ny = pos[2] - pos[3] - 1;
}

// v_med3_i32: the middle of three signed integers.  With lo <= hi it is d
// clamped to [lo, hi] in one instruction (the compiler forms it only for
// constant bounds).  Operands are plain VALU results, so the asm needs no wait
// states.
__device__ __forceinline__ int med3_i32(int d, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(d), "v"(lo), "v"(hi));
    return r;
}

// |a - b| of two codes (both in [0, 2^24)) in one v_sad_u32.
__device__ __forceinline__ int absdiff_u32(int a, int b) {
    int r;
    asm("v_sad_u32 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <int K>
__device__ __forceinline__ void insert_k(int (&best)[K], int d) {
    // best ascending; keep the K smallest of best + {d} (ties kept with
    // multiplicity): best[t] = min(best[t], max(best[t - 1], d)) = d clamped
    // to [best[t - 1], best[t]]
#pragma unroll
    for (int t = K - 1; t > 0; --t) best[t] = med3_i32(d, best[t - 1], best[t]);
    best[0] = min(best[0], d);
}

// LDS of one pair.  The lists of the neighbour search live in `lists` (ksg_lists.hpp),
// entry = (walked coordinate, other coordinate).  Before the lists are written the
// region serves as scratch, and after the walks as the sorted codes xs[N], ys[N] of
// the counts (from its second word on).
struct PairLds {
    int2 *lists;
    int *eps;         // [N] y codes in y order, then walk starts, then k-th distances
    uint16_t *yrank;  // [N] y rank of x-order sample p
    uint16_t *other;  // [N] sample p's place in the y order's lists, then its place in the
                      // other list of its walk
    uint16_t *Tx, *Ty;
    uint16_t *perm;   // [N] members of the x order, where they are not stored (pairs mode)
};

// The bytes of `lists`: both orders' lists, or the exchange buffer of the sort.
template <int W>
__host__ __device__ inline size_t lists_bytes(int N) {
    const size_t l = (size_t)2 * list_entries(N) * 8, x = (size_t)Pair<W>::kMax * 8;
    return l > x ? l : x;
}
template <int W>
__host__ __device__ inline size_t pair_lds_bytes(int N, bool perm) {
    return lists_bytes<W>(N) + (size_t)N * 4 + (size_t)N * 4 + (size_t)Pair<W>::kTab * 4 + (perm ? (size_t)N * 2 : 0);
}
template <int W>
__device__ __forceinline__ PairLds pair_lds(void *raw, int N) {
    PairLds s;
    s.lists = reinterpret_cast<int2 *>(raw);
    s.eps = reinterpret_cast<int *>((char *)raw + lists_bytes<W>(N));
    s.yrank = reinterpret_cast<uint16_t *>(s.eps + N);
    s.other = s.yrank + N;
    s.Tx = s.other + N;
    s.Ty = s.Tx + Pair<W>::kTab;
    s.perm = s.Ty + Pair<W>::kTab;
    return s;
}

// One pair's samples as a thread holds them on entry: x-order sample p = tid + kT i has
// code x[i] and the spread sx[i] of its nearest codes in x; y-order sample j = tid + kT i
// has code y[i], the x code xj[i] and the x-order position pj[i].
struct Samples {
    int x[kPer], sx[kPer], y[kPer], xj[kPer], pj[kPer];
};

constexpr int kSpread = 16;  // the spread of a sample's 2 kSpread nearest codes predicts its
                             // walk's strip (4 % fewer steps than with the k nearest)

__device__ __forceinline__ int spread_at(const int *a, int p, int N) {
    return a[min(p + kSpread, N - 1)] - a[max(p - kSpread, 0)];
}

// Exclusive prefix over the chunk counts c[0 .. C): lane l of every wave gets its own.
template <int C>
__device__ __forceinline__ int chunk_prefix(const int *c) {
    const int lane = threadIdx.x & 63;
    const int v = lane < C ? c[lane] : 0;
    int s = v;
#pragma unroll
    for (int d = 1; d < C; d <<= 1) {
        const int t = __shfl_up(s, d);
        if (lane >= d) s += t;
    }
    return s - v;
}

__device__ __forceinline__ int mask_below(uint64_t m) {  // set bits below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

constexpr int kRefill = 16;  // idle lanes that start new walks together

// Neighbour search and counts for all samples of one pair.  Returns the FP64 sum of
// H_nx + H_ny over all samples in every thread; perm[p] = member of x-order sample p
// (read only for cnt).  Tx is built here from xs = (int *)lists when build_tx, else it
// is already complete.
//
// Lists: sample p's place in its half of the x order is the number of earlier samples
// of the same half (a ballot per 64 samples and a prefix over the chunk counts); its
// place in the other half is p minus that, so a change of lists needs no search.
//
// Walk phase: the x order is dealt to the waves in chunks of 64 samples, the middle
// chunks first (the samples at the ends of an order have short walks, which then fill
// the end of the phase).  A lane walks one sample at a time; once kRefill lanes of the
// wave have finished, they change lists or take the wave's next unclaimed samples
// (handed out in lane order from a wave-uniform counter), so short and long walks do
// not wait for each other.
// A walk takes 4 samples per side per step; a side stops once the farthest of
// its 4 is at least the current k-th distance away along the walked coordinate
// (always so for a sentinel, as the k-th distance starts at kUnset).  Samples
// past that point never change the k smallest, so the overscan is harmless; a
// block starts at most 3 samples past the last real one, and a stopped side
// reads a block of sentinels, so reads stay within the lists.  A step has no branch:
// a lane whose walk is over reads sentinels on both sides, which change nothing, and
// which lanes still walk is a ballot of two comparisons, so the bookkeeping is scalar.
// Where a walk starts and ends, and why it cannot leave the lists: ksg_lists.hpp.
// Count phase: thread t takes samples t, t + kT, ... and counts the marginals
// by bucket table and binary search; the partial sums are combined in a fixed
// order, so the FP64 total is reproducible.
// nx0: the x order's split_rank.
template <int K, int W>
__device__ double ksg_pair(const PairLds &S, const Samples &s, int N, int nx0,
                           const uint16_t *__restrict__ perm, int32_t *__restrict__ cnt,
                           bool build_tx) {
    typedef Pair<W> G;
    constexpr int T = G::kT, C = G::kChunks;
    __shared__ double s_part[W];
    __shared__ int s_cy[C], s_cx[C];   // samples of the upper half per chunk of an order
    __shared__ int s_edge[4];          // x at ranks nx0 - 1, nx0; y at ny0 - 1, ny0
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int LY = list_entries(N);    // first entry of the y order's lists

    // y codes in y order, y ranks, halves of the y order
    uint64_t my[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int j = tid + T * i;
        if (j < N) {
            S.eps[j] = s.y[i];
            S.yrank[s.pj[i]] = (uint16_t)j;
            if (j == nx0 - 1 || j == nx0) s_edge[j - nx0 + 1] = s.x[i];  // j: rank of the x order
        }
        my[i] = __ballot(j < N && s.pj[i] >= nx0);
        if (lane == 0) s_cy[i * W + wave] = __popcll(my[i]);
    }
    tab_fill<W>(S.Ty, N);
    if (build_tx) tab_fill<W>(S.Tx, N);
    __syncthreads();

    // the y order's lists; the x order's halves
    const int ny0 = __builtin_amdgcn_readfirstlane(split_rank(S.eps, N));
    if (tid < 2) s_edge[2 + tid] = S.eps[ny0 - 1 + tid];
    const int py = chunk_prefix<C>(s_cy);
    int yv[kPer], jr[kPer];
    uint64_t mx[kPer];
    uint32_t in_y = 0;  // bit i: sample i walks the y order
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int p = tid + T * i;
        const int q1 = __builtin_amdgcn_readlane(py, i * W + wave) + mask_below(my[i]);
        if (p < N) {  // here p is a rank of the y order
            const int at = LY + list_place(s.pj[i] >= nx0, p, q1, nx0, N - nx0);
            S.lists[kPad + at] = make_int2(s.y[i], s.xj[i]);
            S.other[s.pj[i]] = (uint16_t)at;
        }
        jr[i] = p < N ? min((int)S.yrank[p], N - 1) : 0;
        yv[i] = S.eps[jr[i]];
        if (p < N && spread_at(S.eps, jr[i], N) > s.sx[i]) in_y |= 1u << i;
        mx[i] = __ballot(p < N && jr[i] >= ny0);
        if (lane == 0) s_cx[i * W + wave] = __popcll(mx[i]);
    }
    tab_scatter<W>(S.eps, S.Ty, N);
    if (build_tx) tab_scatter<W>(reinterpret_cast<const int *>(S.lists), S.Tx, N);
    __syncthreads();

    // the x order's lists, the sentinels, the walk starts
    const int px = chunk_prefix<C>(s_cx);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int p = tid + T * i;
        const int q1 = __builtin_amdgcn_readlane(px, i * W + wave) + mask_below(mx[i]);
        if (p < N) {
            const bool up = jr[i] >= ny0;
            const int at = list_place(up, p, q1, ny0, N - ny0);
            S.lists[kPad + at] = make_int2(s.x[i], yv[i]);
            int start = at, sum = place_sum(0, ny0, p);
            int gap = up ? yv[i] - s_edge[2] : s_edge[3] - yv[i];
            if (in_y >> i & 1) {
                start = S.other[p];
                sum = place_sum(LY, nx0, jr[i]);
                gap = p >= nx0 ? s.x[i] - s_edge[0] : s_edge[1] - s.x[i];
            }
            S.other[p] = (uint16_t)walk_other(sum - start, LY);
            S.eps[p] = (int)pack_start(start, gap);
        }
    }
    if (tid < 8 * kPad) {
        // pads 0..3 of each order: left and right of the two lists
        const int pad = (tid >> 2) & 3, u = tid & 3;
        const int n0 = tid >= 4 * kPad ? nx0 : ny0;
        const int at = pad_place(pad, tid >= 4 * kPad ? LY : 0, n0, N - n0) + u;
        S.lists[at] = make_int2(pad_code(pad), 0);
    }
    if (wave == 0) tab_scan<W>(S.Ty);
    if (build_tx && wave == (W > 1 ? 1 : 0)) tab_scan<W>(S.Tx);
    __syncthreads();

    // ---- walks
    typedef __attribute__((address_space(3))) const i32x2 lds_int2;
    lds_int2 *const base = (lds_int2 *)reinterpret_cast<i32x2 *>(S.lists);
    lds_int2 *const endL = base;                  // four sentinels: a finished left side
    lds_int2 *const endR = base + pad_place(3, 0, ny0, N - ny0);  // ... and right side
    const int nchunks = (N + 63) >> 6;
    const int mine = 64 * ((nchunks - wave + W - 1) / W);  // this wave's share, whole chunks
    // first sample of the wave's ci-th chunk, from the middle outwards; the partial
    // chunk, the last one, comes last
    auto chunk0 = [&](int ci) {
        const int g = ci * W + wave, h = (g + 1) >> 1;
        return 64 * (((nchunks - 1) >> 1) + (((g ^ nchunks) & 1) ? h : -h));
    };
    int p = 0, gap = 0;
    i32x2 me = {0, 0};
    lds_int2 *L = endL, *R = endR;
    int best[K];
#pragma unroll
    for (int t = 0; t < K; ++t) best[t] = kUnset;
    int next = 0;  // first unclaimed sample of the wave
    // the lanes of `idle` take the wave's next samples; returns those that got one
    auto claim = [&](uint64_t idle) {
        const int i = next + mask_below(idle), ci = next >> 6;
        const int a0 = chunk0(ci), a1 = chunk0(ci + 1);
        const int np = (i & 63) + ((i >> 6) == ci ? a0 : a1);
        const uint64_t got = idle & __ballot(i < mine && np < N);
        next += __popcll(idle);
        if (__builtin_amdgcn_inverse_ballot_w64(got)) {
            p = np;
            const uint32_t info = (uint32_t)S.eps[p];
            lds_int2 *at = base + kPad + walk_place(start_place(info), LY);
            gap = start_gap(info);
            me = *at;
            me.x = walk_code(me.x);
            L = at - 4;
            R = at + 1;
#pragma unroll
            for (int t = 0; t < K; ++t) best[t] = kUnset;
        }
        return got;
    };
    uint64_t have = claim(~0ull), run = have;  // lanes with a sample; lanes still walking
    while (have) {
        const uint64_t fin = have & ~run;
        // a batch of list changes and claims costs its instructions once for its lanes
        if (__popcll(fin) >= kRefill || !run) {
            // nearer to the other list than to the k-th neighbour: go on there
            const uint64_t more = fin & __ballot(gap < best[K - 1]);
            if (__builtin_amdgcn_inverse_ballot_w64(more)) {
                R = base + kPad + S.other[p];
                L = R - 4;
                gap = kUnset;  // no third list
            }
            const uint64_t done = fin & ~more;
            if (__builtin_amdgcn_inverse_ballot_w64(done)) S.eps[p] = best[K - 1];
            have &= ~done;
            if (next < mine) have |= claim(done);
            if (!have) break;
        }
        i32x2 c[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = L[u];
            c[4 + u] = R[u];
        }
#pragma unroll
        for (int u = 3; u >= 0; --u)
            insert_k<K>(best, max(me.x - c[u].x, absdiff_u32(me.y, c[u].y)));
#pragma unroll
        for (int u = 0; u < 4; ++u)
            insert_k<K>(best, max(c[4 + u].x - me.x, absdiff_u32(me.y, c[4 + u].y)));
        // a side goes on while its farthest sample is nearer than the k-th
        // distance (never for a sentinel, never past the padding)
        const bool al = (me.x - c[0].x) < best[K - 1];
        const bool ar = (c[7].x - me.x) < best[K - 1];
        L = al ? L - 4 : endL;
        R = ar ? R + 4 : endR;
        run = __ballot(al) | __ballot(ar);
    }
    __syncthreads();

    // ---- counts, over the sorted codes
    int *xs = reinterpret_cast<int *>(S.lists) + 1, *ys = xs + N;  // xs[-1] is readable
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int p = tid + T * i;
        if (p < N) {
            xs[p] = s.x[i];
            ys[p] = s.y[i];
        }
    }
    __syncthreads();
    double acc = 0.0;
    for (int i = 0; i < kPer; ++i) {
        const int pp = tid + T * i;
        if (pp >= N) break;
        const int eps = S.eps[pp];
        int nx = 0, ny = 0;
        if (eps > 0)
            marginal_counts<W>(xs, ys, S.Tx, S.Ty, xs[pp], ys[min((int)S.yrank[pp], N - 1)], eps,
                               nx, ny);
        nx = min(max(nx, 0), N - 1);  // no-ops on sorted orders; keep H reads in bounds
        ny = min(max(ny, 0), N - 1);
        acc += kHarmonic.v[nx] + kHarmonic.v[ny];
        if (cnt) {
            const int m = order_member(perm[pp], N);
            cnt[m] = nx;
            cnt[N + m] = ny;
        }
    }
    acc = wave_sum_f64(acc);
    if (lane == 0) s_part[wave] = acc;
    __syncthreads();
    double total = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) total += s_part[w];
    return total;
}

// Ascending bitonic sort of kPer T keys held kPer per thread in registers (thread t
// holds keys kPer t .. kPer t + kPer - 1).  Compare-exchange partners closer than kPer
// are in the thread's own registers, partners up to 64 kPer apart are in the same wave
// (lane shuffles), and only larger strides go through LDS (xchg, kPer T keys).
template <int W>
__device__ __forceinline__ void block_sort_regs(unsigned long long (&k)[kPer],
                                                unsigned long long *xchg) {
    const int tid = threadIdx.x;
    constexpr int E = kPer, PT = Pair<W>::kMax;
    for (int size = 2; size <= PT; size <<= 1) {
        for (int stride = size >> 1; stride >= E; stride >>= 1) {
            const bool cross = stride >= 64 * E;
            if (cross) {
                __syncthreads();
#pragma unroll
                for (int j = 0; j < E; ++j) xchg[E * tid + j] = k[j];
                __syncthreads();
            }
            // the lower index of a pair keeps the smaller key in an ascending
            // block; stride >= E, so that is the same for all E keys of a thread
            const bool keep_min = ((E * tid & stride) == 0) == ((E * tid & size) == 0);
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const int i = E * tid + j;
                const unsigned long long o =
                    cross ? xchg[i ^ stride] : __shfl_xor(k[j], stride / E, kWave);
                // equal keys are interchangeable, so one comparison decides
                k[j] = ((o < k[j]) == keep_min) ? o : k[j];
            }
        }
#pragma unroll
        for (int st = E / 2; st >= 1; st >>= 1) {
            if (st >= size) continue;
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const int jp = j ^ st;
                if (jp < j) continue;
                const bool up = ((E * tid + j) & size) == 0;
                const unsigned long long a = k[j], b = k[jp];
                const bool swap = (a > b) == up;
                k[j] = swap ? b : a;
                k[jp] = swap ? a : b;
            }
        }
    }
    __syncthreads();  // xchg may be reused by the caller
}

// m[i] = member of rank tid + kT i of a column: its stored order, or (order null) the
// column sorted here by (code, member) through `scratch` (lists_bytes).
template <int W>
__device__ __forceinline__ void sorted_members(const int32_t *__restrict__ c,
                                               const uint16_t *__restrict__ order, int N,
                                               void *scratch, int (&m)[kPer]) {
    const int tid = threadIdx.x;
    constexpr int T = Pair<W>::kT;
    if (order) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int r = tid + T * i;
            m[i] = r < N ? order_member(order[r], N) : 0;
        }
        return;
    }
    unsigned long long k[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int r = kPer * tid + j;
        k[j] = r < N ? (((unsigned long long)(uint32_t)c[r]) << 16) | (unsigned)r : ~0ull;
    }
    block_sort_regs<W>(k, reinterpret_cast<unsigned long long *>(scratch));
    uint16_t *list = reinterpret_cast<uint16_t *>(scratch);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int r = kPer * tid + j;
        if (r < N) list[r] = (uint16_t)(k[j] & 0xffff);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) m[i] = tid + T * i < N ? (int)list[tid + T * i] : 0;
    __syncthreads();
}

// ----------------------------------------------------------- field mode ----
// Prologue: for each reference (64 per launch, as a kernel argument), its codes in
// ascending (code, member) order, the member permutation and its inverse, and its
// entry of the reference list.
constexpr int kSortRefs = 64;
struct SortRefs {
    int64_t v[kSortRefs];
};

__global__ void ksg_sort_ref_kernel(const int32_t *__restrict__ code,
                                    const uint16_t *__restrict__ order, int N, SortRefs rs,
                                    int64_t *__restrict__ refs, int32_t *__restrict__ xs,
                                    uint16_t *__restrict__ perm, uint16_t *__restrict__ invp) {
    extern __shared__ unsigned long long s_keys[];
    const int r = blockIdx.x;
    const int P = pow2_ceil(N);
    const int64_t v = rs.v[r];
    const int32_t *c = code + v * N;
    if (threadIdx.x == 0) refs[r] = v;
    if (order) {  // the column's stored order
        const uint16_t *o = order + v * N;
        for (int p = threadIdx.x; p < N; p += kKsgThreads) {
            const int m = order_member(o[p], N);
            xs[(int64_t)r * N + p] = c[m];
            perm[(int64_t)r * N + p] = (uint16_t)m;
            invp[(int64_t)r * N + m] = (uint16_t)p;
        }
    } else {
        for (int m = threadIdx.x; m < P; m += kKsgThreads)
            s_keys[m] = m < N ? (((unsigned long long)(uint32_t)c[m]) << 16) | (unsigned)m : ~0ull;
        __syncthreads();
        block_bitonic_sort(s_keys, P);
        for (int p = threadIdx.x; p < N; p += kKsgThreads) {
            const int m = (int)(s_keys[p] & 0xffff);
            xs[(int64_t)r * N + p] = (int32_t)(s_keys[p] >> 16);
            perm[(int64_t)r * N + p] = (uint16_t)m;
            invp[(int64_t)r * N + m] = (uint16_t)p;
        }
    }
}

// Waves per SIMD the registers are held to: of E = 16 four waves cover the LDS latencies
// better than three of 144 registers (3.31 -> 2.95 ms before code 0 had its own bucket);
// five and more spill (12 ms).
constexpr int order_waves(int E) { return E == 16 ? 4 : 1; }

// One column per wave, N <= 64 E.  Bound by VALU issue (787 per column of 1000 members)
// and LDS beside 6 B/sample of HBM: 1.76M columns of 1000 members 9.56 -> 3.1 ms
// (3.4 TB/s) against a register bitonic sort of every column, 704,000 of 2048 members (1966
// VALU) 7.8 ms.  Holding the place in the code's word and reading the counters twice took
// fewer registers, but more LDS: 3.3 against 2.95 ms then.
template <int E>
__global__ __launch_bounds__(kKsgThreads, order_waves(E)) void ksg_order_kernel(const int32_t *__restrict__ code,
                                                                int N, int64_t ncol,
                                                                uint16_t *__restrict__ order) {
    __shared__ __attribute__((aligned(16))) uint32_t s_lds[kKsgWaves][ColumnSort<E>::kLds];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * kKsgWaves;
    for (int64_t v = (int64_t)blockIdx.x * kKsgWaves + wave; v < ncol; v += waves)
    {
        uint32_t c[E];
        load_codes<E>(code + v * N, N, c);
        wave_sort_codes<E, ColumnSort<E>::kLowMask>(c, N, order + v * N, s_lds[wave]);
    }
}

// N > 2048 (no KSG call takes such columns): one column per workgroup, in LDS.
__global__ __launch_bounds__(kKsgThreads) void ksg_order_block_kernel(
    const int32_t *__restrict__ code, int N, int64_t ncol, uint16_t *__restrict__ order) {
    extern __shared__ unsigned long long s_x[];
    const int P = pow2_ceil(N);
    for (int64_t v = blockIdx.x; v < ncol; v += gridDim.x) {
        const int32_t *c = code + v * N;
        uint16_t *o = order + v * N;
        for (int m = threadIdx.x; m < P; m += kKsgThreads)
            s_x[m] = m < N ? (((unsigned long long)(uint32_t)c[m]) << 16) | (unsigned)m : ~0ull;
        __syncthreads();
        block_bitonic_sort(s_x, P);
        for (int p = threadIdx.x; p < N; p += kKsgThreads) o[p] = (uint16_t)(s_x[p] & 0xffff);
        __syncthreads();
    }
}

template <int K, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(6))) void ksg_field_kernel(
    const int32_t *__restrict__ code_q, const int32_t *__restrict__ flags_r,
    const int32_t *__restrict__ flags_q, int N, int64_t V, const int64_t *__restrict__ refs,
    int n_ref, const int32_t *__restrict__ xs_all, const uint16_t *__restrict__ perm_all,
    float *__restrict__ out, int32_t *__restrict__ counts, const int32_t *__restrict__ code_r,
    const uint16_t *__restrict__ order_q, const uint16_t *__restrict__ invp_all) {
    extern __shared__ int4 s_raw[];
    constexpr int T = Pair<W>::kT;
    const PairLds S = pair_lds<W>(s_raw, N);
    const int tid = threadIdx.x;
    const double base = kHarmonic.v[K - 1] + kHarmonic.v[N - 1];

    for (int r = 0; r < n_ref; ++r) {
        const int32_t fr = flags_r[refs[r]];
        const int32_t *xs = xs_all + (int64_t)r * N;
        const uint16_t *invp = invp_all + (int64_t)r * N, *perm = perm_all + (int64_t)r * N;
        const int32_t *cr = code_r + refs[r] * N;
        // the reference's codes in its own order and its bucket table, shared by all
        // its queries
        Samples s;
        int *xl = reinterpret_cast<int *>(S.lists);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = tid + T * i;
            s.x[i] = p < N ? xs[p] : 0;
            if (p < N) xl[p] = s.x[i];
        }
        tab_fill<W>(S.Tx, N);
        __syncthreads();
        tab_scatter<W>(xl, S.Tx, N);
#pragma unroll
        for (int i = 0; i < kPer; ++i) s.sx[i] = spread_at(xl, min(tid + T * i, N - 1), N);
        const int nx0 = __builtin_amdgcn_readfirstlane(split_rank(xl, N));
        __syncthreads();
        if (tid < 64) tab_scan<W>(S.Tx);
        __syncthreads();
        for (int64_t q = blockIdx.x; q < V; q += gridDim.x) {
            const int32_t *cq = code_q + q * N;
            const int32_t fq = flags_q[q];
            int32_t *cnt = counts ? counts + ((int64_t)r * V + q) * 2 * N : nullptr;
            if ((fr | fq) & (NDF_FLAG_CONSTANT | NDF_FLAG_NONFINITE)) {
                if (tid == 0)
                    out[(int64_t)r * V + q] = ((fr | fq) & NDF_FLAG_NONFINITE) ? __builtin_nanf("")
                                                                                : 0.0f;
                if (cnt)
                    for (int i = tid; i < 2 * N; i += T) cnt[i] = 0;
                continue;
            }
            int m[kPer];
            sorted_members<W>(cq, order_q ? order_q + q * N : nullptr, N, S.lists, m);
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                s.y[i] = cq[m[i]];
                s.xj[i] = cr[m[i]];
                s.pj[i] = min((int)invp[m[i]], N - 1);
            }
            const double acc = ksg_pair<K, W>(S, s, N, nx0, perm, cnt, false);
            if (tid == 0) out[(int64_t)r * V + q] = (float)(base - acc / (double)N);
        }
    }
}

// ----------------------------------------------------------- pairs mode ----
template <int K, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(6))) void ksg_pairs_kernel(
    const int32_t *__restrict__ code_a, const int32_t *__restrict__ code_b,
    const int32_t *__restrict__ flags_a, const int32_t *__restrict__ flags_b, int N, int64_t V,
    const int64_t *__restrict__ pairs, int64_t B, float *__restrict__ out,
    int32_t *__restrict__ counts, const uint16_t *__restrict__ order_a,
    const uint16_t *__restrict__ order_b) {
    extern __shared__ int4 s_raw[];
    constexpr int T = Pair<W>::kT;
    const PairLds S = pair_lds<W>(s_raw, N);
    const int tid = threadIdx.x;
    const double base = kHarmonic.v[K - 1] + kHarmonic.v[N - 1];

    for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
        const int64_t va = pairs[2 * b], vb = pairs[2 * b + 1];
        int32_t *cnt = counts ? counts + b * 2 * N : nullptr;
        if (va < 0 || va >= V || vb < 0 || vb >= V) {  // out-of-range pair: NaN, no reads
            if (tid == 0) out[b] = __builtin_nanf("");
            if (cnt)
                for (int i = tid; i < 2 * N; i += T) cnt[i] = -1;
            continue;
        }
        const int32_t f = flags_a[va] | flags_b[vb];
        if (f & (NDF_FLAG_CONSTANT | NDF_FLAG_NONFINITE)) {
            if (tid == 0) out[b] = (f & NDF_FLAG_NONFINITE) ? __builtin_nanf("") : 0.0f;
            if (cnt)
                for (int i = tid; i < 2 * N; i += T) cnt[i] = 0;
            continue;
        }
        const int32_t *ca = code_a + va * N, *cb = code_b + vb * N;
        Samples s;
        int ma[kPer], mb[kPer];
        const uint16_t *perm = order_a ? order_a + va * N : S.perm;
        sorted_members<W>(ca, order_a ? order_a + va * N : nullptr, N, S.lists, ma);
        if (cnt && !order_a)
            for (int i = 0; i < kPer; ++i)
                if (tid + T * i < N) S.perm[tid + T * i] = (uint16_t)ma[i];
        sorted_members<W>(cb, order_b ? order_b + vb * N : nullptr, N, S.lists, mb);
        // xs and the inverse x permutation in the lists' region until they are written
        int *xl = reinterpret_cast<int *>(S.lists);
        uint16_t *inv = reinterpret_cast<uint16_t *>(xl + N);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = tid + T * i;
            s.x[i] = ca[ma[i]];
            if (p < N) {
                xl[p] = s.x[i];
                inv[ma[i]] = (uint16_t)p;
            }
            s.y[i] = cb[mb[i]];
            s.xj[i] = ca[mb[i]];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            s.sx[i] = spread_at(xl, min(tid + T * i, N - 1), N);
            s.pj[i] = min((int)inv[mb[i]], N - 1);
        }
        const int nx0 = __builtin_amdgcn_readfirstlane(split_rank(xl, N));
        const double acc = ksg_pair<K, W>(S, s, N, nx0, perm, cnt, true);
        if (tid == 0) out[b] = (float)(base - acc / (double)N);
    }
}

// ------------------------------------------------------------ launchers ----
static int p2(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// Workspace: FP64 [N + 1] (unused: the harmonic numbers are a constant; the size stays what
// callers have laid out) | refs |
// x codes in x order [n_ref][N] | x-order members [n_ref][N] | inverse x permutation
// [n_ref][N].
size_t ksg_field_ws_bytes(int N, int n_ref) {
    return align_up((size_t)(N + 1) * sizeof(double), 256) +
           align_up((size_t)n_ref * sizeof(int64_t), 256) +
           align_up((size_t)n_ref * N * sizeof(int32_t), 256) +
           2 * align_up((size_t)n_ref * N * sizeof(uint16_t), 256);
}

// Grid of a striding kernel: `rounds` times as many workgroups of `waves` waves as the
// CUs hold at once given the LDS of one item (160 KB per CU), never more than there are
// items.  Items differ in cost (walk lengths) and CUs in speed, so a grid of
// only resident workgroups ends with a tail of the slowest ones; a larger grid
// lets the hardware hand the waiting workgroups to whichever CU frees up first
// (measured on a KSG field of 50 ms: 20 % longer with 1 round of workgroups than with
// 16).  Every workgroup of a field first loads its reference and writes its register
// spills once, so a field takes 16 rounds (1000 members x 1.76M vertices: the same time
// as 64 with 1.3 GB less written); pairs take 64 (2^18 pairs: 0.7 % faster than 16).
static int ksg_grid(int64_t items, size_t lds, int waves, int rounds) {
    int64_t per_cu = (int64_t)(163840 / (lds > 0 ? lds : 1));
    const int64_t cap = 32 / waves;
    per_cu = per_cu < 1 ? 1 : (per_cu > cap ? cap : per_cu);
    const int64_t g = 256 * per_cu * rounds;
    return (int)(items < g ? items : g);
}
constexpr int kFieldRounds = 16;
constexpr int kPairRounds = 64;
constexpr int kOrderRounds = 16;

// f(waves as a constant) for N members: one wave per 256
template <typename F>
static void with_pair_waves(int N, F f) {
    if (N <= Pair<1>::kMax)
        f(std::integral_constant<int, 1>{});
    else if (N <= Pair<2>::kMax)
        f(std::integral_constant<int, 2>{});
    else if (N <= Pair<4>::kMax)
        f(std::integral_constant<int, 4>{});
    else
        f(std::integral_constant<int, 8>{});
}

// f(k as a constant), 1 <= k <= 8
template <typename F>
static void with_k(int k, F f) {
    switch (k) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
        default: f(std::integral_constant<int, 8>{}); break;
    }
}

// Sorted member orders of every column of every variable (ndf_prepare).
int launch_ksg_orders(const ndf_ensemble *e, hipStream_t st) {
    const int N = e->n_members;
    const int64_t ncol = (int64_t)e->n_vars * e->nx * e->ny * e->nz;
    if (N > 2048) {
        const size_t lds = (size_t)p2(N) * sizeof(unsigned long long);
        hipLaunchKernelGGL(ksg_order_block_kernel,
                           dim3((unsigned)ksg_grid(ncol, lds, kKsgWaves, kOrderRounds)), dim3(kKsgThreads),
                           lds, st, e->code, N, ncol, e->order);
        return status_of_launch();
    }
    const int64_t wgs = ceil_div(ncol, kKsgWaves);
    const int64_t cap = 256 * 8 * kOrderRounds;
    const dim3 g((unsigned)(wgs < cap ? wgs : cap));
#define NDF_ORDER_CASE(E)                                                                    \
    if (N <= 64 * E) {                                                                       \
        hipLaunchKernelGGL(ksg_order_kernel<E>, g, dim3(kKsgThreads), 0, st, e->code, N, ncol, \
                           e->order);                                                        \
        return status_of_launch();                                                           \
    }
    NDF_ORDER_CASE(1) NDF_ORDER_CASE(2) NDF_ORDER_CASE(4)
    NDF_ORDER_CASE(8) NDF_ORDER_CASE(16) NDF_ORDER_CASE(32)
#undef NDF_ORDER_CASE
    return NDF_E_UNSUPPORTED;
}

int launch_ksg_field(const ndf_ensemble *e, int var_ref, int var_qry, const int64_t *ref_v,
                     int n_ref, int k, float *out, int32_t *counts, void *ws, hipStream_t st) {
    const int N = e->n_members;
    if (N > kKsgMaxN || k < 1 || k > 8) return NDF_E_UNSUPPORTED;
    const int64_t V = (int64_t)e->nx * e->ny * e->nz;
    char *w = (char *)ws + align_up((size_t)(N + 1) * sizeof(double), 256);
    int64_t *refs = (int64_t *)w;
    w += align_up((size_t)n_ref * sizeof(int64_t), 256);
    int32_t *xs = (int32_t *)w;
    w += align_up((size_t)n_ref * N * sizeof(int32_t), 256);
    uint16_t *perm = (uint16_t *)w;
    w += align_up((size_t)n_ref * N * sizeof(uint16_t), 256);
    uint16_t *invp = (uint16_t *)w;
    const int32_t *cr = e->code + (int64_t)var_ref * V * N;
    const int32_t *cq = e->code + (int64_t)var_qry * V * N;
    const int32_t *fr = e->flags + (int64_t)var_ref * V, *fq = e->flags + (int64_t)var_qry * V;
    const uint16_t *ordr = e->order ? e->order + (int64_t)var_ref * V * N : nullptr;
    const uint16_t *ordq = e->order ? e->order + (int64_t)var_qry * V * N : nullptr;
    for (int r0 = 0; r0 < n_ref; r0 += kSortRefs) {
        const int n = n_ref - r0 < kSortRefs ? n_ref - r0 : kSortRefs;
        SortRefs rs{};
        for (int i = 0; i < n; ++i) rs.v[i] = ref_v[r0 + i];
        const int64_t o = (int64_t)r0 * N;
        hipLaunchKernelGGL(ksg_sort_ref_kernel, dim3(n), dim3(kKsgThreads),
                           ordr ? 0 : (size_t)p2(N) * 8, st, cr, ordr, N, rs, refs + r0, xs + o,
                           perm + o, invp + o);
    }
    with_pair_waves(N, [&](auto wc) {
        constexpr int W = decltype(wc)::value;
        const size_t lds = pair_lds_bytes<W>(N, false);
        const dim3 g((unsigned)ksg_grid(V, lds, W, kFieldRounds));
        with_k(k, [&](auto kc) {
            constexpr int K = decltype(kc)::value;
            hipLaunchKernelGGL((ksg_field_kernel<K, W>), g, dim3(64 * W), lds, st, cq, fr, fq, N, V,
                               refs, n_ref, xs, perm, out, counts, cr, ordq, invp);
        });
    });
    return status_of_launch();
}

// The pairs kernels keep nothing in a workspace; its size stays what callers have laid out.
size_t ksg_pairs_ws_bytes(int N) { return align_up((size_t)(N + 1) * sizeof(double), 256); }

int launch_ksg_pairs(const ndf_ensemble *e, int var_a, int var_b, const int64_t *pairs, int64_t B,
                     int k, float *out, int32_t *counts, hipStream_t st) {
    const int N = e->n_members;
    if (N > kKsgMaxN || k < 1 || k > 8) return NDF_E_UNSUPPORTED;
    const int64_t V = (int64_t)e->nx * e->ny * e->nz;
    const int32_t *ca = e->code + (int64_t)var_a * V * N;
    const int32_t *cb = e->code + (int64_t)var_b * V * N;
    const int32_t *fa = e->flags + (int64_t)var_a * V;
    const int32_t *fb = e->flags + (int64_t)var_b * V;
    const uint16_t *oa = e->order ? e->order + (int64_t)var_a * V * N : nullptr;
    const uint16_t *ob = e->order ? e->order + (int64_t)var_b * V * N : nullptr;
    with_pair_waves(N, [&](auto wc) {
        constexpr int W = decltype(wc)::value;
        const size_t lds = pair_lds_bytes<W>(N, counts && !oa);
        const dim3 g((unsigned)ksg_grid(B, lds, W, kPairRounds));
        with_k(k, [&](auto kc) {
            constexpr int K = decltype(kc)::value;
            hipLaunchKernelGGL((ksg_pairs_kernel<K, W>), g, dim3(64 * W), lds, st, ca, cb, fa, fb, N,
                               V, pairs, B, out, counts, oa, ob);
        });
    });
    return status_of_launch();
}

}  // namespace ndf
