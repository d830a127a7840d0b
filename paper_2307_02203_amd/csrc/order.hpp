// Sorted member order of one column of codes by one wave (prepare.hip, ksg.hip).
#pragma once
#include "common.hpp"

namespace ndf {

constexpr int log2_int(int n) { return n <= 1 ? 0 : 1 + log2_int(n / 2); }

// Ascending bitonic sort of 64 E 32-bit keys held E per lane, in the form whose
// merge of two sorted halves starts by comparing element i with its mirror
// i ^ (size - 1): every comparator then puts the minimum at the lower index, so a
// pair in one lane is one v_min and one v_max, and a pair across lanes one lane
// shuffle plus a min or max.  The stages are template instances: a loop over them that
// the compiler leaves rolled (E = 32) indexes the registers at run time (2048 members
// 200 us a column).
template <int E>
__device__ __forceinline__ void sort_in_lane(uint32_t (&k)[E], int mask) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int jp = j ^ mask;
        if (jp > j) {
            const uint32_t a = k[j], b = k[jp];
            k[j] = min(a, b);
            k[jp] = max(a, b);
        }
    }
}
// Strides 2^LS2, 2^(LS2 - 1), ..., 1 of a merge.
template <int E, int LS2>
__device__ __forceinline__ void sort_strides(uint32_t (&k)[E]) {
    constexpr int stride = 1 << LS2;
    if constexpr (stride >= E) {
        const bool lower = ((E * (threadIdx.x & 63)) & stride) == 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const uint32_t o = __shfl_xor(k[j], stride / E, kWave);
            k[j] = lower ? min(k[j], o) : max(k[j], o);
        }
    } else {
        sort_in_lane<E>(k, stride);
    }
    if constexpr (LS2 > 0) sort_strides<E, LS2 - 1>(k);
}
// Merges into sorted runs of 2^LS keys, then the longer ones.
template <int E, int LS = 1>
__device__ __forceinline__ void wave_sort_regs32(uint32_t (&k)[E]) {
    constexpr int size = 1 << LS;
    if constexpr (size <= E) {
        sort_in_lane<E>(k, size - 1);
    } else {
        // partner of (lane, j) is (lane ^ (size / E - 1), E - 1 - j)
        const bool lower = ((E * (threadIdx.x & 63)) & (size >> 1)) == 0;
        uint32_t t[E];
#pragma unroll
        for (int j = 0; j < E; ++j) t[j] = __shfl_xor(k[E - 1 - j], size / E - 1, kWave);
#pragma unroll
        for (int j = 0; j < E; ++j) k[j] = lower ? min(k[j], t[j]) : max(k[j], t[j]);
    }
    if constexpr (LS >= 2) sort_strides<E, LS - 2>(k);
    if constexpr (LS < 6 + log2_int(E)) wave_sort_regs32<E, LS + 1>(k);
}

// Sorted member order of one column of N <= 64 E members by one wave, as a bucket
// sort in LDS.  Codes spread over [0, 2^23], so two (E = 32: four) buckets of equal width
// per slot hold one or two samples each: every sample takes a place in its bucket from an
// LDS counter, a scan of the counters gives the bucket starts, and the samples go to LDS in
// bucket order, where lane l then holds positions E l .. E l + E - 1.  Their 32-bit keys
//   (start of the bucket, code bits below the bucket, member)
// order like (code, member), as the start grows with the bucket.  Odd-even passes finish
// the buckets.
// Repeated values crowd their buckets.  Code 0, the column's minimum (fields with many
// zeros), has a bucket of its own, and the counters are taken in member order, so that
// equal codes lie in order as they come.  A column with more than 70 % of its lanes still out
// of order after kLook passes (far outliers: many codes in few buckets) goes through the full
// bitonic sort of the same keys at once, others that need more than odd_even_passes (a full
// sort costs 11 passes at E = 4, 17 to 30 above) then.  ndf_prepare of 80,000 columns, us,
// against a bitonic sort of every column: 200 members smooth 60 (132), 90 % zeros 88 (139),
// lognormal 70 (134), Cauchy 132 (140), one member at 10^4 deviations 164 (147); 1000
// members 284 (659), 447 (681), 351 (672), 606 (732), 740 (720); 2000 members 1491 (3820),
// 1714 (3665), 1734 (3819), 2542 (3818), 2643 (3830).  A look after two passes at more than 16
// lanes, and eight passes, sorted many skewed columns in full that a few passes more
// finish: lognormal 72, 546 and 2435; with no look 2000 members Cauchy took 17,552.
constexpr int kLook = 3;  // passes (each both parities) before the look
// ... and before the full sort at the latest
constexpr int odd_even_passes(int E) { return E <= 4 ? 8 : 12; }

template <int E>
struct ColumnSort {
    static constexpr int kLN = 6 + log2_int(E);          // log2 of the slots
    // 2 buckets per slot; 4 at E = 32 so that start, code bits and member fit 32 bits
    static constexpr int kLB = kLN <= 10 ? kLN + 1 : kLN + 2;
    static constexpr int kLow = 23 - kLB;                // code bits inside a bucket
    static constexpr uint32_t kLowMask = (1u << kLow) - 1;
    static constexpr int kWords = (1 << kLB) / 2;        // two 16-bit counters a word
    static constexpr int kPer = kWords / 64;             // counter words per lane
    static constexpr int kLds = kWords + 4;              // + the last bucket
    static_assert(2 * kLN + kLow <= 32, "key bits");
    static_assert(kWords >= 64 * E, "the keys reuse the counters");
};

__device__ __forceinline__ void wave_lds_fence() {
    // LDS operations of a wave complete in order; this only keeps the compiler from
    // moving them across
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8u __attribute__((ext_vector_type(8), aligned(2)));

// Member of a lane's j-th code: a counter's places then follow the members (in a wave's
// LDS operation the lanes come in order).
__device__ __forceinline__ int sort_member(int j, int lane) { return 64 * j + lane; }

// The codes of a column as wave_sort_codes takes them: code[j] of member sort_member(j).
template <int E>
__device__ __forceinline__ void load_codes(const int32_t *__restrict__ c, int N,
                                           uint32_t (&code)[E]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int m = sort_member(j, lane);
        code[j] = m < N ? (uint32_t)c[m] : 0u;
    }
}

// The sort (codes past N are not read); lds: kLds words of the wave, 16-byte aligned.  ADD:
// kLowMask where the codes come as they are, 0 where the caller has added it.  (Without the
// opaque values below the compiler adds beside every load and waits for one before the
// next: 1000 members 2.8 -> 4.1 ms.  With the bucket formed again at its second use, each
// time in three operations, ndf_prepare of 100 to 1000 members took 1 to 3 % more.)
template <int E, uint32_t ADD>
__device__ __forceinline__ void wave_sort_codes(const uint32_t (&code)[E], int N,
                                                uint16_t *__restrict__ o, uint32_t *lds) {
    typedef ColumnSort<E> C;
    const int lane = threadIdx.x & 63;
    auto member = [&](int j) { return sort_member(j, lane); };
    // codes with kLowMask added: bucket 0 is that of code 0, the next that of codes 1 ..
    // 2^kLow, the last one ends at 2^23
    uint32_t t[E];
    // counters to zero
    for (int i = lane; i < C::kLds / 4; i += 64)
        reinterpret_cast<u32x4v *>(lds)[i] = u32x4v{0u, 0u, 0u, 0u};
    wave_lds_fence();
    // a place in the bucket (16-bit counters: at most 2048 samples)
    uint32_t place[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        // opaque: the addition is not moved up to its load, and t is formed once
        uint32_t c = code[j];
        asm volatile("" : "+v"(c));
        t[j] = min(c + ADD, (1u << 23) + C::kLowMask);
        asm volatile("" : "+v"(t[j]));
        const uint32_t b = t[j] >> C::kLow;
        if (member(j) < N) {
            const uint32_t sh = (b & 1) * 16;
            place[j] = (atomicAdd(&lds[b >> 1], 1u << sh) >> sh) & 0xffffu;
        }
    }
    wave_lds_fence();
    // exclusive scan over the buckets: lane l owns words kPer l .. kPer l + kPer - 1
    uint32_t w[C::kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < C::kPer; ++i) {
        w[i] = lds[C::kPer * lane + i];
        sum += (w[i] & 0xffffu) + (w[i] >> 16);
    }
    uint32_t run = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(run, d, kWave);
        if (lane >= d) run += t;
    }
    if (lane == 63) lds[C::kWords] = run;  // start of the last bucket
    run -= sum;
#pragma unroll
    for (int i = 0; i < C::kPer; ++i) {
        const uint32_t lo = w[i] & 0xffffu, hi = w[i] >> 16;
        lds[C::kPer * lane + i] = run | ((run + lo) << 16);
        run += lo + hi;
    }
    wave_lds_fence();
    uint32_t k[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const uint32_t b = t[j] >> C::kLow;
        const uint32_t start = (lds[b >> 1] >> ((b & 1) * 16)) & 0xffffu;
        place[j] += start;
        k[j] = (start << (C::kLow + C::kLN)) |
               ((t[j] & C::kLowMask) << C::kLN) | (uint32_t)member(j);
    }
    wave_lds_fence();  // every start is read: the keys reuse the counters' LDS
#pragma unroll
    for (int j = 0; j < E; ++j)
        if (member(j) < N) lds[place[j]] = k[j];
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < E; ++j) k[j] = lds[E * lane + j];
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < E; ++j)
        if (E * lane + j >= N) k[j] = 0xffffffffu;  // above every key: sorts last
    int pass = 0;
    for (;; ++pass) {
        const uint32_t nk = __shfl_down(k[0], 1, kWave);
        bool bad = lane < 63 && k[E - 1] > nk;
#pragma unroll
        for (int j = 0; j + 1 < E; ++j) bad |= k[j] > k[j + 1];
        const int far = __popcll(__ballot(bad));
        if (far == 0 || pass == odd_even_passes(E) ||
            (pass == kLook && 10 * E * far > 7 * (N + E - 1))) {
            if (far) wave_sort_regs32<E>(k);
            break;
        }
#pragma unroll
        for (int j = 0; j + 1 < E; j += 2) {  // pairs (2i, 2i + 1) of a lane
            const uint32_t a = k[j], b = k[j + 1];
            k[j] = min(a, b);
            k[j + 1] = max(a, b);
        }
        if constexpr (E == 1) {
            // one key per lane: pairs (2l, 2l + 1), then (2l + 1, 2l + 2)
            const uint32_t p = __shfl_xor(k[0], 1, kWave);
            k[0] = lane & 1 ? max(k[0], p) : min(k[0], p);
            const uint32_t up = __shfl_down(k[0], 1, kWave), dn = __shfl_up(k[0], 1, kWave);
            if (lane & 1) {
                if (lane < 63) k[0] = min(k[0], up);
            } else if (lane > 0) {
                k[0] = max(k[0], dn);
            }
        } else {
            const uint32_t up = __shfl_down(k[0], 1, kWave), dn = __shfl_up(k[E - 1], 1, kWave);
#pragma unroll
            for (int j = 1; j + 1 < E; j += 2) {  // pairs (2i + 1, 2i + 2) of a lane
                const uint32_t a = k[j], b = k[j + 1];
                k[j] = min(a, b);
                k[j + 1] = max(a, b);
            }
            // the pair across a lane boundary
            if (lane < 63) k[E - 1] = min(k[E - 1], up);
            if (lane > 0) k[0] = max(k[0], dn);
        }
    }
    // positions E lane .. E lane + E - 1 of the order
    constexpr uint32_t kMask = (1u << C::kLN) - 1;
    if constexpr (E >= 8) {
#pragma unroll
        for (int j = 0; j < E; j += 8) {
            const int p = E * lane + j;
            if (p + 7 < N) {
                u16x8u q;
#pragma unroll
                for (int e = 0; e < 8; ++e) q[e] = (uint16_t)(k[j + e] & kMask);
                *reinterpret_cast<u16x8u *>(o + p) = q;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (p + e < N) o[p + e] = (uint16_t)(k[j + e] & kMask);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (E * lane + j < N) o[E * lane + j] = (uint16_t)(k[j] & kMask);
    }
}

}  // namespace ndf
