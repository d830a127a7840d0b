// Per-vertex standardisation statistics and KSG integer codes.
//
// Pearson's r (Sec. 3.1, Eq. 1) needs per-vertex means and variances; the KSG
// estimator (Sec. 3.2) compares samples under the max-norm, for which every
// vertex is mapped onto integer codes in [0, 2^23] by min-max normalisation.
// The codes use only correctly rounded IEEE double operations (subtract,
// multiply, divide) and round-half-even, so they are the same integers on any
// conforming implementation; all later KSG distances are exact int32.
//
// Up to 1039 members (prepare_kernel) a workgroup reads its 32 vertices' members once
// and keeps them in registers for both passes (sum / min / max, then centred squares and
// codes); more members, and few without orders, are read twice (prepare_long_kernel).  The ensemble
// is member-major, so each member row contributes a coalesced segment; codes, and the
// vertex-major copy of x where the caller wants one, leave through an LDS transpose.
#include "order.hpp"

#pragma clang fp contract(off)

namespace ndf {

// ------------------------------------------------------- up to 1039 members ----
// Thread (vertex vl, phase ph) of eight waves holds members ph, ph + 16, ... (up to E, and
// one of the last partial row) of vertex vl in registers, every load in flight at once;
// two workgroups of eight waves per CU cover each other's load and coding phases.
// Whole rows are guarded by uniform tests, so no load needs a clamped 64-bit address
// (with one per load and lane the kernel spilled: 4.7 ms).  Bound by HBM: x read once,
// codes written once, past the caches (non-temporal stores: 0.5 ms less), 14.1 GB for
// 1000 members x 1.76M vertices in 3.14 ms, 4.5 TB/s, a large copy's rate (reading x twice
// with 16 loads in flight: 21.1 GB in 5.24 ms).  One workgroup of eight waves with 168
// registers is as fast; eight phases of 128 members each take 5.4 ms.
constexpr int kRegV = 32;        // vertices per workgroup: 128-byte row segments
constexpr int kRegPh = 16;       // member phases
constexpr int kRegThreads = kRegV * kRegPh;
// Workgroups along x, the rest along z: a launch takes fewer than 2^32 threads per axis,
// which 16 per vertex reach at 2^28 vertices.
constexpr int64_t kRegGridX = 1 << 22;

// Rows of the transpose tile: 16 J members of a vertex, padded by four words (the 32
// vertices of a half wave fall into banks 4 apart).
template <int J>
constexpr int prep_row() {
    return kRegPh * J + 4;
}

// dst[v][m] = tile for the members 16 J k .. of the workgroup's vertices: 4 J lanes per
// vertex row, 16 bytes each, at any alignment.
template <int J>
__device__ __forceinline__ void prep_store(const int32_t *tile, int32_t *__restrict__ dst, int N,
                                           int64_t V, int64_t v0, int m0) {
    for (int i = threadIdx.x; i < kRegV * 4 * J; i += kRegThreads) {
        const int row = i / (4 * J), c4 = i % (4 * J);
        const int64_t v = v0 + row;
        const int m = m0 + 4 * c4;
        const int32_t *src = tile + row * prep_row<J>() + 4 * c4;
        if (v >= V || m >= N) continue;
        int32_t *d = dst + v * N + m;
        if (m + 3 < N) {
            const i32x4 q = *reinterpret_cast<const i32x4 *>(src);
            __builtin_nontemporal_store((i32x4u)q, reinterpret_cast<i32x4u *>(d));
        } else {
            for (int e = 0; m + e < N; ++e) d[e] = src[e];
        }
    }
}

template <int E, int OE>
__global__ __launch_bounds__(kRegThreads) __attribute__((amdgpu_waves_per_eu(4))) void
prepare_kernel(const float *__restrict__ x, int N, int64_t V, double *__restrict__ mean,
               double *__restrict__ inv_std, int32_t *__restrict__ code,
               int32_t *__restrict__ flags, int32_t *__restrict__ status,
               float *__restrict__ xt, uint16_t *__restrict__ order) {
    constexpr int J = E < 16 ? E : 16;  // rows of 16 members per transpose tile
    constexpr int K = E / J + 1;        // tiles: E whole rows and a partial one
    constexpr int kCols = kRegV / (kRegThreads / 64);  // columns a wave sorts
    constexpr int kSort = OE ? (kRegThreads / 64) * ColumnSort<OE ? OE : 1>::kLds : 0;
    constexpr int kTile = kRegV * prep_row<J>();
    __shared__ __attribute__((aligned(16))) int32_t s_tile[kTile > kSort ? kTile : kSort];
    __shared__ double s_sum[kRegPh / 2][kRegV];
    __shared__ float s_lo[kRegPh / 2][kRegV], s_hi[kRegPh / 2][kRegV];
    __shared__ int s_bad[kRegPh / 2][kRegV];
    const int var = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int vl = lane & 31, ph = 2 * wave + (lane >> 5);
    const int64_t v0 = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * kRegV, v = v0 + vl;
    if (v0 >= V) return;  // uniform: past the last tile of a grid with several z
    const float *col = x + (int64_t)var * N * V + (v < V ? v : V - 1);

    // every member once: NF whole rows of 16 members, and a row of the remaining ones
    const int NF = N / kRegPh, rem = N % kRegPh;
    const bool has = ph < rem;
    const int64_t step = (int64_t)kRegPh * V;
    col += (int64_t)(has || NF ? ph : 0) * V;
    float a[E], al = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j)
        if (j < NF) a[j] = __builtin_nontemporal_load(col + j * step);
    if (has) al = __builtin_nontemporal_load(col + NF * step);

    // pass 1: sum, min, max, finiteness
    double sum = 0.0;
    float lo = INFINITY, hi = -INFINITY;
    int bad = 0;
    auto accumulate = [&](float q) {
        sum += (double)q;
        lo = fminf(lo, q);
        hi = fmaxf(hi, q);
        bad |= !isfinite(q);
    };
#pragma unroll
    for (int j = 0; j < E; ++j)
        if (j < NF) accumulate(a[j]);
    if (has) accumulate(al);
    // the two phases of a wave, then the eight waves
    sum += __shfl_xor(sum, 32);
    lo = fminf(lo, __shfl_xor(lo, 32));
    hi = fmaxf(hi, __shfl_xor(hi, 32));
    bad |= __shfl_xor(bad, 32);
    if (lane < 32) {
        s_sum[wave][vl] = sum;
        s_lo[wave][vl] = lo;
        s_hi[wave][vl] = hi;
        s_bad[wave][vl] = bad;
    }
    __syncthreads();
    sum = 0.0;
#pragma unroll
    for (int p = 0; p < kRegPh / 2; ++p) {
        sum += s_sum[p][vl];
        lo = fminf(lo, s_lo[p][vl]);
        hi = fmaxf(hi, s_hi[p][vl]);
        bad |= s_bad[p][vl];
    }
    const double mu = sum / (double)N;
    const bool flat = !(hi > lo);
    const double dlo = (double)lo;
    const double scale = flat ? 0.0 : 8388608.0 / ((double)hi - dlo);
    __syncthreads();  // s_sum is reused

    // pass 2: centred sum of squares; codes (and x) transposed through LDS into
    // vertex-major rows, 16 J members at a time
    double ss = 0.0;
    int32_t *cv = code + (int64_t)var * V * N;
    int32_t *tv = reinterpret_cast<int32_t *>(xt ? xt + (int64_t)var * V * N : nullptr);
    int32_t *row = s_tile + vl * prep_row<J>() + ph;
    auto encode = [&](float q) {
        const double d = (double)q - mu;
        ss += d * d;
        return flat ? 0 : (int32_t)__builtin_rint(((double)q - dlo) * scale);
    };
    uint32_t sc[kCols][OE ? OE : 1];  // this wave's columns, for wave_sort_codes<OE, 0>
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int m0 = kRegPh * J * k;
        if (m0 >= N) break;  // uniform
        if (k) __syncthreads();
#pragma unroll
        for (int i = 0; i < J; ++i)
            if (J * k + i < E && J * k + i < NF) row[kRegPh * i] = encode(a[J * k + i]);
        const bool tail = has && NF / J == k;
        if (tail) row[kRegPh * (NF - J * k)] = encode(al);
        __syncthreads();
        prep_store<J>(s_tile, cv, N, V, v0, m0);
        if constexpr (OE > 0) {
            constexpr int kTileCodes = kRegPh * J / 64;  // of a lane
            if (kTileCodes * k < OE) {
#pragma unroll
                for (int c = 0; c < kCols; ++c)
#pragma unroll
                    for (int e = 0; e < kTileCodes; ++e)
                        sc[c][kTileCodes * k + e] =
                            (uint32_t)s_tile[(kCols * wave + c) * prep_row<J>() + 64 * e + lane] +
                            ColumnSort<OE>::kLowMask;
            }
        }
        if (tv) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < J; ++i)
                if (J * k + i < E && J * k + i < NF) row[kRegPh * i] = __float_as_int(a[J * k + i]);
            if (tail) row[kRegPh * (NF - J * k)] = __float_as_int(al);
            __syncthreads();
            prep_store<J>(s_tile, tv, N, V, v0, m0);
        }
    }
    ss += __shfl_xor(ss, 32);
    if (lane < 32) s_sum[wave][vl] = ss;
    __syncthreads();
    if (tid < kRegV && v < V) {
        double s2 = 0.0;
#pragma unroll
        for (int p = 0; p < kRegPh / 2; ++p) s2 += s_sum[p][vl];
        const double var_pop = s2 / (double)N;
        mean[(int64_t)var * V + v] = mu;
        inv_std[(int64_t)var * V + v] = (var_pop > 0.0 && !flat) ? 1.0 / sqrt(var_pop) : 0.0;
        flags[(int64_t)var * V + v] =
            (bad ? NDF_FLAG_NONFINITE : 0) | (flat ? NDF_FLAG_CONSTANT : 0);
        // every writer stores the same value, so the unordered stores agree
        if (bad && status) *status = NDF_E_NONFINITE;
    }
    if constexpr (OE > 0) {
        uint16_t *ov = order + (int64_t)var * V * N;
        uint32_t *lds = reinterpret_cast<uint32_t *>(s_tile) + wave * ColumnSort<OE>::kLds;
#pragma unroll
        for (int c = 0; c < kCols; ++c) {
            const int64_t vc = v0 + kCols * wave + c;
            if (vc >= V) break;  // uniform
            wave_sort_codes<OE, 0>(sc[c], N, ov + vc * N, lds);
            wave_lds_fence();
        }
    }
}

// ------------------------------------- more than 1039 members, or few ----------
// One workgroup owns 64 consecutive vertices of one variable and reads their
// members twice (sum / min / max, then centred squares and codes).  Each thread keeps 8
// (first pass) or 16 (second pass) of its member loads in flight; one load at a time
// left the kernel latency-bound at 3.3 TB/s.  (Two vertices per thread with 8-byte loads
// measured slower: the larger tile cut the resident workgroups per CU.)
constexpr int kPrepV = 64;                    // vertices per workgroup
constexpr int kPrepPh = 4;                    // member phases per vertex
constexpr int kPrepThreads = kPrepV * kPrepPh;

__global__ __launch_bounds__(kPrepThreads) void prepare_long_kernel(
    const float *__restrict__ x, int N, int64_t V, double *__restrict__ mean,
    double *__restrict__ inv_std, int32_t *__restrict__ code, int32_t *__restrict__ flags,
    int32_t *__restrict__ status) {
    const int var = blockIdx.y;
    const float *xv = x + (int64_t)var * N * V;
    const int t = threadIdx.x;
    const int vl = t % kPrepV;
    const int ph = t / kPrepV;
    const int64_t v0 = (int64_t)blockIdx.x * kPrepV;
    const int64_t v = v0 + vl;

    __shared__ double s_sum[kPrepPh][kPrepV];
    __shared__ float s_lo[kPrepPh][kPrepV];
    __shared__ float s_hi[kPrepPh][kPrepV];
    __shared__ int s_bad[kPrepPh][kPrepV];
    __shared__ int32_t s_tile[64][kPrepV + 1];

    // pass 1: sum, min, max, finiteness
    double sum = 0.0;
    float lo = INFINITY, hi = -INFINITY;
    int bad = 0;
    auto accumulate = [&](float a) {
        sum += (double)a;
        lo = fminf(lo, a);
        hi = fmaxf(hi, a);
        bad |= !isfinite(a);
    };
    if (v < V) {
        // eight members' loads in flight at a time; the sums keep member order
        constexpr int U = 8;
        int m = ph;
        for (; m + kPrepPh * (U - 1) < N; m += kPrepPh * U) {
            float a[U];
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = xv[(int64_t)(m + kPrepPh * u) * V + v];
#pragma unroll
            for (int u = 0; u < U; ++u) accumulate(a[u]);
        }
        for (; m < N; m += kPrepPh) accumulate(xv[(int64_t)m * V + v]);
    }
    s_sum[ph][vl] = sum;
    s_lo[ph][vl] = lo;
    s_hi[ph][vl] = hi;
    s_bad[ph][vl] = bad;
    __syncthreads();
    sum = 0.0;
    lo = INFINITY;
    hi = -INFINITY;
    bad = 0;
    for (int p = 0; p < kPrepPh; ++p) {
        sum += s_sum[p][vl];
        lo = fminf(lo, s_lo[p][vl]);
        hi = fmaxf(hi, s_hi[p][vl]);
        bad |= s_bad[p][vl];
    }
    const double mu = sum / (double)N;
    const bool flat = !(hi > lo);
    const double dlo = (double)lo;
    const double scale = flat ? 0.0 : 8388608.0 / ((double)hi - dlo);
    __syncthreads();

    // pass 2: centred sum of squares and the codes, transposed through LDS into
    // vertex-major rows.  A thread visits members ph, ph + 4, ... in increasing
    // order, so its FP64 sum is the plain two-pass one.
    int32_t *cv = code + (int64_t)var * V * N;
    double ss = 0.0;
    for (int m0 = 0; m0 < N; m0 += 64) {
        // the tile's 16 loads of this thread in flight together
        float a[64 / kPrepPh];
#pragma unroll
        for (int i = 0; i < 64 / kPrepPh; ++i) {
            const int m = m0 + ph + kPrepPh * i;
            if (v < V && m < N) a[i] = xv[(int64_t)m * V + v];
        }
#pragma unroll
        for (int i = 0; i < 64 / kPrepPh; ++i) {
            const int mm = ph + kPrepPh * i;
            int32_t c = 0;
            if (v < V && m0 + mm < N) {
                const double d = (double)a[i] - mu;
                ss += d * d;
                if (!flat) c = (int32_t)__builtin_rint(((double)a[i] - dlo) * scale);
            }
            s_tile[mm][vl] = c;
        }
        __syncthreads();
        // kPrepV rows (vertices) of up to 64 members; 16 threads per row, 4 members each
        for (int pass = 0; pass < kPrepV / 16; ++pass) {
            const int row = t / 16 + 16 * pass;
            const int c4 = t % 16;
            const int64_t vr = v0 + row;
            const int mb = m0 + 4 * c4;
            if (vr < V) {
                int32_t *dst = cv + vr * N + mb;
                if (mb + 3 < N && ((N & 3) == 0)) {
                    i32x4 q;
                    q.x = s_tile[4 * c4 + 0][row];
                    q.y = s_tile[4 * c4 + 1][row];
                    q.z = s_tile[4 * c4 + 2][row];
                    q.w = s_tile[4 * c4 + 3][row];
                    *reinterpret_cast<i32x4 *>(dst) = q;
                } else {
                    for (int e = 0; e < 4; ++e)
                        if (mb + e < N) dst[e] = s_tile[4 * c4 + e][row];
                }
            }
        }
        __syncthreads();
    }
    s_sum[ph][vl] = ss;
    __syncthreads();
    if (ph == 0 && v < V) {
        double s2 = 0.0;
        for (int p = 0; p < kPrepPh; ++p) s2 += s_sum[p][vl];
        const double var_pop = s2 / (double)N;
        mean[(int64_t)var * V + v] = mu;
        inv_std[(int64_t)var * V + v] = (var_pop > 0.0 && !flat) ? 1.0 / sqrt(var_pop) : 0.0;
        flags[(int64_t)var * V + v] =
            (bad ? NDF_FLAG_NONFINITE : 0) | (flat ? NDF_FLAG_CONSTANT : 0);
        // every writer stores the same value, so the unordered stores agree
        if (bad && status) *status = NDF_E_NONFINITE;
    }
}

// Vertex-major copy xt[v][m] of the member-major ensemble x[m][v] (for the
// reads of a few scattered vertices' full columns, as interpolation at
// continuous positions does): 64 x 64 tiles through LDS.  VEC (V and N multiples
// of 4): 16-byte loads of four vertices of a member row and 16-byte stores of
// four members of a vertex row, 16 threads per 256-byte row segment.
template <bool VEC>
__global__ __launch_bounds__(256) void transpose_kernel(const float *__restrict__ x, int N,
                                                        int64_t V, float *__restrict__ xt) {
    __shared__ float tile[64][65];
    const int var = blockIdx.z;
    const float *xv = x + (int64_t)var * N * V;
    float *tv = xt + (int64_t)var * V * N;
    const int64_t v0 = (int64_t)blockIdx.x * 64;
    const int m0 = blockIdx.y * 64;
    if (VEC) {
        const int c4 = threadIdx.x & 15, r = threadIdx.x >> 4;  // 16 rows of 16 x 16 B
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + r + 16 * i;
            const int64_t v = v0 + 4 * c4;
            f32x4 q = {0.f, 0.f, 0.f, 0.f};
            if (m < N && v < V)
                q = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(xv + (int64_t)m * V + v));
#pragma unroll
            for (int e = 0; e < 4; ++e) tile[r + 16 * i][4 * c4 + e] = q[e];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int vl = r + 16 * i;
            const int64_t v = v0 + vl;
            const int m = m0 + 4 * c4;
            if (v < V && m < N) {
                f32x4 q;
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = tile[4 * c4 + e][vl];
                *reinterpret_cast<f32x4 *>(tv + v * N + m) = q;
            }
        }
        return;
    }
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) {
        const int m = m0 + i;
        const int64_t v = v0 + tx;
        tile[i][tx] = (m < N && v < V) ? __builtin_nontemporal_load(xv + (int64_t)m * V + v) : 0.f;
    }
    __syncthreads();
    for (int i = ty; i < 64; i += 4) {
        const int64_t v = v0 + i;
        const int m = m0 + tx;
        if (v < V && m < N) tv[v * N + m] = tile[tx][i];
    }
}

__global__ void status_clear_kernel(int32_t *status) { *status = NDF_OK; }

int launch_status_clear(int32_t *status, hipStream_t st) {
    hipLaunchKernelGGL(status_clear_kernel, dim3(1), dim3(1), 0, st, status);
    return status_of_launch();
}

int launch_prepare(const ndf_ensemble *e, int32_t *status, bool *sorted, hipStream_t st) {
    const int64_t V = (int64_t)e->nx * e->ny * e->nz;
    if (status) launch_status_clear(status, st);
    const int N = e->n_members;
    const int64_t tiles = ceil_div(V, kRegV);
    const dim3 rg((unsigned)(tiles < kRegGridX ? tiles : kRegGridX), (unsigned)e->n_vars,
                  (unsigned)ceil_div(tiles, kRegGridX));
    // the fewest registers that hold a thread's members: waves in flight against loads
    // past the last member.  Up to 512 members the columns are sorted here too, from codes
    // kept in registers (450 members of 1.76M vertices 2.86 -> 2.59 ms, 250 members 1.44 ->
    // 1.33); with more the codes of a wave's four columns spill (1000 members 6.52 ms
    // against 6.22 with a kernel of its own).
    *sorted = false;
    // Few members with neither orders nor the vertex-major copy: the two-read kernel, which
    // holds them in one 64-member tile (its second read comes from the caches) and spends
    // four threads instead of sixteen on a vertex.  1.76M vertices, us, one read against
    // two: 2 members 156 / 118, 16 169 / 137, 32 189 / 144, 48 206 / 223, 56 218 / 267, 63
    // 240 / 312, 64 (a whole tile) 227 / 208, 68 252 / 268; 65536 vertices: 2 members
    // 8.5 / 7.0, 48 10.4 / 8.8, 56 10.6 / 10.0, 64 10.7 / 8.7, 68 11.8 / 12.1.
    // With the copy, which the two-read kernel leaves to a launch of its own, up to 16 members
    // and 32 (whole rows of both kernels' stores) from 2^17 vertices on.  1.76M vertices: 2
    // members 179 / 129, 4 169 / 110, 15 216 / 204, 16 198 / 177, 17 205 / 225, 20 203 /
    // 210, 31 256 / 317, 32 226 / 202, 40 239 / 260; 131,072: 2 members 15.9 / 14.6, 16 17.3
    // / 14.7, 20 17.8 / 15.7, 28 19.0 / 18.2, 32 19.7 / 17.3, 40 20.9 / 20.3; 65536: 2 members
    // 9.3 / 9.9, 8 9.0 / 8.8; 11,803: 6.4 / 8.6.
    const bool two_reads =
        !e->order && (e->xt ? V >= 1 << 17 && (N <= 16 || N == 32) : N <= 48 || N == 64);
#define NDF_PREP_LAUNCH(E, OE)                                                                   \
    hipLaunchKernelGGL((prepare_kernel<E, OE>), rg, dim3(kRegThreads), 0, st, e->x, N, V, e->mean, \
                       e->inv_std, e->code, e->flags, status, e->xt, e->order)
#define NDF_PREP_CASE(E, OE)                                                                     \
    if (!two_reads && N < kRegPh * (E + 1)) {                                                    \
        *sorted = OE && e->order && N <= 64 * OE;                                                \
        if (*sorted)                                                                             \
            NDF_PREP_LAUNCH(E, OE);                                                              \
        else                                                                                     \
            NDF_PREP_LAUNCH(E, 0);                                                               \
        return status_of_launch();                                                               \
    }
    NDF_PREP_CASE(4, 1) NDF_PREP_CASE(8, 2) NDF_PREP_CASE(16, 4)
    NDF_PREP_CASE(32, 8) NDF_PREP_CASE(48, 0) NDF_PREP_CASE(64, 0)
#undef NDF_PREP_CASE
#undef NDF_PREP_LAUNCH
    dim3 grid((unsigned)ceil_div(V, kPrepV), (unsigned)e->n_vars);
    hipLaunchKernelGGL(prepare_long_kernel, grid, dim3(kPrepThreads), 0, st, e->x, N, V, e->mean,
                       e->inv_std, e->code, e->flags, status);
    if (e->xt) {
        dim3 tg((unsigned)ceil_div(V, 64), (unsigned)ceil_div(N, 64), (unsigned)e->n_vars);
        if (V % 4 == 0 && N % 4 == 0)
            hipLaunchKernelGGL(transpose_kernel<true>, tg, dim3(256), 0, st, e->x, N, V, e->xt);
        else
            hipLaunchKernelGGL(transpose_kernel<false>, tg, dim3(256), 0, st, e->x, N, V, e->xt);
    }
    return status_of_launch();
}

}  // namespace ndf
