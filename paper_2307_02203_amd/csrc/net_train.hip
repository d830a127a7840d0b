// Training kernels of the learned dependence field (Sec. 4, Eq. 3; Sec. 4.3).
//
// The mean L1 loss is differentiated by hand:
//   forward   grid gather -> [X W^T + b, ReLU] x2 -> X W3^T + b3 -> product
//             -> [X W^T + b, ReLU] x2 -> w6 . d2 + b6
//   adjoint   dY W (masked by the forward ReLU), dW += dY^T X, db += sum dY,
//             the product rule across the merge, FP32 atomic scatter into the
//             grid levels with the trilinear weights.
// Layer products run on MFMA 32x32x16 bf16 with FP32 accumulate: activations
// and weights are rounded to bf16 as they enter the MFMA; latents, parameters, parameter
// gradients and Adam moments are FP32.
//
// Networks with an encoder MLP run in the fused kernels below ("fused step").  Two kinds of
// call run row-wise, layer by layer: a grid-only network (no encoder MLP), and a
// two-encoder network whose caller brings a workspace that is too small for the fused
// step's slabs and packed weights but holds the layers' rows (few pairs: 8 KB against
// 0.6 MB for one; fewer bytes below 224 pairs and at some counts up to 293).  The R = 2B
// positions (all first endpoints, then all second endpoints) go through the grid lookup (and
// the encoders), the two feature rows of a pair are multiplied, and the decoder gives Phi:
//  rows_mma_kernel  Y[rows][NOUT] = epilogue(X[rows][KIN] A^T), A staged once per
//                   workgroup in LDS in MFMA operand order (A = W forward,
//                   A = W^T for the data adjoint); 64 rows per wave and tile.
//  wgrad_kernel     dW[128][KIN] += G^T X over rows: 64-row tiles of G and X are
//                   transposed through LDS so both operands are row-contiguous.
#include "net.hpp"

namespace ndf {

constexpr int kThreads = 256;

struct GridOffs {
    int64_t off[2][kL];
};

__device__ __forceinline__ int64_t grid_off(const GridOffs &go, int e, int l) {
    // each offset is read before the choice, which else becomes one of addresses and
    // moves the struct to scratch memory
    int64_t r = 0;
#pragma unroll
    for (int i = 0; i < 2 * kL; ++i) {
        const int64_t o = go.off[i / kL][i % kL];
        r |= e * kL + l == i ? o : 0;
    }
    return r;
}

// ------------------------------------------------------------- helpers ----
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t i) {
    // i-th output of SplitMix64 (Steele, Lea, Flood 2014) started from `seed`
    uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void fill_kernel(float *__restrict__ p, int64_t n, float v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void uniform_kernel(float *__restrict__ p, int64_t n, float a, uint64_t seed,
                               int64_t ctr0) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double u = (double)(splitmix64_at(seed, (uint64_t)(ctr0 + i)) >> 11) * 0x1.0p-53;
        p[i] = (float)(a * (2.0 * u - 1.0));
    }
}

static unsigned gs_blocks(int64_t n) {
    int64_t b = ceil_div(n, kThreads);
    return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

__device__ __forceinline__ int64_t row_vertex(const int64_t *pairs, int64_t B, int64_t n) {
    return n < B ? pairs[2 * n] : pairs[2 * (n - B) + 1];
}

// Row n's position as continuous coordinates in [-1, 1]^3 when the pairs are
// given as positions pos[B][2][3] (the training pairs of Sec. 4.3).
__device__ __forceinline__ const float *row_pos(const float *pos, int64_t B, int64_t n) {
    return pos + 3 * (n < B ? 2 * n : 2 * (n - B) + 1);
}

// Trilinear corners of row n on level l: from its vertex index (pairs) or its
// continuous position (pos, when non-null); cells hashed on hashed levels.
__device__ __forceinline__ void row_corners(const GridGeom &g, int l, const int64_t *pairs,
                                            const float *pos, int64_t B, int64_t n, int idx[8],
                                            float w[8]) {
    int R[3];
    level_dims(g, l, R);
    const uint32_t hm = level_hmask(g, l);
    if (pos) {
        const float *p = row_pos(pos, B, n);
        const float pp[3] = {p[0], p[1], p[2]};
        corners_pos32<true>(R, pp, idx, w, hm);
    } else {
        int64_t v = row_vertex(pairs, B, n);
        const int64_t V = (int64_t)g.nx * g.ny * g.nz;
        v = v < 0 ? 0 : (v >= V ? V - 1 : v);  // out-of-range pairs are clamped
        corners_R32<true>(g, R, v, idx, w, hm);
    }
}

// ----------------------------------------------------------- grid fwd ----
// H0[n][l*8 + f] for rows n < 2B (first endpoints, then second endpoints).
__global__ __launch_bounds__(kThreads) void grid_fwd_kernel(const float *__restrict__ params,
                                                            GridOffs go, GridGeom g, int n_enc,
                                                            const int64_t *__restrict__ pairs,
                                                            const float *__restrict__ pos,
                                                            int64_t B, float *__restrict__ H0) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * B * kL) return;
    const int64_t n = t / kL;
    const int l = (int)(t % kL);
    const int e = (n_enc == 2 && n >= B) ? 1 : 0;
    int idx[8];
    float w[8];
    row_corners(g, l, pairs, pos, B, n, idx, w);
    const f32x4 *grid = reinterpret_cast<const f32x4 *>(params + grid_off(go, e, l));
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
    for (int cn = 0; cn < 8; ++cn) {
        const f32x4 c0 = grid[idx[cn] * 2], c1 = grid[idx[cn] * 2 + 1];
        a0 += w[cn] * c0;
        a1 += w[cn] * c1;
    }
    f32x4 *out = reinterpret_cast<f32x4 *>(H0 + n * kK0 + l * kF);
    out[0] = a0;
    out[1] = a1;
}

// ----------------------------------------------------------- grid bwd ----
// Scatter-add of dL/dh0 into the grid gradient: a wave takes four (row, level)
// items, lane = (item i, corner bit dx, feature f).  Each lane evaluates its
// item's trilinear lookup (the forward's arithmetic, so the same weights bit for
// bit) and issues one atomic per corner pair (dx = 0, 1 at equal dy, dz): on a
// dense level the two cells are neighbours in memory, so every atomic
// instruction of the wave adds four 64-byte runs.
__global__ __launch_bounds__(kThreads) void grid_bwd_kernel(float *__restrict__ grad, GridOffs go,
                                                            GridGeom g, int n_enc,
                                                            const int64_t *__restrict__ pairs,
                                                            const float *__restrict__ pos,
                                                            int64_t B,
                                                            const float *__restrict__ dH0) {
    const int lane = threadIdx.x & 63, i = lane >> 4, dx = (lane >> 3) & 1, f = lane & 7;
    const int64_t items = 2 * B * kL;
    const int64_t waves = (int64_t)gridDim.x * (kThreads / 64);
    for (int64_t w0 = ((int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)) * 4;
         w0 < items; w0 += waves * 4) {
        const int64_t it = w0 + i;
        if (it >= items) continue;
        const int64_t n = it / kL;
        const int l = (int)(it % kL);
        const int e = (n_enc == 2 && n >= B) ? 1 : 0;
        int idx[8];
        float w[8];
        row_corners(g, l, pairs, pos, B, n, idx, w);
        const float d = dH0[n * kK0 + l * kF + f];
        float *gl = grad + grid_off(go, e, l) + f;
        // this lane's corner of each pair by bit blending (a select between two
        // elements is turned into a lane-dependent index, which moves idx and w
        // to memory)
        const int m = -dx;
        int ic[4];
        float wc[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            ic[c] = idx[2 * c] ^ (m & (idx[2 * c] ^ idx[2 * c + 1]));
            wc[c] = __int_as_float(__float_as_int(w[2 * c]) ^
                                   (m & (__float_as_int(w[2 * c]) ^ __float_as_int(w[2 * c + 1]))));
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (wc[c] != 0.f) unsafeAtomicAdd(gl + (int64_t)ic[c] * kF, wc[c] * d);
    }
}

// ---------------------------------------------------- sorted grid scatter ----
// Large batches add to every cell of the coarser levels many times (2^18 pairs: 154, 38
// and 9 times on the 250 x 352 x 20 grid's three coarser levels).  The rows are therefore
// sorted by the spatial tile of the data grid they lie in (grid_sort_count_kernel,
// grid_sort_place_kernel), and a workgroup takes up to TilePlan::rows rows of one tile
// (grid_tile_kernel): the tile's cells of those levels are boxes that fit in LDS, where
// the rows' contributions are summed; one global atomic per touched cell and feature
// remains.  Hashed levels (no box) and the finest one (a cell is hit about
// once) are added to directly by a wave of their own, as grid_bwd_kernel does for small
// batches.  Added directly, the batch is bound by the L2 atomics (one level 0.25 ns per
// row) and on small grids by the adds to one cell, which follow each other: 2^18 pairs of
// 250 x 352 x 20 vertices took 466 us, now 142 (sort 27, tiles 115; at positions 623 and
// 262), of 37 x 29 x 11 1363 and 125, 150000 pairs of 16 x 14 x 5 2467 and 80.
constexpr int kSortWgs = 64;        // workgroups (row ranges) of the sort
constexpr int kSortThreads = 1024;
constexpr int kMaxTiles = 4096;     // tiles of all encoders
constexpr int64_t kMinSorted = 4096;  // rows below which the sort's launches cost more
constexpr size_t kTileLds = 55 * 1024;  // boxes of a tile; with the stages 64 KB of LDS

struct TilePlan {
    int t[3];             // tile edges in data-grid vertices
    int nt[3];            // tiles per axis
    uint32_t m[3];        // ceil(2^32 / t)
    int n_tiles;          // of one encoder
    int box[kL - 1][3];   // cells of a tile's box per axis
    int off[kL - 1];      // the box's first cell in LDS
    int cells;            // of all boxes
    int rows;             // rows of a workgroup, at most
    int boxed;            // levels 0 .. boxed - 1 have boxes (at most kL - 1)
};

// A sorted row: data-grid coordinates of its vertex, or its position.
struct __attribute__((aligned(16))) SortedRow {
    int n;
    int x, y, z;  // vertex (i, j, k), or the bits of the position's floats
};

__device__ __forceinline__ void vertex_ijk(const GridGeom &g, int64_t v64, int (&c)[3]) {
    const uint32_t v = (uint32_t)v64;
    const uint32_t t = (uint32_t)(((uint64_t)v * g.mx) >> 40);  // v / nx
    const uint32_t k = (uint32_t)(((uint64_t)t * g.my) >> 40);  // t / ny
    c[0] = (int)(v - t * (uint32_t)g.nx);
    c[1] = (int)(t - k * (uint32_t)g.ny);
    c[2] = (int)k;
}

// Row n as a sorted entry and its tile (encoder e's tiles follow encoder e - 1's).
__device__ __forceinline__ int row_tile(const GridGeom &g, const TilePlan &tp, int n_enc,
                                        const int64_t *pairs, const float *pos, int64_t B,
                                        int64_t n, SortedRow &r) {
    int c[3];
    r.n = (int)n;
    if (pos) {
        const float *p = row_pos(pos, B, n);
        const int nn[3] = {g.nx, g.ny, g.nz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float hn = 0.5f * (float)(nn[a] - 1);
            c[a] = min((int)fminf(fmaxf(fmaf(p[a], hn, hn), 0.f), (float)(nn[a] - 1)), nn[a] - 1);
        }
        r.x = __float_as_int(p[0]);
        r.y = __float_as_int(p[1]);
        r.z = __float_as_int(p[2]);
    } else {
        int64_t v = row_vertex(pairs, B, n);
        const int64_t V = (int64_t)g.nx * g.ny * g.nz;
        v = v < 0 ? 0 : (v >= V ? V - 1 : v);  // out-of-range pairs are clamped
        vertex_ijk(g, v, c);
        r.x = c[0];
        r.y = c[1];
        r.z = c[2];
    }
    int ti[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ti[a] = (int)(((uint64_t)(uint32_t)c[a] * tp.m[a]) >> 32);
    const int e = (n_enc == 2 && n >= B) ? 1 : 0;
    return e * tp.n_tiles + ti[0] + tp.nt[0] * (ti[1] + tp.nt[1] * ti[2]);
}

// Workgroup w counts the rows of its range per tile: hist[w][tile].
__global__ __launch_bounds__(kSortThreads) void grid_sort_count_kernel(
    GridGeom g, TilePlan tp, int n_enc, const int64_t *__restrict__ pairs,
    const float *__restrict__ pos, int64_t B, int *__restrict__ hist) {
    __shared__ int s_n[kMaxTiles];
    const int tiles = n_enc * tp.n_tiles;
    for (int i = threadIdx.x; i < tiles; i += kSortThreads) s_n[i] = 0;
    __syncthreads();
    const int64_t rows = 2 * B, lo = rows * blockIdx.x / kSortWgs,
                  hi = rows * (blockIdx.x + 1) / kSortWgs;
    for (int64_t n = lo + threadIdx.x; n < hi; n += kSortThreads) {
        SortedRow r;
        atomicAdd(&s_n[row_tile(g, tp, n_enc, pairs, pos, B, n, r)], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < tiles; i += kSortThreads)
        hist[(int64_t)blockIdx.x * tiles + i] = s_n[i];
}

// Exclusive scan of v over the workgroup's threads (kSortThreads), total in `total`.
__device__ __forceinline__ int block_scan(int v, int *s_w, int &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int s = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(s, d);
        if (lane >= d) s += t;
    }
    if (lane == 63) s_w[w] = s;
    __syncthreads();
    int base = 0;
    total = 0;
    for (int i = 0; i < kSortThreads / 64; ++i) {
        base += i < w ? s_w[i] : 0;
        total += s_w[i];
    }
    __syncthreads();
    return base + s - v;
}

// Workgroup w places the rows of its range: tile starts from all counts, then the rows of
// earlier ranges, then an LDS counter.  Workgroup 0 also writes the work list of
// grid_tile_kernel: list[0].x = entries, list[1 + i] = (tile, first row, end row, -).
__global__ __launch_bounds__(kSortThreads) void grid_sort_place_kernel(
    GridGeom g, TilePlan tp, int n_enc, const int64_t *__restrict__ pairs,
    const float *__restrict__ pos, int64_t B, const int *__restrict__ hist,
    SortedRow *__restrict__ out, int4 *__restrict__ list) {
    __shared__ int s_at[kMaxTiles];
    __shared__ int s_w[kSortThreads / 64];
    const int tiles = n_enc * tp.n_tiles;
    int start0 = 0, item0 = 0;
    for (int t0 = 0; t0 < tiles; t0 += kSortThreads) {
        const int t = t0 + threadIdx.x;
        int all = 0, before = 0;
        if (t < tiles) {
#pragma unroll 16
            for (int w = 0; w < kSortWgs; ++w) {
                const int h = hist[(int64_t)w * tiles + t];
                all += h;
                before += w < (int)blockIdx.x ? h : 0;
            }
        }
        int sum, items;
        const int start = start0 + block_scan(all, s_w, sum);
        if (t < tiles) s_at[t] = start + before;
        start0 += sum;
        if (blockIdx.x == 0) {  // uniform
            const int n_item = (all + tp.rows - 1) / tp.rows;
            const int item = item0 + block_scan(n_item, s_w, items);
            for (int i = 0; i < n_item; ++i)
                list[1 + item + i] = make_int4(t, start + i * tp.rows,
                                               start + min(all, (i + 1) * tp.rows), 0);
            item0 += items;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) list[0] = make_int4(item0, 0, 0, 0);
    __syncthreads();
    const int64_t rows = 2 * B, lo = rows * blockIdx.x / kSortWgs,
                  hi = rows * (blockIdx.x + 1) / kSortWgs;
    for (int64_t n = lo + threadIdx.x; n < hi; n += kSortThreads) {
        SortedRow r;
        const int t = row_tile(g, tp, n_enc, pairs, pos, B, n, r);
        out[atomicAdd(&s_at[t], 1)] = r;
    }
}

// Base cell and fraction of a sorted row on a level along axis a: the arithmetic of
// corners_R32 and corners_pos32, so the same weights bit for bit.
template <bool POS>
__device__ __forceinline__ void axis_cell(const GridGeom &g, int R, int a, int c, int &b,
                                          float &f) {
    if (POS) {
        const float hr = 0.5f * (float)(R - 1);
        const float x = fminf(fmaxf(fmaf(__int_as_float(c), hr, hr), 0.f), (float)(R - 1));
        b = min(max((int)x, 0), R - 2);
        f = x - (float)b;
    } else {
        const int n1 = (a == 0 ? g.nx : a == 1 ? g.ny : g.nz) - 1;
        const uint32_t p = (uint32_t)c * (uint32_t)(R - 1);
        const uint32_t q = (uint32_t)(((uint64_t)p * g.md[a]) >> 40);
        const uint32_t rem = p - q * (uint32_t)n1;
        b = min((int)q, R - 2);
        f = (float)((int)q - b) + (float)rem * g.inv[a];
    }
}

// Rows [lo, hi) of one tile on a level without a box, by one wave: kAhead rows in turn per
// lane group, their loads in flight together; rows of one cell that follow each other
// are summed before the global atomics.  PAIR: a group is (x-neighbour, feature), so an
// instruction adds four 64-byte runs, as in grid_bwd_kernel; else (vertices of a level of
// the data grid's size, one corner each) a group is the feature.
template <bool POS, bool PAIR>
__device__ __forceinline__ void tile_direct(float *__restrict__ gl, const GridGeom &g,
                                            const int (&R)[3], uint32_t hm, int l,
                                            const SortedRow *__restrict__ rows, int lo, int hi,
                                            const float *__restrict__ dH0) {
    constexpr int kGroup = PAIR ? 16 : 8, kRows = 64 / kGroup, kAhead = 8, kC = PAIR ? 4 : 8;
    const int lane = threadIdx.x & 63, f = lane & 7, dx = PAIR ? (lane >> 3) & 1 : 0;
    auto add = [&](const int (&b)[3], const float (&v)[kC]) {
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const int x = PAIR ? dx : c & 1, y = PAIR ? c & 1 : (c >> 1) & 1,
                      z = PAIR ? c >> 1 : c >> 2;
            if (v[c] != 0.f)
                unsafeAtomicAdd(gl + (int64_t)cell_index<true>(b[0] + x, b[1] + y, b[2] + z, R, hm) * kF + f,
                                v[c]);
        }
    };
    for (int i0 = lo + lane / kGroup * kAhead; i0 < hi; i0 += kRows * kAhead) {
        SortedRow r[kAhead];
        float d[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) r[u] = rows[min(i0 + u, hi - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) d[u] = dH0[(int64_t)r[u].n * kK0 + l * kF + f];
        int at[3] = {-1, -1, -1};  // cell of the rows in `sum`
        float sum[kC] = {};
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (i0 + u >= hi) break;
            const int rc[3] = {r[u].x, r[u].y, r[u].z};
            int b[3];
            float w[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) axis_cell<POS>(g, R[a], a, rc[a], b[a], w[a]);
            if (b[0] != at[0] || b[1] != at[1] || b[2] != at[2]) {
                add(at, sum);
#pragma unroll
                for (int a = 0; a < 3; ++a) at[a] = b[a];
#pragma unroll
                for (int c = 0; c < kC; ++c) sum[c] = 0.f;
            }
#pragma unroll
            for (int c = 0; c < kC; ++c) {
                const int x = PAIR ? dx : c & 1, y = PAIR ? c & 1 : (c >> 1) & 1,
                          z = PAIR ? c >> 1 : c >> 2;
                const float wc = (x ? w[0] : 1.f - w[0]) * (y ? w[1] : 1.f - w[1]) *
                                 (z ? w[2] : 1.f - w[2]);
                if (wc != 0.f) sum[c] += wc * d[u];
            }
        }
        add(at, sum);
    }
}

// A workgroup takes one item (rows of one tile), wave l level l.  A boxed level's LDS box
// belongs to that wave alone, so a row is one read, add and write of 64 words, lane =
// (corner, feature), with no atomics: LDS float atomics take four cycles a lane (256 a row
// and level, measured; the kernel with them took 665 us for 2^18 pairs), the chain of
// read, add and write about half.  The cells, fractions and dL/dh0 of 64 rows are
// computed and loaded at once, a row per lane, and pass through LDS, from where every
// lane reads the row's at one address (through scalar registers, lane by lane, a row took
// 430 cycles); the next 64 rows' loads are in flight meanwhile.
constexpr int kBatch = 64;

struct TileStage {
    f32x4 row[kBatch];   // entry of the box (int bits), fractions
    float d[kBatch][kF];
};
static_assert(kTileLds + (kL - 1) * sizeof(TileStage) <= 64 * 1024, "LDS of a launch");

template <bool POS>
__global__ __launch_bounds__(64 * kL) void grid_tile_kernel(
    float *__restrict__ grad, GridOffs go, GridGeom g, TilePlan tp,
    const SortedRow *__restrict__ rows, const int4 *__restrict__ list,
    const float *__restrict__ dH0) {
    extern __shared__ f32x4 s_tile[];  // TileStage[boxed] | [cells][8]
    if ((int)blockIdx.x >= list[0].x) return;
    const int4 item = list[1 + blockIdx.x];
    const int e = item.x >= tp.n_tiles ? 1 : 0, tile = item.x - e * tp.n_tiles;
    const int ti[3] = {tile % tp.nt[0], tile / tp.nt[0] % tp.nt[1], tile / (tp.nt[0] * tp.nt[1])};
    const int nn[3] = {g.nx, g.ny, g.nz};
    const int lane = threadIdx.x & 63, f = lane & 7;
    const int l = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int R[3], box[3], o[3];  // level sizes; the box's edges and first cell
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        R[a] = 0;
#pragma unroll
        for (int i = 0; i < kL; ++i) {
            const int r = g.R[i][a];
            R[a] |= l == i ? r : 0;
        }
    }
    float *gl = grad + grid_off(go, e, l);
    if (l >= tp.boxed) {
        const uint32_t hm = level_hmask(g, l);
        if (!POS && R[0] == nn[0] && R[1] == nn[1] && R[2] == nn[2])
            tile_direct<POS, false>(gl, g, R, hm, l, rows, item.y, item.z, dH0);
        else
            tile_direct<POS, true>(gl, g, R, hm, l, rows, item.y, item.z, dH0);
        return;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        box[a] = l == 0 ? tp.box[0][a] : l == 1 ? tp.box[1][a] : tp.box[2][a];
        o[a] = max(min((int)((int64_t)ti[a] * tp.t[a] * (R[a] - 1) / (nn[a] - 1)), R[a] - box[a]), 0);
    }
    const int cells = box[0] * box[1] * box[2];
    TileStage &S = reinterpret_cast<TileStage *>(s_tile)[l];
    float *acc = reinterpret_cast<float *>(reinterpret_cast<TileStage *>(s_tile) + tp.boxed) +
                 (l == 0 ? tp.off[0] : l == 1 ? tp.off[1] : tp.off[2]) * kF;
    for (int i = lane; i < cells * kF; i += 64) acc[i] = 0.f;
    // this lane's corner: weight factor s_a f_a + t_a per axis, offset in the box
    const int dx = (lane >> 3) & 1, dy = (lane >> 4) & 1, dz = lane >> 5;
    const float sx = dx ? 1.f : -1.f, sy = dy ? 1.f : -1.f, sz = dz ? 1.f : -1.f;
    const float tx = dx ? 0.f : 1.f, ty = dy ? 0.f : 1.f, tz = dz ? 0.f : 1.f;
    float *const mine = acc + (dx + box[0] * (dy + box[1] * dz)) * kF + f;

    const int last = item.z - 1;
    auto load_d = [&](int n, f32x4 &a, f32x4 &b) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(dH0 + (int64_t)n * kK0 + l * kF);
        a = p[0];
        b = p[1];
    };
    SortedRow r = rows[min(item.y + lane, last)];
    SortedRow r1 = rows[min(item.y + kBatch + lane, last)];
    f32x4 d0, d1;
    load_d(r.n, d0, d1);
    for (int i0 = item.y; i0 < item.z; i0 += kBatch) {
        const int rc[3] = {r.x, r.y, r.z};
        int b[3];
        float w[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) axis_cell<POS>(g, R[a], a, rc[a], b[a], w[a]);
        const int lx = b[0] - o[0], ly = b[1] - o[1], lz = b[2] - o[2];
        const bool real = i0 + lane < item.z;
        const bool in = (uint32_t)lx < (uint32_t)(box[0] - 1) &&
                        (uint32_t)ly < (uint32_t)(box[1] - 1) &&
                        (uint32_t)lz < (uint32_t)(box[2] - 1);
        if (real && !in) {  // a position's rounding at a tile's edge: added to directly
            for (int c = 0; c < 8; ++c) {
                const int cx = c & 1, cy = (c >> 1) & 1, cz = c >> 2;
                const float wc = (cx ? w[0] : 1.f - w[0]) * (cy ? w[1] : 1.f - w[1]) *
                                 (cz ? w[2] : 1.f - w[2]);
                float *at = gl + (int64_t)(b[0] + cx + R[0] * (b[1] + cy + R[1] * (b[2] + cz))) * kF;
                if (wc != 0.f)
                    for (int k = 0; k < kF; ++k) unsafeAtomicAdd(at + k, wc * (k < 4 ? d0[k] : d1[k - 4]));
            }
        }
        const bool use = real && in;  // else a row of zeros
        const int at = use ? (lx + box[0] * (ly + box[1] * lz)) * kF : 0;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        S.row[lane] = f32x4{__int_as_float(at), w[0], w[1], w[2]};
        *reinterpret_cast<f32x4 *>(&S.d[lane][0]) = use ? d0 : zero;
        *reinterpret_cast<f32x4 *>(&S.d[lane][4]) = use ? d1 : zero;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the next batch
        r = r1;
        load_d(r.n, d0, d1);
        r1 = rows[min(i0 + 2 * kBatch + lane, last)];
        const int n = min(item.z - i0, kBatch);
        for (int j0 = 0; j0 < n; j0 += 8) {
            float wd[8];
            int where[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const f32x4 q = S.row[j0 + j];
                where[j] = __float_as_int(q[0]);
                const float wc = fmaf(sx, q[1], tx) * fmaf(sy, q[2], ty) * fmaf(sz, q[3], tz);
                // a corner of weight 0 adds nothing, also where dL/dh0 is no number
                const int m = wc != 0.f ? -1 : 0;
                wd[j] = __int_as_float(__float_as_int(wc * S.d[j0 + j][f]) & m);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) mine[where[j]] += wd[j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    // one global atomic per touched cell and feature, x-neighbours in one run
    for (int i = lane; i < cells * kF; i += 64) {
        const float v = acc[i];
        const int c = i >> 3, x = c % box[0], yz = c / box[0], y = yz % box[1], z = yz / box[1];
        if (v != 0.f)
            unsafeAtomicAdd(gl + (int64_t)((o[0] + x) + R[0] * ((o[1] + y) + R[1] * (o[2] + z))) * kF + f, v);
    }
}

// ----------------------------------------------------- row-wise MFMA ----
enum { EPI_BIAS = 0, EPI_BIAS_RELU = 1, EPI_MASK = 2, EPI_PLAIN = 3 };

__device__ __forceinline__ bf16x8 load_row8(const float *__restrict__ X, int64_t rows, int64_t r,
                                            int ld, int k0) {
    bf16x8 b;
    if (r < rows) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(X + r * ld + k0);
        const f32x4 u = p[0], w = p[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            b[e] = f2bf(u[e]);
            b[4 + e] = f2bf(w[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) b[e] = f2bf(0.f);
    }
    return b;
}

// Y[rows][NOUT] = epi(X[rows][KIN] * A^T) with A[i][k] = W[i*w_si + k*w_sk].
template <int KIN, int NOUT, int EPI>
__global__ __launch_bounds__(kThreads) void rows_mma_kernel(
    const float *__restrict__ X, int64_t rows, const float *__restrict__ W, int w_si, int w_sk,
    const float *__restrict__ bias, const float *__restrict__ mask, float *__restrict__ Y) {
    constexpr int KB = KIN / 16, OB = NOUT / 32;
    __shared__ bf16x8 s_a[OB * KB * 64];
    __shared__ float s_bias[NOUT];
    __bf16 *sa = reinterpret_cast<__bf16 *>(s_a);
    for (int idx = threadIdx.x; idx < NOUT * KIN; idx += kThreads) {
        const int i = idx / KIN, k = idx % KIN;
        const float wv = W[(int64_t)i * w_si + (int64_t)k * w_sk];
        const int ob = i >> 5, il = i & 31, kb = k >> 4, hh = (k >> 3) & 1, e = k & 7;
        sa[((ob * KB + kb) * 64 + hh * 32 + il) * 8 + e] = f2bf(wv);
    }
    if (EPI == EPI_BIAS || EPI == EPI_BIAS_RELU)
        for (int i = threadIdx.x; i < NOUT; i += kThreads) s_bias[i] = bias[i];
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, jl = lane & 31;
    const int64_t ntiles = ceil_div(rows, 64);
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wave; tile < ntiles;
         tile += (int64_t)gridDim.x * 4) {
        f32x16 acc[OB][2];
#pragma unroll
        for (int ob = 0; ob < OB; ++ob)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ob][0][r] = acc[ob][1][r] = 0.f;
        const int64_t r0 = tile * 64 + jl, r1 = r0 + 32;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const bf16x8 b0 = load_row8(X, rows, r0, KIN, kb * 16 + 8 * h);
            const bf16x8 b1 = load_row8(X, rows, r1, KIN, kb * 16 + 8 * h);
#pragma unroll
            for (int ob = 0; ob < OB; ++ob) {
                const bf16x8 a = s_a[(ob * KB + kb) * 64 + lane];
                acc[ob][0] = mfma32(a, b0, acc[ob][0]);
                acc[ob][1] = mfma32(a, b1, acc[ob][1]);
            }
        }
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int64_t row = tile * 64 + jb * 32 + jl;
            if (row >= rows) continue;
#pragma unroll
            for (int ob = 0; ob < OB; ++ob)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const int i0 = ob * 32 + 8 * gq + 4 * h;
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[ob][jb][4 * gq + e];
                    if (EPI == EPI_BIAS || EPI == EPI_BIAS_RELU) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += s_bias[i0 + e];
                    }
                    if (EPI == EPI_BIAS_RELU) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
                    }
                    if (EPI == EPI_MASK) {
                        const f32x4 m = *reinterpret_cast<const f32x4 *>(mask + row * NOUT + i0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = m[e] > 0.f ? v[e] : 0.f;
                    }
                    *reinterpret_cast<f32x4 *>(Y + row * NOUT + i0) = v;
                }
        }
    }
}

// ------------------------------------------------------- weight grads ----
constexpr int kLD = 64 + 8;  // bf16 per LDS row of a transposed 64-row tile

// dW[128][KIN] += sum_rows G[row][o] X[row][k];  db[o] += sum_rows G[row][o]
template <int KIN>
__global__ __launch_bounds__(kThreads) void wgrad_kernel(const float *__restrict__ G,
                                                         const float *__restrict__ X,
                                                         int64_t rows, float *__restrict__ dW,
                                                         float *__restrict__ db) {
    constexpr int JB = KIN / 32;
    __shared__ __attribute__((aligned(16))) __bf16 s_g[kH * kLD];
    __shared__ __attribute__((aligned(16))) __bf16 s_x[KIN * kLD];
    __shared__ float s_red[8][kH];
    const int tid = threadIdx.x;
    const int lane = tid & 63, ob = tid >> 6, h = lane >> 5, jl = lane & 31;
    f32x16 acc[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[jb][r] = 0.f;
    float bsum[4] = {0.f, 0.f, 0.f, 0.f};
    const int c4 = tid & 31;
    const int64_t ntiles = ceil_div(rows, 64);
    // the next tile's rows are loaded into registers while the current one's
    // MFMAs run
    constexpr int XQ = 64 * KIN / 4;             // float4 per X tile
    constexpr int XPT = XQ / kThreads;           // per thread
    f32x4 gv[8], xv[XPT];
    auto fetch = [&](int64_t tile) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int64_t gr = tile * 64 + s * 8 + (tid >> 5);
            gv[s] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (gr < rows) gv[s] = *reinterpret_cast<const f32x4 *>(G + gr * kH + 4 * c4);
        }
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int q = tid + i * kThreads;
            const int64_t gr = tile * 64 + q / (KIN / 4);
            xv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (gr < rows) xv[i] = *reinterpret_cast<const f32x4 *>(X + gr * KIN + 4 * (q % (KIN / 4)));
        }
    };
    if ((int64_t)blockIdx.x < ntiles) fetch(blockIdx.x);
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int row = s * 8 + (tid >> 5);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bsum[e] += (float)f2bf(gv[s][e]);  // the bf16 G that the MFMA takes
                s_g[(4 * c4 + e) * kLD + row] = f2bf(gv[s][e]);
            }
        }
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int q = tid + i * kThreads;
            const int row = q / (KIN / 4), cc = q % (KIN / 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) s_x[(4 * cc + e) * kLD + row] = f2bf(xv[i][e]);
        }
        __syncthreads();
        if (tile + gridDim.x < ntiles) fetch(tile + gridDim.x);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&s_g[(ob * 32 + jl) * kLD + kb * 16 + 8 * h]);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                const bf16x8 b =
                    *reinterpret_cast<const bf16x8 *>(&s_x[(jb * 32 + jl) * kLD + kb * 16 + 8 * h]);
                acc[jb] = mfma32(a, b, acc[jb]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = ob * 32 + d_row(r, lane);
            unsafeAtomicAdd(dW + o * KIN + jb * 32 + jl, acc[jb][r]);
        }
#pragma unroll
    for (int e = 0; e < 4; ++e) s_red[tid >> 5][4 * c4 + e] = bsum[e];
    __syncthreads();
    if (tid < kH) {
        float s = 0.f;
        for (int p = 0; p < 8; ++p) s += s_red[p][tid];
        unsafeAtomicAdd(db + tid, s);
    }
}

// ------------------------------------------------------- small kernels ----
// M[b] = E[b] * E[B + b] over latents of `width` features (128, or the 32 grid
// features of a grid-only network)
__global__ void merge_fwd_kernel(const float *__restrict__ E, int64_t B, float *__restrict__ M,
                                 int width) {
    const int64_t n4 = B * width / 4;
    const f32x4 *a = reinterpret_cast<const f32x4 *>(E);
    const f32x4 *b = reinterpret_cast<const f32x4 *>(E + B * width);
    f32x4 *m = reinterpret_cast<f32x4 *>(M);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * blockDim.x)
        m[i] = a[i] * b[i];
}

__global__ void merge_bwd_kernel(const float *__restrict__ dM, const float *__restrict__ E,
                                 int64_t B, float *__restrict__ dE, int width) {
    const int64_t n4 = B * width / 4;
    const f32x4 *d = reinterpret_cast<const f32x4 *>(dM);
    const f32x4 *a = reinterpret_cast<const f32x4 *>(E);
    const f32x4 *b = reinterpret_cast<const f32x4 *>(E + B * width);
    f32x4 *da = reinterpret_cast<f32x4 *>(dE);
    f32x4 *dbp = reinterpret_cast<f32x4 *>(dE + B * width);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * blockDim.x) {
        const f32x4 g = d[i];
        da[i] = g * b[i];
        dbp[i] = g * a[i];
    }
}

// y = w6 . d2 + b6; with targets: gy = sign(y - t) / B and per-block sums of |y - t|.
__global__ __launch_bounds__(kThreads) void head_fwd_kernel(
    const float *__restrict__ D2, const float *__restrict__ w6, const float *__restrict__ b6,
    const float *__restrict__ targets, int64_t B, float *__restrict__ y, float *__restrict__ gy,
    double *__restrict__ partial) {
    __shared__ float s_w[kH];
    __shared__ double s_sum[kThreads / 64];
    for (int i = threadIdx.x; i < kH; i += kThreads) s_w[i] = w6[i];
    __syncthreads();
    const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double ab = 0.0;
    if (b < B) {
        const f32x4 *d = reinterpret_cast<const f32x4 *>(D2 + b * kH);
        float s = 0.f;
#pragma unroll 8
        for (int q = 0; q < kH / 4; ++q) {
            const f32x4 v = d[q];
            s = fmaf(v[0], s_w[4 * q], s);
            s = fmaf(v[1], s_w[4 * q + 1], s);
            s = fmaf(v[2], s_w[4 * q + 2], s);
            s = fmaf(v[3], s_w[4 * q + 3], s);
        }
        const float yy = s + b6[0];
        y[b] = yy;
        if (targets) {
            const float r = yy - targets[b];
            gy[b] = (r > 0.f ? 1.f : (r < 0.f ? -1.f : 0.f)) / (float)B;
            ab = fabs((double)r);
        }
    }
    if (targets) {
        ab = wave_sum_f64(ab);
        if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = ab;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int i = 0; i < kThreads / 64; ++i) t += s_sum[i];
            partial[blockIdx.x] = t;
        }
    }
}

// Mean of the per-block sums; a non-finite loss (a NaN or infinite target or
// output) sets the call's status word, which stops the optimiser step.
// One wave.
__device__ __forceinline__ void loss_reduce(const double *__restrict__ partial, int n, int64_t B,
                                            float *__restrict__ loss,
                                            int32_t *__restrict__ status) {
    double t = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64) t += partial[i];
    t = wave_sum_f64(t);
    if ((threadIdx.x & 63) == 0) {
        const float l = (float)(t / (double)B);
        loss[0] = l;
        if (!isfinite(l)) status[0] = NDF_E_NONFINITE;
    }
}

__global__ void loss_reduce_kernel(const double *__restrict__ partial, int n, int64_t B,
                                   float *__restrict__ loss, int32_t *__restrict__ status) {
    loss_reduce(partial, n, B, loss, status);
}

// dPre5 = gy w6 (masked by d2 > 0);  gw6 += sum_b gy d2;  gb6 += sum_b gy
__global__ __launch_bounds__(kThreads) void head_bwd_kernel(const float *__restrict__ D2,
                                                            const float *__restrict__ gy,
                                                            const float *__restrict__ w6, int64_t B,
                                                            float *__restrict__ dpre,
                                                            float *__restrict__ gw6,
                                                            float *__restrict__ gb6) {
    __shared__ float s_red[2][kH];
    __shared__ float s_b[2];
    const int c = threadIdx.x & (kH - 1);
    const int ph = threadIdx.x >> 7;
    const float wc = w6[c];
    float acc = 0.f, accb = 0.f;
    for (int64_t b = (int64_t)blockIdx.x * 2 + ph; b < B; b += (int64_t)gridDim.x * 2) {
        const float g = gy[b];
        const float d = D2[b * kH + c];
        dpre[b * kH + c] = d > 0.f ? g * wc : 0.f;
        acc = fmaf(g, (float)f2bf(d), acc);  // d2 as a bf16 operand, like every weight grad
        accb += g;
    }
    s_red[ph][c] = acc;
    if (c == 0) s_b[ph] = accb;
    __syncthreads();
    if (threadIdx.x < kH) unsafeAtomicAdd(gw6 + c, s_red[0][c] + s_red[1][c]);
    if (threadIdx.x == 0) unsafeAtomicAdd(gb6, s_b[0] + s_b[1]);
}

__global__ void adam_kernel(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                            const float *__restrict__ g, int64_t n, float lr, float c1, float c2,
                            const int32_t *__restrict__ status) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    if (status[0] != NDF_OK) return;  // the step's loss was not finite: keep p, m, v
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    }
}

// ------------------------------------------------------------ host side ----
namespace {

struct TrainWS {
    int32_t *status;
    float *H0, *H1, *H2, *E, *M, *D1, *D2, *y, *gy, *dA, *dB, *dH0;
    double *partial;
    size_t bytes;
};

TrainWS carve(void *ws, int64_t B) {
    TrainWS t{};
    const int64_t R = 2 * B;
    char *base = (char *)ws;
    size_t pos = 0;
    auto take = [&](size_t n) {
        char *p = base ? base + pos : nullptr;
        pos += align_up(n, 256);
        return p;
    };
    t.status = (int32_t *)take(kStatusBytes);
    t.H0 = (float *)take(R * kK0 * 4);
    t.H1 = (float *)take(R * kH * 4);
    t.H2 = (float *)take(R * kH * 4);
    t.E = (float *)take(R * kH * 4);
    t.M = (float *)take(B * kH * 4);
    t.D1 = (float *)take(B * kH * 4);
    t.D2 = (float *)take(B * kH * 4);
    t.y = (float *)take(B * 4);
    t.gy = (float *)take(B * 4);
    t.dA = (float *)take(R * kH * 4);
    t.dB = (float *)take(R * kH * 4);
    t.dH0 = (float *)take(R * kK0 * 4);
    t.partial = (double *)take(ceil_div(B, kThreads) * 8);
    t.bytes = pos;
    return t;
}

unsigned mma_blocks(int64_t rows) {
    int64_t b = ceil_div(ceil_div(rows, 64), 4);
    return (unsigned)(b < 1024 ? (b > 0 ? b : 1) : 1024);
}
// dL/dh0 of 2 B rows added to the grid levels directly.
void scatter_direct(float *G, const GridOffs &go, const GridGeom &g, int n_enc,
                    const int64_t *pairs, const float *pos, int64_t B, const float *dh0,
                    hipStream_t st) {
    const int64_t b = ceil_div(2 * B * kL, 4 * (kThreads / 64));  // 4 items per wave
    hipLaunchKernelGGL(grid_bwd_kernel, dim3((unsigned)(b < 8192 ? b : 8192)), dim3(kThreads), 0,
                       st, G, go, g, n_enc, pairs, pos, B, dh0);
}
unsigned wgrad_blocks(int64_t rows) {
    int64_t b = ceil_div(rows, 64);
    return (unsigned)(b < 512 ? (b > 0 ? b : 1) : 512);  // 2 per CU: 222 -> 156 us at 2^19 rows
}

GridOffs grid_offs(const NetOffsets &o) {
    GridOffs g{};
    for (int e = 0; e < 2; ++e)
        for (int l = 0; l < kL; ++l) g.off[e][l] = o.grid[e][l];
    return g;
}

// Y = X A^T of one layer over `rows` rows (rows_mma_kernel).
template <int KIN, int NOUT, int EPI>
void rows_layer(const float *X, int64_t rows, const float *W, int w_si, int w_sk,
                const float *bias, const float *mask, float *Y, hipStream_t st) {
    hipLaunchKernelGGL((rows_mma_kernel<KIN, NOUT, EPI>), dim3(mma_blocks(rows)), dim3(kThreads),
                       0, st, X, rows, W, w_si, w_sk, bias, mask, Y);
}
template <int KIN>
void rows_wgrad(const float *G, const float *X, int64_t rows, float *dW, float *db,
                hipStream_t st) {
    hipLaunchKernelGGL(wgrad_kernel<KIN>, dim3(wgrad_blocks(rows)), dim3(kThreads), 0, st, G, X,
                       rows, dW, db);
}

// Forward pass, layer by layer, into the workspace; with targets also the loss and gy.
void forward(const ndf_net_config *c, const NetOffsets &o, const float *P, const int64_t *pairs,
             const float *pos, const float *targets, int64_t B, const TrainWS &t,
             hipStream_t st) {
    const int64_t R = 2 * B;
    const GridGeom g = grid_geom(c);
    const GridOffs go = grid_offs(o);
    hipLaunchKernelGGL(grid_fwd_kernel, dim3((unsigned)ceil_div(R * kL, kThreads)), dim3(kThreads),
                       0, st, P, go, g, c->n_enc, pairs, pos, B, t.H0);
    if (c->grid_only) {
        // the grid features are the latents: merge them and decode (W4 is [128][32])
        hipLaunchKernelGGL(merge_fwd_kernel, dim3(gs_blocks(B * kK0 / 4)), dim3(kThreads), 0, st,
                           t.H0, B, t.M, kK0);
        rows_layer<kK0, kH, EPI_BIAS_RELU>(t.M, B, P + o.W4, kK0, 1, P + o.b4, nullptr, t.D1, st);
    } else {  // two encoders
        for (int e = 0; e < 2; ++e) {
            const int64_t r0 = e * B;
            rows_layer<kK0, kH, EPI_BIAS_RELU>(t.H0 + r0 * kK0, B, P + o.W1[e], kK0, 1, P + o.b1[e],
                                               nullptr, t.H1 + r0 * kH, st);
            rows_layer<kH, kH, EPI_BIAS_RELU>(t.H1 + r0 * kH, B, P + o.W2[e], kH, 1, P + o.b2[e],
                                              nullptr, t.H2 + r0 * kH, st);
            rows_layer<kH, kH, EPI_BIAS>(t.H2 + r0 * kH, B, P + o.W3[e], kH, 1, P + o.b3[e],
                                         nullptr, t.E + r0 * kH, st);
        }
        hipLaunchKernelGGL(merge_fwd_kernel, dim3(gs_blocks(B * kH / 4)), dim3(kThreads), 0, st,
                           t.E, B, t.M, kH);
        rows_layer<kH, kH, EPI_BIAS_RELU>(t.M, B, P + o.W4, kH, 1, P + o.b4, nullptr, t.D1, st);
    }
    rows_layer<kH, kH, EPI_BIAS_RELU>(t.D1, B, P + o.W5, kH, 1, P + o.b5, nullptr, t.D2, st);
    hipLaunchKernelGGL(head_fwd_kernel, dim3((unsigned)ceil_div(B, kThreads)), dim3(kThreads), 0,
                       st, t.D2, P + o.w6, P + o.b6, targets, B, t.y, t.gy, t.partial);
}

// ========================================================== fused step ====
// The step of a network with one encoder shared by both endpoints (the
// symmetric pair encoding of Sec. 4.1) runs in these kernels after a packing one: a forward
// kernel (grid gather, encoder for both endpoints, latent product, decoder, head, the
// L1 loss and its gradient), a backward kernel (the data adjoint from the head
// back to dL/dh0), the grid scatter (grid_bwd_kernel, or grid_tile_kernel after a sort)
// and one kernel for every weight and bias gradient.  A wave takes 32 pairs: the first endpoints are
// MFMA column block q = 0, the second endpoints q = 1, so both share every
// weight fragment and the latent product is register-local; the decoder runs
// on the pair rows (q = 0).
// What the backward pass and the weight gradients need is stored per 32-row
// block ("slab") in the register order of the MFMA operands: chunk (kb, lane)
// = 16 bytes = row lane % 32, features feat_perm(kb, lane / 32, e) for layer
// outputs (the order the MFMA accumulators pack into) and feat_nat for the grid
// features h0.  Every store and load of a slab is a coalesced 16-byte access.
// With two encoders (cross-variable fields) the weights of both and the decoder exceed a
// CU's LDS, so the forward and the backward kernel each become an encoder and a decoder
// kernel: the encoder kernels take 64 rows of one endpoint per wave (both MFMA column
// blocks, its encoder's weights in LDS), the decoder kernels 32 pairs.  Slab block of pair
// block t and endpoint e: 2 t + e with a shared encoder, e T + t with two (an encoder's
// slabs are then one range for the weight gradients).
// Numerics are those of a layer-by-layer evaluation: bf16 operands into every
// MFMA, FP32 accumulators, FP32 latents into the product; the stored operands
// of the weight gradients are the same bf16 values the MFMAs take, and bias
// gradients sum those bf16 values (a bias is the weight of a constant input 1).
__host__ __device__ inline int feat_perm(int kb, int h, int e) {
    return 16 * kb + 8 * (e >> 2) + 4 * h + (e & 3);
}
__host__ __device__ inline int feat_nat(int kb, int h, int e) { return 16 * kb + 8 * h + e; }

constexpr int kTW = 8;                 // waves per workgroup of the fused kernels
constexpr int kTThreads = 64 * kTW;
constexpr int kFragH = 4 * 8 * 64;     // bf16x8 per 128 x 128 layer fragment set
constexpr int kFrag1 = 4 * 2 * 64;     // W1 (128 x 32), and W1^T (32 x 128): 8 x 64
constexpr int kFrag1F = 4 * 7 * 64;    // W1 with Fourier features (128 x 112)

// Packed weights of one step.  Matrices: W1, W2, W3 of each encoder, then W4, W5 (index
// 3 e + l, 3 n_enc + l).  f: forward A fragments (W[o][k], lane l
// of fragment (ob, kb) holds row 32 ob + l % 32, inputs 8 (l / 32) + 16 kb + e in
// the order of the layer's input); t: the adjoint's A fragments of the
// transposed matrices (row = the layer's input k, inputs = its outputs o in the packed
// gradient's order feat_perm; of W1 the 32 grid inputs only, since no gradient flows
// into the Fourier features).  With two encoders every layer's inputs are in the order
// feat_nat (operand<true>) and biases are added last, as in the layer-by-layer kernels:
// every activation and gradient is then the same number bit for bit, whichever run.
constexpr int kMaxMats = 8;

struct TrainFrags {
    bf16x8 *f[kMaxMats];
    bf16x8 *t[kMaxMats];
};

// With G the gradient (n floats, 256-byte aligned) and the status word are cleared too:
// one launch in front of the forward kernel instead of three.
constexpr int kPackBlocks = 16;  // per matrix

struct PackArgs {
    int64_t w[kMaxMats];  // offsets of the matrices in P
    int n_enc, kin1;
    TrainFrags F;
};

__global__ void pack_train_kernel(const float *__restrict__ P, PackArgs A, float *__restrict__ G,
                                  int64_t n, int32_t *__restrict__ status) {
    const int n_mat = 3 * A.n_enc + 2, pack = kPackBlocks * n_mat;
    if ((int)blockIdx.x >= pack) {
        const int64_t n4 = n / 4, step = (int64_t)(gridDim.x - pack) * blockDim.x;
        const int64_t t0 = (int64_t)(blockIdx.x - pack) * blockDim.x + threadIdx.x;
        for (int64_t i = t0; i < n4; i += step)
            reinterpret_cast<f32x4 *>(G)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int64_t i = 4 * n4 + t0; i < n; i += step) G[i] = 0.f;
        return;
    }
    if (status && blockIdx.x == 0 && threadIdx.x == 0) *status = NDF_OK;
    const int L = blockIdx.x / kPackBlocks;
    const bool first = L < 3 * A.n_enc && L % 3 == 0;  // a W1
    const bool nat = A.n_enc == 2;
    const int KIN = first ? A.kin1 : kH, KB = KIN / 16;
    const int nf = kH * KIN, na = kH * (first ? kK0 : kH);
    const float *W = P + A.w[L];
    __bf16 *df = reinterpret_cast<__bf16 *>(A.F.f[L]), *dt = reinterpret_cast<__bf16 *>(A.F.t[L]);
    for (int u = (blockIdx.x % kPackBlocks) * blockDim.x + threadIdx.x; u < nf + na;
         u += kPackBlocks * blockDim.x) {
        const bool adj = u >= nf;
        const int v = adj ? u - nf : u;
        const int e = v & 7, lane = (v >> 3) & 63, fi = v >> 9;
        const int h = lane >> 5, il = lane & 31;
        if (!adj) {
            const int ob = fi / KB, kb = fi % KB;
            const int k = first || nat ? feat_nat(kb, h, e) : feat_perm(kb, h, e);
            df[v] = f2bf(W[(int64_t)(32 * ob + il) * KIN + k]);
        } else {
            const int mb = fi / 8, kb = fi % 8;
            const int o = nat ? feat_nat(kb, h, e) : feat_perm(kb, h, e);
            dt[v] = f2bf(W[(int64_t)o * KIN + 32 * mb + il]);
        }
    }
}

struct FusedArgs {
    const float *P;
    int64_t grid[kL];  // offsets of the (first) encoder's grid levels in P
    const bf16x8 *wf[5], *wt[5];
    const float *b[5], *w6, *b6;
    // two encoders: the second one's grid levels, W1..W3 and b1..b3
    int64_t grid1[kL];
    const bf16x8 *wf1[3], *wt1[3];
    const float *b1[3];
    GridGeom g;
    const int64_t *pairs;
    const float *pos;
    const float *targets;
    int64_t B;
    // slabs: enc = [2 T] (block 2 t + q), dec = [T]
    u32x4 *h0, *h1, *h2, *m, *d1, *d2, *da5, *da4, *dlat, *da2, *da1;
    f32x4 *lat;     // FP32 latents [2 T][4 ob][4 g][64]
    float *gy;      // [T * 32]
    float *y;       // [B] or null
    float *dh0;     // [2 B][32] FP32, rows q B + pair
    double *partial;
    int n_partial;  // workgroups of the forward kernel
    float *loss;
    int32_t *status;
};

__device__ __forceinline__ int64_t slab_chunk(int64_t blk, int nkb, int kb, int lane) {
    return (blk * nkb + kb) * 64 + lane;
}

// Pack one output block's accumulators (acc index 8 s + e <-> chunk 2 ob + s,
// element e) into two bf16 chunks.
__device__ __forceinline__ void pack_block(const f32x16 &acc, u32x4 &c0, u32x4 &c1) {
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
        c0[e2] = pack_bf16x2(acc[2 * e2], acc[2 * e2 + 1]);
        c1[e2] = pack_bf16x2(acc[8 + 2 * e2], acc[8 + 2 * e2 + 1]);
    }
}

// A packed chunk as the next layer's operand: as it is (inputs in the order feat_perm), or
// (NAT) in the order feat_nat, which exchanges the second four features of lanes 0-31
// with the first four of lanes 32-63.
template <bool NAT>
__device__ __forceinline__ bf16x8 operand(u32x4 c) {
    if (NAT) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const auto r = __builtin_amdgcn_permlane32_swap(c[i], c[2 + i], false, false);
            c[i] = r[0];
            c[2 + i] = r[1];
        }
    }
    return __builtin_bit_cast(bf16x8, c);
}

// Keep the halves of g whose forward activation (bf16 pair h, a ReLU output, so
// +0 or positive) is non-zero: the ReLU derivative on packed pairs.
__device__ __forceinline__ uint32_t relu_mask2(uint32_t g, uint32_t h) {
    const uint32_t lo = (h & 0xffffu) ? 0xffffu : 0u;
    const uint32_t hi = (h >> 16) ? 0xffff0000u : 0u;
    return g & (lo | hi);
}

// acc[q] = bias (or 0) + W-block ob x in[.][q] over KB k-blocks; NAT adds the bias last.
template <int KB, int NQ, bool NAT = false>
__device__ __forceinline__ void mma_block(const bf16x8 *__restrict__ wf, int ob,
                                          const float *__restrict__ bias_h,
                                          const bf16x8 (&in)[8][2], f32x16 (&acc)[2], int lane) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        f32x4 bv = {0.f, 0.f, 0.f, 0.f};
        if (bias_h && !NAT) bv = *reinterpret_cast<const f32x4 *>(bias_h + 32 * ob + 8 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q][4 * g + i] = bv[i];
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const bf16x8 a = wf[(ob * KB + kb) * 64 + lane];
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q] = mfma32(a, in[kb][q], acc[q]);
    }
    if (bias_h && NAT) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias_h + 32 * ob + 8 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int q = 0; q < NQ; ++q) acc[q][4 * g + i] += bv[i];
        }
    }
}

// Grid features of one endpoint for k-block kb: lane half h gathers level
// 2 kb + h (8 FP32 features per cell, trilinear over 8 corners).
template <bool POS>
__device__ __forceinline__ bf16x8 gather_h0(const FusedArgs &A, const int64_t (&goff)[kL], int kb,
                                            int h, int64_t v, const float (&p)[3], bool few) {
    const int l = 2 * kb + h;
    int R[3];
    level_dims(A.g, l, R);
    const uint32_t hm = level_hmask(A.g, l);
    int idx[8];
    float w[8];
    if (POS)
        corners_pos32<true>(R, p, idx, w, hm);
    else
        corners_R32<true>(A.g, R, v, idx, w, hm);
    const f32x4 *grid = reinterpret_cast<const f32x4 *>(A.P + (h ? goff[2 * kb + 1] : goff[2 * kb]));
    // A corner of weight 0 adds nothing, and on a level of the vertex grid's size only one
    // corner of eight has weight.  With many waves in flight the others are skipped; a
    // branch around each read waits for it before the next is issued, so with few waves
    // (`few`, uniform) they read the last weighted corner's cell instead and leave it out of
    // the sum (0 times an infinite feature is not 0).
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
    auto add = [&](float wc, const f32x4 &c0, const f32x4 &c1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a0 = fmaf(wc, c0[i], s0[i]), a1 = fmaf(wc, c1[i], s1[i]);
            s0[i] = wc != 0.f ? a0 : s0[i];
            s1[i] = wc != 0.f ? a1 : s1[i];
        }
    };
    if (few) {
        int some = idx[0];
#pragma unroll
        for (int c = 1; c < 8; ++c) some = w[c] != 0.f ? idx[c] : some;
        f32x4 c0[8], c1[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int64_t at = 2 * (int64_t)(w[c] != 0.f ? idx[c] : some);
            c0[c] = grid[at];
            c1[c] = grid[at + 1];
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) add(w[c], c0[c], c1[c]);
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (w[c] != 0.f) add(w[c], grid[2 * (int64_t)idx[c]], grid[2 * (int64_t)idx[c] + 1]);
    }
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        t[i] = f2bf(s0[i]);
        t[4 + i] = f2bf(s1[i]);
    }
    return t;
}

__device__ __forceinline__ u32x4 as_u(const bf16x8 &v) { return __builtin_bit_cast(u32x4, v); }
__device__ __forceinline__ bf16x8 as_b(const u32x4 &v) { return __builtin_bit_cast(bf16x8, v); }

// Decoder of 32 pairs from the packed latent product b: W4, W5, the head
// y = w6 . d2 + b6; with targets gy, da5 and this lane's |y - t|, which is returned.
template <bool NAT>
__device__ __forceinline__ double decode_pairs(const FusedArgs &A, int64_t tile,
                                               const bf16x8 *__restrict__ w4,
                                               const bf16x8 *__restrict__ w5,
                                               const float *__restrict__ s_b4,
                                               const float *__restrict__ s_b5,
                                               const float *__restrict__ s_w6, bf16x8 (&b)[8][2],
                                               bf16x8 (&a)[8][2], int lane, int h4) {
    const int h = lane >> 5, jl = lane & 31;
    const int64_t pair = tile * 32 + jl;
    const bool ok = pair < A.B;
    const float b6 = A.b6[0], inv_b = 1.f / (float)A.B;
    double loss_part = 0.0;
    f32x16 acc[2];
    // layer 4: ReLU (pair rows)
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        mma_block<8, 1, NAT>(w4, ob, s_b4 + h4, b, acc, lane);
        u32x4 c0, c1;
        pack_block(acc[0], c0, c1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c0[i] = relu_bf16x2(c0[i]);
            c1[i] = relu_bf16x2(c1[i]);
        }
        a[2 * ob][0] = operand<NAT>(c0);
        a[2 * ob + 1][0] = operand<NAT>(c1);
        A.d1[slab_chunk(tile, 8, 2 * ob, lane)] = c0;
        A.d1[slab_chunk(tile, 8, 2 * ob + 1, lane)] = c1;
        __builtin_amdgcn_sched_barrier(0);
    }
    // layer 5: ReLU, and the head y = w6 . d2 + b6 in FP32
    float part = 0.f;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        mma_block<8, 1, NAT>(w5, ob, s_b5 + h4, a, acc, lane);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 wv = *reinterpret_cast<const f32x4 *>(s_w6 + h4 + 32 * ob + 8 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[0][4 * g + i] = relu_f32(acc[0][4 * g + i]);
                part = fmaf(wv[i], acc[0][4 * g + i], part);
            }
        }
        u32x4 c0, c1;
        pack_block(acc[0], c0, c1);
        b[2 * ob][0] = as_b(c0);
        b[2 * ob + 1][0] = as_b(c1);
        A.d2[slab_chunk(tile, 8, 2 * ob, lane)] = c0;
        A.d2[slab_chunk(tile, 8, 2 * ob + 1, lane)] = c1;
        __builtin_amdgcn_sched_barrier(0);
    }
    const float y = part + __shfl_xor(part, 32, 64) + b6;
    if (A.y && h == 0 && ok) A.y[pair] = y;
    if (A.targets) {
        const float r = ok ? y - A.targets[pair] : 0.f;
        const float gyv = (r > 0.f ? 1.f : (r < 0.f ? -1.f : 0.f)) * inv_b;
        if (h == 0) {
            A.gy[tile * 32 + jl] = gyv;
            loss_part = ok ? fabs((double)r) : 0.0;
        }
        // da5 = gy w6 where d2 > 0, in the packed order of d2
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32x4 dd = as_u(b[j][0]);
            u32x4 c;
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                const int f0 = feat_perm(j, 0, 2 * e2) + h4;
                c[e2] = relu_mask2(pack_bf16x2(gyv * s_w6[f0], gyv * s_w6[f0 + 1]), dd[e2]);
            }
            A.da5[slab_chunk(tile, 8, j, lane)] = c;
        }
    }
    return loss_part;
}

// Per-workgroup loss partial sum (with targets).
__device__ __forceinline__ void store_loss_part(const FusedArgs &A, double loss_part,
                                                double *s_part) {
    if (A.targets) {
        loss_part = wave_sum_f64(loss_part);
        if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = loss_part;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < kTW; ++w) t += s_part[w];
            A.partial[blockIdx.x] = t;
        }
    }
}

// First tile of a wave; the next ones follow at gridDim.x kTW.  Up to one tile per wave
// the tiles are dealt to the workgroups first (few tiles then run on many CUs), else a
// workgroup's waves take neighbouring tiles (their slabs are neighbours in memory).
__device__ __forceinline__ int64_t first_tile(int64_t T, int wave) {
    return T <= (int64_t)gridDim.x * kTW ? blockIdx.x + (int64_t)gridDim.x * wave
                                         : (int64_t)blockIdx.x * kTW + wave;
}

// Forward of 32 pairs per wave; with targets also the loss partial sums, gy and
// the first gradient da5 = gy w6 (masked by d2 > 0).
template <bool POS, bool FF>
__global__ __launch_bounds__(kTThreads) void train_fwd_kernel(FusedArgs A) {
    constexpr int KB1 = FF ? kK0F / 16 : kK0 / 16;  // k-blocks of the encoder input
    __shared__ bf16x8 s_w1[4 * KB1 * 64];
    __shared__ bf16x8 s_w[4][kFragH];
    __shared__ __attribute__((aligned(16))) float s_b[5][kH];
    __shared__ __attribute__((aligned(16))) float s_w6[kH];
    __shared__ double s_part[kTW];
    const int tid = threadIdx.x;
    stage_lds<4 * KB1 * 64, kTThreads>(s_w1, A.wf[0], tid);
#pragma unroll
    for (int L = 0; L < 4; ++L) stage_lds<kFragH, kTThreads>(s_w[L], A.wf[L + 1], tid);
    for (int i = tid; i < 5 * kH; i += kTThreads) s_b[i / kH][i % kH] = A.b[i / kH][i % kH];
    for (int i = tid; i < kH; i += kTThreads) s_w6[i] = A.w6[i];
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    const int64_t T = ceil_div(A.B, 32);
    const int64_t V = (int64_t)A.g.nx * A.g.ny * A.g.nz;
    const bool few = T <= 2 * (int64_t)gridDim.x;  // at most two waves of a CU gather
    double loss_part = 0.0;
    for (int64_t tile = first_tile(T, wave); tile < T; tile += (int64_t)gridDim.x * kTW) {
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        const int64_t pair = tile * 32 + jl;
        const bool ok = pair < A.B;
        bf16x8 a[8][2], b[8][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int64_t v = 0;
            float p[3] = {0.f, 0.f, 0.f};
            if (ok) {
                if (POS) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) p[c] = A.pos[(2 * pair + q) * 3 + c];
                } else {
                    v = A.pairs[2 * pair + q];
                    v = v < 0 ? 0 : (v >= V ? V - 1 : v);  // out-of-range pairs are clamped
                }
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                a[kb][q] = gather_h0<POS>(A, A.grid, kb, h, v, p, few);
                A.h0[slab_chunk(2 * tile + q, KB1, kb, lane)] = as_u(a[kb][q]);
            }
            if (FF) {  // the raw position and its Fourier features
                float pp[3];
                if (POS)
                    clamp_p(p, pp);
                else
                    vertex_p(A.g, v, pp);
#pragma unroll
                for (int kb = 2; kb < KB1; ++kb) {
                    a[kb][q] = ff_chunk(kb, h, pp);
                    A.h0[slab_chunk(2 * tile + q, KB1, kb, lane)] = as_u(a[kb][q]);
                }
            }
        }
        f32x16 acc[2];
        // layer 1: 32 -> 128, ReLU (both endpoints)
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            mma_block<KB1, 2>(s_w1, ob, s_b[0] + h4, a, acc, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 c0, c1;
                pack_block(acc[q], c0, c1);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    c0[i] = relu_bf16x2(c0[i]);
                    c1[i] = relu_bf16x2(c1[i]);
                }
                b[2 * ob][q] = as_b(c0);
                b[2 * ob + 1][q] = as_b(c1);
                A.h1[slab_chunk(2 * tile + q, 8, 2 * ob, lane)] = c0;
                A.h1[slab_chunk(2 * tile + q, 8, 2 * ob + 1, lane)] = c1;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // layer 2: ReLU
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            mma_block<8, 2>(s_w[0], ob, s_b[1] + h4, b, acc, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 c0, c1;
                pack_block(acc[q], c0, c1);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    c0[i] = relu_bf16x2(c0[i]);
                    c1[i] = relu_bf16x2(c1[i]);
                }
                a[2 * ob][q] = as_b(c0);
                a[2 * ob + 1][q] = as_b(c1);
                A.h2[slab_chunk(2 * tile + q, 8, 2 * ob, lane)] = c0;
                A.h2[slab_chunk(2 * tile + q, 8, 2 * ob + 1, lane)] = c1;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // layer 3: the latents (FP32, kept for the product rule) and their product
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            mma_block<8, 2>(s_w[1], ob, s_b[2] + h4, a, acc, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 t;
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] = acc[q][4 * g + i];
                    A.lat[((2 * tile + q) * 4 + ob) * 256 + g * 64 + lane] = t;
                }
            f32x16 mm;
#pragma unroll
            for (int r = 0; r < 16; ++r) mm[r] = acc[0][r] * acc[1][r];
            u32x4 c0, c1;
            pack_block(mm, c0, c1);
            b[2 * ob][0] = as_b(c0);
            b[2 * ob + 1][0] = as_b(c1);
            A.m[slab_chunk(tile, 8, 2 * ob, lane)] = c0;
            A.m[slab_chunk(tile, 8, 2 * ob + 1, lane)] = c1;
            __builtin_amdgcn_sched_barrier(0);
        }
        loss_part += decode_pairs<false>(A, tile, s_w[2], s_w[3], s_b[3], s_b[4], s_w6, b, a, lane, h4);
    }
    store_loss_part(A, loss_part, s_part);
}

// One encoder adjoint layer for both endpoints: out = pack(W^T in) masked by the
// forward activation hm > 0; the result is also stored as the layer's G slab.
__device__ __forceinline__ void adj_masked_layer(const bf16x8 *__restrict__ wt,
                                                 const u32x4 *__restrict__ hm,
                                                 u32x4 *__restrict__ gout, int64_t tile,
                                                 const bf16x8 (&in)[8][2], bf16x8 (&out)[8][2],
                                                 int lane) {
    f32x16 acc[2];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        mma_block<8, 2>(wt, ob, nullptr, in, acc, lane);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            u32x4 c0, c1;
            pack_block(acc[q], c0, c1);
            const u32x4 m0 = hm[slab_chunk(2 * tile + q, 8, 2 * ob, lane)];
            const u32x4 m1 = hm[slab_chunk(2 * tile + q, 8, 2 * ob + 1, lane)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                c0[i] = relu_mask2(c0[i], m0[i]);
                c1[i] = relu_mask2(c1[i], m1[i]);
            }
            out[2 * ob][q] = as_b(c0);
            out[2 * ob + 1][q] = as_b(c1);
            gout[slab_chunk(2 * tile + q, 8, 2 * ob, lane)] = c0;
            gout[slab_chunk(2 * tile + q, 8, 2 * ob + 1, lane)] = c1;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// W5^T of 32 pairs: y = d(d1) masked by d1 > 0 from da5 (x, read here), stored as da4.
template <bool NAT>
__device__ __forceinline__ void adj_layer5(const FusedArgs &A, int64_t tile,
                                           const bf16x8 *__restrict__ w5t, bf16x8 (&x)[8][2],
                                           bf16x8 (&y)[8][2], int lane) {
    f32x16 acc[2];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) x[kb][0] = operand<NAT>(A.da5[slab_chunk(tile, 8, kb, lane)]);
    // W5^T: d(d1), masked by d1 > 0 -> da4
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        mma_block<8, 1>(w5t, ob, nullptr, x, acc, lane);
        u32x4 c0, c1;
        pack_block(acc[0], c0, c1);
        const u32x4 m0 = A.d1[slab_chunk(tile, 8, 2 * ob, lane)];
        const u32x4 m1 = A.d1[slab_chunk(tile, 8, 2 * ob + 1, lane)];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c0[i] = relu_mask2(c0[i], m0[i]);
            c1[i] = relu_mask2(c1[i], m1[i]);
        }
        y[2 * ob][0] = operand<NAT>(c0);
        y[2 * ob + 1][0] = operand<NAT>(c1);
        A.da4[slab_chunk(tile, 8, 2 * ob, lane)] = c0;
        A.da4[slab_chunk(tile, 8, 2 * ob + 1, lane)] = c1;
        __builtin_amdgcn_sched_barrier(0);
    }
}

// dL/dh0 of one row (32 features: level g = 0..3, features 4 h + i).
__device__ __forceinline__ void store_dh0(const FusedArgs &A, int64_t row, const f32x16 &acc,
                                          int h) {
    float *dst = A.dh0 + row * kK0 + 4 * h;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        f32x4 t;
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = acc[4 * g + i];
        *reinterpret_cast<f32x4 *>(dst + 8 * g) = t;
    }
}

// Data adjoint of 32 pairs per wave: da5 -> da4 -> dlat (both endpoints) -> da2
// -> da1 -> dL/dh0 (FP32, rows q B + pair, for the grid scatter).  Every G slab
// is stored for the weight gradients.
__global__ __launch_bounds__(kTThreads) void train_bwd_kernel(FusedArgs A) {
    __shared__ bf16x8 s_t1[kFrag1];
    __shared__ bf16x8 s_t[4][kFragH];  // W2^T .. W5^T
    const int tid = threadIdx.x;
    stage_lds<kFrag1, kTThreads>(s_t1, A.wt[0], tid);
#pragma unroll
    for (int L = 0; L < 4; ++L) stage_lds<kFragH, kTThreads>(s_t[L], A.wt[L + 1], tid);
    if (blockIdx.x == 0 && tid < 64) loss_reduce(A.partial, A.n_partial, A.B, A.loss, A.status);
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    const int64_t T = ceil_div(A.B, 32);
    for (int64_t tile = first_tile(T, wave); tile < T; tile += (int64_t)gridDim.x * kTW) {
        const int64_t pair = tile * 32 + jl;
        const bool ok = pair < A.B;
        bf16x8 x[8][2], y[8][2];
        f32x16 acc[2];
        adj_layer5<false>(A, tile, s_t[3], x, y, lane);
        // W4^T: dm, then the product rule: dlat_A = dm lat_B, dlat_B = dm lat_A
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            mma_block<8, 1>(s_t[2], ob, nullptr, y, acc, lane);
            f32x16 la, lb;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 ta = A.lat[((2 * tile) * 4 + ob) * 256 + g * 64 + lane];
                const f32x4 tb = A.lat[((2 * tile + 1) * 4 + ob) * 256 + g * 64 + lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    la[4 * g + i] = acc[0][4 * g + i] * tb[i];
                    lb[4 * g + i] = acc[0][4 * g + i] * ta[i];
                }
            }
            u32x4 c0, c1;
            pack_block(la, c0, c1);
            x[2 * ob][0] = as_b(c0);
            x[2 * ob + 1][0] = as_b(c1);
            A.dlat[slab_chunk(2 * tile, 8, 2 * ob, lane)] = c0;
            A.dlat[slab_chunk(2 * tile, 8, 2 * ob + 1, lane)] = c1;
            pack_block(lb, c0, c1);
            x[2 * ob][1] = as_b(c0);
            x[2 * ob + 1][1] = as_b(c1);
            A.dlat[slab_chunk(2 * tile + 1, 8, 2 * ob, lane)] = c0;
            A.dlat[slab_chunk(2 * tile + 1, 8, 2 * ob + 1, lane)] = c1;
            __builtin_amdgcn_sched_barrier(0);
        }
        // W3^T: dh2, masked by h2 > 0 -> da2;  W2^T: dh1, masked by h1 > 0 -> da1
        adj_masked_layer(s_t[1], A.h2, A.da2, tile, x, y, lane);
        adj_masked_layer(s_t[0], A.h1, A.da1, tile, y, x, lane);
        // W1^T: dL/dh0 (32 features: level g = 0..3, features 4 h + i)
        mma_block<8, 2>(s_t1, 0, nullptr, x, acc, lane);
        if (ok) {
#pragma unroll
            for (int q = 0; q < 2; ++q) store_dh0(A, (int64_t)q * A.B + pair, acc[q], h);
        }
    }
}

// ------------------------------------------------------- two encoders ----
// Bound by the slabs' HBM stream like the shared-encoder kernels, plus the latents read back
// (32 KB per pair block in each direction).  A step of 2^16 pairs of the 250 x 352 x 20 grid:
// 165 us in these four kernels, 0.62 ms with packing, scatter, weight gradients and Adam
// over 37.8M parameters (0.21 ms); one kernel per layer with FP32 activations in HBM took
// 1.40 ms.
// One ReLU (MASKED: adjoint) layer of 64 rows: out = relu(W in + b), or W^T in masked by
// the forward activation hm > 0; stored as slab blocks blk[q] where st[q].
template <int KB, bool MASKED>
__device__ __forceinline__ void rows64_layer(const bf16x8 *__restrict__ wf,
                                             const float *__restrict__ bias_h,
                                             const u32x4 *__restrict__ hm,
                                             u32x4 *__restrict__ slab, const int64_t (&blk)[2],
                                             const bool (&st)[2], const bf16x8 (&in)[8][2],
                                             bf16x8 (&out)[8][2], int lane) {
    f32x16 acc[2];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        mma_block<KB, 2, true>(wf, ob, bias_h, in, acc, lane);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            u32x4 c0, c1;
            pack_block(acc[q], c0, c1);
            const int64_t i0 = slab_chunk(blk[q], 8, 2 * ob, lane),
                          i1 = slab_chunk(blk[q], 8, 2 * ob + 1, lane);
            u32x4 m0, m1;
            if (MASKED) {  // blk[q] is a real block even where nothing is stored
                m0 = hm[i0];
                m1 = hm[i1];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                c0[i] = MASKED ? relu_mask2(c0[i], m0[i]) : relu_bf16x2(c0[i]);
                c1[i] = MASKED ? relu_mask2(c1[i], m1[i]) : relu_bf16x2(c1[i]);
            }
            out[2 * ob][q] = operand<true>(c0);
            out[2 * ob + 1][q] = operand<true>(c1);
            if (st[q]) {
                slab[i0] = c0;
                slab[i1] = c1;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The two 32-pair blocks of a wave's tile of one endpoint: q = 1 of the last tile may lie
// past the last block (it then repeats the last one and stores nothing).
__device__ __forceinline__ void rows64_blocks(int64_t tile, int64_t T, int e, int64_t (&pb)[2],
                                              int64_t (&blk)[2], bool (&st)[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        st[q] = 2 * tile + q < T;
        pb[q] = st[q] ? 2 * tile + q : T - 1;
        blk[q] = e * T + pb[q];
    }
}

// Encoder forward: blockIdx.y = endpoint = encoder, 64 rows per wave.
template <bool POS>
__global__ __launch_bounds__(kTThreads) void train_enc_fwd_kernel(FusedArgs A) {
    __shared__ bf16x8 s_w1[kFrag1];
    __shared__ bf16x8 s_w[2][kFragH];
    __shared__ __attribute__((aligned(16))) float s_b[3][kH];
    const int tid = threadIdx.x, e = blockIdx.y;
    stage_lds<kFrag1, kTThreads>(s_w1, e ? A.wf1[0] : A.wf[0], tid);
    stage_lds<kFragH, kTThreads>(s_w[0], e ? A.wf1[1] : A.wf[1], tid);
    stage_lds<kFragH, kTThreads>(s_w[1], e ? A.wf1[2] : A.wf[2], tid);
    if (tid < kH) {
        s_b[0][tid] = (e ? A.b1[0] : A.b[0])[tid];
        s_b[1][tid] = (e ? A.b1[1] : A.b[1])[tid];
        s_b[2][tid] = (e ? A.b1[2] : A.b[2])[tid];
    }
    int64_t goff[kL];
#pragma unroll
    for (int l = 0; l < kL; ++l) goff[l] = e ? A.grid1[l] : A.grid[l];
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    const int64_t T = ceil_div(A.B, 32), T2 = ceil_div(T, 2);
    const int64_t V = (int64_t)A.g.nx * A.g.ny * A.g.nz;
    const bool few = T2 <= 2 * (int64_t)gridDim.x;
    for (int64_t tile = first_tile(T2, wave); tile < T2; tile += (int64_t)gridDim.x * kTW) {
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        int64_t pb[2], blk[2];
        bool st[2];
        rows64_blocks(tile, T, e, pb, blk, st);
        bf16x8 a[8][2], b[8][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t pair = pb[q] * 32 + jl;
            int64_t v = 0;
            float p[3] = {0.f, 0.f, 0.f};
            if (pair < A.B) {
                if (POS) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) p[c] = A.pos[(2 * pair + e) * 3 + c];
                } else {
                    v = A.pairs[2 * pair + e];
                    v = v < 0 ? 0 : (v >= V ? V - 1 : v);  // out-of-range pairs are clamped
                }
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                a[kb][q] = gather_h0<POS>(A, goff, kb, h, v, p, few);
                if (st[q]) A.h0[slab_chunk(blk[q], 2, kb, lane)] = as_u(a[kb][q]);
            }
        }
        rows64_layer<2, false>(s_w1, s_b[0] + h4, nullptr, A.h1, blk, st, a, b, lane);
        rows64_layer<8, false>(s_w[0], s_b[1] + h4, nullptr, A.h2, blk, st, b, a, lane);
        f32x16 acc[2];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {  // the latents, FP32
            mma_block<8, 2, true>(s_w[1], ob, s_b[2] + h4, a, acc, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 t;
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] = acc[q][4 * g + i];
                    if (st[q]) A.lat[(blk[q] * 4 + ob) * 256 + g * 64 + lane] = t;
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// The FP32 latents of pair block t, output block ob, of both endpoints.
__device__ __forceinline__ void load_latents(const FusedArgs &A, int64_t t, int64_t T, int ob,
                                             int lane, f32x16 (&lat)[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 v = A.lat[((q * T + t) * 4 + ob) * 256 + g * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) lat[q][4 * g + i] = v[i];
        }
}

// Decoder forward of 32 pairs per wave: the latent product, W4, W5, the head, and with
// targets the loss partial sums, gy and da5.
__global__ __launch_bounds__(kTThreads) void train_dec_fwd_kernel(FusedArgs A) {
    __shared__ bf16x8 s_w[2][kFragH];
    __shared__ __attribute__((aligned(16))) float s_b[2][kH];
    __shared__ __attribute__((aligned(16))) float s_w6[kH];
    __shared__ double s_part[kTW];
    const int tid = threadIdx.x;
    stage_lds<kFragH, kTThreads>(s_w[0], A.wf[3], tid);
    stage_lds<kFragH, kTThreads>(s_w[1], A.wf[4], tid);
    if (tid < kH) {
        s_b[0][tid] = A.b[3][tid];
        s_b[1][tid] = A.b[4][tid];
        s_w6[tid] = A.w6[tid];
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5;
    const int64_t T = ceil_div(A.B, 32);
    double loss_part = 0.0;
    for (int64_t tile = first_tile(T, wave); tile < T; tile += (int64_t)gridDim.x * kTW) {
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        bf16x8 a[8][2], b[8][2];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            f32x16 lat[2], mm;
            load_latents(A, tile, T, ob, lane, lat);
#pragma unroll
            for (int r = 0; r < 16; ++r) mm[r] = lat[0][r] * lat[1][r];
            u32x4 c0, c1;
            pack_block(mm, c0, c1);
            b[2 * ob][0] = operand<true>(c0);
            b[2 * ob + 1][0] = operand<true>(c1);
            A.m[slab_chunk(tile, 8, 2 * ob, lane)] = c0;
            A.m[slab_chunk(tile, 8, 2 * ob + 1, lane)] = c1;
        }
        loss_part += decode_pairs<true>(A, tile, s_w[0], s_w[1], s_b[0], s_b[1], s_w6, b, a, lane, h4);
    }
    store_loss_part(A, loss_part, s_part);
}

// Decoder adjoint of 32 pairs per wave: da5 -> da4 -> dlat of both endpoints.
__global__ __launch_bounds__(kTThreads) void train_dec_bwd_kernel(FusedArgs A) {
    __shared__ bf16x8 s_t[2][kFragH];  // W4^T, W5^T
    const int tid = threadIdx.x;
    stage_lds<kFragH, kTThreads>(s_t[0], A.wt[3], tid);
    stage_lds<kFragH, kTThreads>(s_t[1], A.wt[4], tid);
    if (blockIdx.x == 0 && tid < 64) loss_reduce(A.partial, A.n_partial, A.B, A.loss, A.status);
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t T = ceil_div(A.B, 32);
    for (int64_t tile = first_tile(T, wave); tile < T; tile += (int64_t)gridDim.x * kTW) {
        bf16x8 x[8][2], y[8][2];
        adj_layer5<true>(A, tile, s_t[1], x, y, lane);
        f32x16 acc[2];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            mma_block<8, 1>(s_t[0], ob, nullptr, y, acc, lane);
            f32x16 lat[2];
            load_latents(A, tile, T, ob, lane, lat);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                f32x16 d;
#pragma unroll
                for (int r = 0; r < 16; ++r) d[r] = acc[0][r] * lat[1 - q][r];
                u32x4 c0, c1;
                pack_block(d, c0, c1);
                A.dlat[slab_chunk(q * T + tile, 8, 2 * ob, lane)] = c0;
                A.dlat[slab_chunk(q * T + tile, 8, 2 * ob + 1, lane)] = c1;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Encoder adjoint: blockIdx.y = endpoint = encoder, 64 rows per wave: dlat -> da2 -> da1
// -> dL/dh0.
__global__ __launch_bounds__(kTThreads) void train_enc_bwd_kernel(FusedArgs A) {
    __shared__ bf16x8 s_t1[kFrag1];
    __shared__ bf16x8 s_t[2][kFragH];  // W2^T, W3^T
    const int tid = threadIdx.x, e = blockIdx.y;
    stage_lds<kFrag1, kTThreads>(s_t1, e ? A.wt1[0] : A.wt[0], tid);
    stage_lds<kFragH, kTThreads>(s_t[0], e ? A.wt1[1] : A.wt[1], tid);
    stage_lds<kFragH, kTThreads>(s_t[1], e ? A.wt1[2] : A.wt[2], tid);
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    const int64_t T = ceil_div(A.B, 32), T2 = ceil_div(T, 2);
    for (int64_t tile = first_tile(T2, wave); tile < T2; tile += (int64_t)gridDim.x * kTW) {
        int64_t pb[2], blk[2];
        bool st[2];
        rows64_blocks(tile, T, e, pb, blk, st);
        bf16x8 x[8][2], y[8][2];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int q = 0; q < 2; ++q) x[kb][q] = operand<true>(A.dlat[slab_chunk(blk[q], 8, kb, lane)]);
        rows64_layer<8, true>(s_t[1], nullptr, A.h2, A.da2, blk, st, x, y, lane);
        rows64_layer<8, true>(s_t[0], nullptr, A.h1, A.da1, blk, st, y, x, lane);
        f32x16 acc[2];
        mma_block<8, 2>(s_t1, 0, nullptr, x, acc, lane);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t pair = pb[q] * 32 + jl;
            if (st[q] && pair < A.B) store_dh0(A, e * A.B + pair, acc[q], h);
        }
    }
}

// Weight and bias gradients of every layer in one launch: workgroup ranges
// [wg0[L], wg0[L + 1]) take layer L (the packed matrices, then the head w6, b6), each
// workgroup a strided share of its layer's 64-row slab pairs.  A slab pair of
// G (the layer's output gradient) and X (its input) is loaded with 16-byte
// reads (4 rows x 8 features per thread), transposed in registers and written
// to LDS feature-major, s[f][row]; the waves then accumulate
// dW[o][k] += sum_rows G[row][o] X[row][k] on MFMA (K = rows) and threads
// f < 128 sum the bf16 G column f for the bias.  One atomic flush per workgroup
// at the end.
struct WgradArgs {
    int n_mat;  // matrices; layer n_mat is the head
    const u32x4 *g[kMaxMats], *x[kMaxMats];
    int kin[kMaxMats];  // inputs (W1: 32, or 112 with Fourier features)
    int64_t nslab[kMaxMats + 1];
    float *dW[kMaxMats + 1], *db[kMaxMats + 1];
    const u32x4 *d2;
    const float *gy;
    int wg0[kMaxMats + 2];
};

constexpr int kWgLD = 64 + 8;  // bf16 per LDS feature row (64 rows + pad)

// rows r = 0..3 of 8 features each (c[r]) -> features e = 0..7 of 4 rows each
__device__ __forceinline__ void transpose4(const u32x4 (&c)[4], uint2 (&t)[8]) {
#pragma unroll
    for (int p = 0; p < 4; ++p)      // word p = features 2 p, 2 p + 1
#pragma unroll
        for (int i = 0; i < 2; ++i) {  // rows 2 i, 2 i + 1
            const uint32_t a = c[2 * i][p], b = c[2 * i + 1][p];
            const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x05040100u);
            const uint32_t hi = __builtin_amdgcn_perm(b, a, 0x07060302u);
            if (i == 0) {
                t[2 * p].x = lo;
                t[2 * p + 1].x = hi;
            } else {
                t[2 * p].y = lo;
                t[2 * p + 1].y = hi;
            }
        }
}

// The 4 x 8 block (slab blk, k-block kb, half h, rows r0 .. r0 + 3) of a slab
// with nkb k-blocks: 4 coalesced 16-byte loads (zeros past the last slab) ...
__device__ __forceinline__ void load4(const u32x4 *__restrict__ src, int64_t blk, int64_t nslab,
                                      int nkb, int kb, int h, int r0, u32x4 (&c)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
        c[r] = blk < nslab ? src[slab_chunk(blk, nkb, kb, 32 * h + r0 + r)]
                           : u32x4{0u, 0u, 0u, 0u};
}
// ... written feature-major into s (the slab's rows at 32 sl).
__device__ __forceinline__ void write4(const u32x4 (&c)[4], int kb, int h, int r0, int sl,
                                       bool nat, __bf16 *__restrict__ s) {
    uint2 t[8];
    transpose4(c, t);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int f = nat ? feat_nat(kb, h, e) : feat_perm(kb, h, e);
        *reinterpret_cast<uint2 *>(s + f * kWgLD + 32 * sl + r0) = t[e];
    }
}

// Eight waves: wave w accumulates output rows 32 (w % 4) .. + 31 against input
// columns 64 (w / 4) .. + 63 (two 32-column blocks).  Threads t < 256 stage G
// (the head: t < 64 stage gy), t >= 256 stage X, four rows of one 8-feature
// block each; the next slab pair's loads are in flight while the MFMAs run.
__global__ __launch_bounds__(512, 4) void wgrad_all_kernel(WgradArgs A) {
    __shared__ __attribute__((aligned(16))) __bf16 s_g[kH * kWgLD];
    __shared__ __attribute__((aligned(16))) __bf16 s_x[kH * kWgLD];
    __shared__ float s_gy[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    int L = 0;
    while (L < A.n_mat && (int)blockIdx.x >= A.wg0[L + 1]) ++L;
    const bool head = L == A.n_mat;
    const int part = (int)blockIdx.x - A.wg0[L], nparts = A.wg0[L + 1] - A.wg0[L];
    const int64_t nslab = A.nslab[L];
    if (2 * (int64_t)part >= nslab) return;
    const int kin = head ? kH : A.kin[L];
    const int xkb = kin / 16, xcb = (kin + 31) / 32;
    const int ob = wave & 3, cb0 = 2 * (wave >> 2);
    // this thread's block
    const int u = tid & 255, sl = u >> 7, kb = (u >> 4) & 7, hh = (u >> 3) & 1,
              r0 = 4 * (u & 7);
    const bool is_g = tid < 256;
    const bool active = head ? (is_g ? tid < 64 : true) : (is_g || kb < xkb);
    const u32x4 *src = head ? A.d2 : (is_g ? A.g[L] : A.x[L]);
    const int nkb = is_g ? 8 : xkb;
    const bool nat = !is_g && kin != kH;  // a W1: h0 in natural order
    u32x4 c[4];
    float gyv = 0.f;
    auto fetch = [&](int64_t sp) {
        if (!active) return;
        if (head && is_g) {
            const int64_t r = 2 * sp * 32 + tid;
            gyv = r < nslab * 32 ? A.gy[r] : 0.f;
        } else {
            load4(src, 2 * sp + sl, nslab, nkb, kb, hh, r0, c);
        }
    };
    f32x16 acc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
    float bsum = 0.f;
    fetch(part);
    for (int64_t sp = part; 2 * sp < nslab; sp += nparts) {
        if (active) {
            if (head && is_g)
                s_gy[tid] = gyv;
            else
                write4(c, kb, hh, r0, sl, nat, is_g && !head ? s_g : s_x);
        }
        __syncthreads();
        if (2 * (sp + nparts) < nslab) fetch(sp + nparts);
        if (head) {
            // dw6[k] = sum_rows gy d2[row][k] (thread k), db6 = sum_rows gy (thread kH + row:
            // equal addends round alike, so one thread over all rows was 1e-5 off)
            if (tid < kH) {
                const __bf16 *xr = s_x + tid * kWgLD;
#pragma unroll 8
                for (int r = 0; r < 64; ++r) bsum = fmaf(s_gy[r], (float)xr[r], bsum);
            } else if (wave == 2) {
                bsum += s_gy[lane];
            }
        } else {
            if (cb0 < xcb) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(
                        s_g + (32 * ob + jl) * kWgLD + 16 * kk + 8 * h);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        if (cb0 + q >= xcb) continue;
                        const bf16x8 b = *reinterpret_cast<const bf16x8 *>(
                            s_x + (32 * (cb0 + q) + jl) * kWgLD + 16 * kk + 8 * h);
                        acc[q] = mfma32(a, b, acc[q]);
                    }
                }
            }
            if (tid < kH) {
                const u32x4 *gr = reinterpret_cast<const u32x4 *>(s_g + tid * kWgLD);
#pragma unroll
                for (int cc = 0; cc < 8; ++cc) {
                    const u32x4 v = gr[cc];
#pragma unroll
                    for (int i = 0; i < 4; ++i) bsum += bf_lo(v[i]) + bf_hi(v[i]);
                }
            }
        }
        __syncthreads();
    }
    if (head) {
        if (tid < kH) unsafeAtomicAdd(A.dW[L] + tid, bsum);
        if (wave == 2) {
#pragma unroll
            for (int d = 32; d; d >>= 1) bsum += __shfl_xor(bsum, d);
            if (lane == 0) unsafeAtomicAdd(A.db[L], bsum);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        // columns past the input width (W1 with 112 inputs: 112..127) hold
        // nothing and are not written
        if (cb0 + q >= xcb || 32 * (cb0 + q) + jl >= kin) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            unsafeAtomicAdd(A.dW[L] + (32 * ob + d_row(r, lane)) * kin + 32 * (cb0 + q) + jl,
                            acc[q][r]);
    }
    if (tid < kH) unsafeAtomicAdd(A.db[L] + tid, bsum);
}

// ------------------------------------------------------- fused host ----
static bool fused_path(const ndf_net_config *c) { return !c->grid_only; }

static int n_mats(const ndf_net_config *c) { return 3 * c->n_enc + 2; }

struct FusedWS {
    int32_t *status;
    TrainFrags fr;
    u32x4 *h0, *h1, *h2, *m, *d1, *d2, *da5, *da4, *dlat, *da2, *da1;
    f32x4 *lat;
    float *gy, *dh0;
    double *partial;
    size_t bytes;
};

constexpr int kFusedBlocksMax = 512;

static FusedWS carve_fused(const ndf_net_config *c, void *ws, int64_t B) {
    FusedWS t{};
    const int64_t T = ceil_div(B, 32);
    char *base = (char *)ws;
    size_t pos = 0;
    auto take = [&](size_t n) {
        char *p = base ? base + pos : nullptr;
        pos += align_up(n, 256);
        return p;
    };
    t.status = (int32_t *)take(kStatusBytes);
    const int kb1 = enc_in(c) / 16;
    auto first = [&](int L) { return L < 3 * c->n_enc && L % 3 == 0; };  // a W1
    for (int L = 0; L < n_mats(c); ++L)
        t.fr.f[L] = (bf16x8 *)take((first(L) ? 4 * kb1 * 64 : kFragH) * 16);
    for (int L = 0; L < n_mats(c); ++L)
        t.fr.t[L] = (bf16x8 *)take((first(L) ? kFrag1 : kFragH) * 16);
    const size_t slab = 8 * 64 * 16;  // 128 features x 32 rows, bf16
    t.h0 = (u32x4 *)take(2 * T * kb1 * 64 * 16);
    t.h1 = (u32x4 *)take(2 * T * slab);
    t.h2 = (u32x4 *)take(2 * T * slab);
    t.lat = (f32x4 *)take(2 * T * 2 * slab);
    t.m = (u32x4 *)take(T * slab);
    t.d1 = (u32x4 *)take(T * slab);
    t.d2 = (u32x4 *)take(T * slab);
    t.da5 = (u32x4 *)take(T * slab);
    t.da4 = (u32x4 *)take(T * slab);
    t.dlat = (u32x4 *)take(2 * T * slab);
    t.da2 = (u32x4 *)take(2 * T * slab);
    t.da1 = (u32x4 *)take(2 * T * slab);
    t.gy = (float *)take(T * 32 * 4);
    t.dh0 = (float *)take(2 * B * kK0 * 4);
    t.partial = (double *)take(kFusedBlocksMax * 8);
    t.bytes = pos;
    return t;
}

// One workgroup per 32-pair tile up to one per CU (a workgroup's 140 KB of weights fill a
// CU's LDS), then a tile for each of its waves, and two rounds of workgroups once one
// round's waves would have more than one.
static unsigned fused_blocks(int64_t B) {
    const int64_t T = ceil_div(B, 32);
    return (unsigned)(T < 256 ? T : T <= 256 * kTW ? 256 : kFusedBlocksMax);
}

// Bytes the sorted scatter needs beside the gradient: rows, work list, counts.
static size_t tile_scratch(int64_t rows, int64_t tiles, int rows_wg, size_t *list, size_t *hist) {
    *list = align_up((size_t)rows * sizeof(SortedRow), 256);
    *hist = *list + align_up((size_t)(tiles + rows / rows_wg + 1) * sizeof(int4), 256);
    return *hist + (size_t)tiles * kSortWgs * sizeof(int);
}

// How the grid gradient of `rows` rows is added up: true and a plan for the sorted scatter
// where it is the faster one by this model (us; measured on grids of 16 x 14 x 5 to
// 400 x 400 x 11).  Directly, a level takes 0.25 ns per row (0.45 in tables far beyond the
// L2s; 0.15 at vertices of a level of the data grid's size, where a row has one corner)
// and, since adds to one cell follow each other, 150 ns per row and cell.  Sorted: the
// sort 12 us and 0.023 ns per row, a boxed row 0.106 us in a workgroup's chain (512
// workgroups run at once) and 1/32 ns per cell of every workgroup's boxes, beside which
// the levels without boxes are added to.  Tiles of three depths and nearly square
// footprints (of up to 400 vertices; a longer axis is cut) are tried for the one to three
// coarsest dense levels, as far as the lists stay within `scratch` bytes and, in order of
// growing edges, up to the first whose boxes exceed kTileLds.  The one smaller footprint
// that may follow it is left out on purpose: on the 7 of 3000 random grids tried where the
// model prefers it, its boxes nearly fill kTileLds and the step measured 2 to 11 % slower
// (43 x 26 x 40 vertices, tables of 2^16, 195651 pairs: 634 -> 691 us; 544 x 260 x 11 at
// 44623 pairs of positions: 246 -> 273).  The model spreads the rows evenly over the
// tiles.  Rows crowded on a few cells are mostly still faster sorted (40000 pairs of one
// vertex of 250 x 352 x 20: 1171 us directly, 392 sorted); slower were 40000 pairs of
// positions in a twentieth of 37 x 29 x 11 (1190 directly, 1348 sorted) and 4000 pairs of
// one vertex there (201 and 214).
static bool tile_plan(const ndf_net_config *c, const GridGeom &g, int64_t rows, bool vertices,
                      size_t scratch, TilePlan &best) {
    if (rows < kMinSorted || rows >= (1ll << 31)) return false;
    const int n[3] = {c->nx, c->ny, c->nz};
    const double nr = (double)rows;
    double direct[kL], cost = 0.0;
    for (int l = 0; l < kL; ++l) {
        const int *R = g.R[l];
        const bool one = vertices && R[0] == n[0] && R[1] == n[1] && R[2] == n[2];
        const double cells = g.hmask[l] ? g.hmask[l] + 1.0 : (double)R[0] * R[1] * R[2];
        direct[l] = nr * (one ? 0.15e-3 + 0.02 / cells
                              : (cells > 1 << 19 ? 0.45e-3 : 0.25e-3) + 0.15 / cells);
        cost += direct[l];
    }
    const int64_t even = ceil_div(rows, 512);  // rows of a workgroup if all tiles were one
    const int rows_wg = (int)(even < 128 ? 128 : even > 1024 ? 1024 : align_up((size_t)even, 64));
    bool found = false;
    constexpr int kSizes[] = {4, 6, 8, 10, 12, 14, 16, 20, 24, 32, 48, 64, 96, 400};
    constexpr int kN = sizeof(kSizes) / sizeof(kSizes[0]);
    const int depth[3] = {n[2], n[2] < 32 ? n[2] : 32, n[2] < 16 ? n[2] : 16};
    for (int boxed = 1; boxed < kL && !g.hmask[boxed - 1]; ++boxed) {  // levels 0 .. boxed - 1
        double left = 0.0;
        for (int l = boxed; l < kL; ++l) left += direct[l];
        for (int zi = 0; zi < 3; ++zi) {
            if (zi && depth[zi] == depth[zi - 1]) continue;
            for (int k = 0; k < 2 * kN; ++k) {
                const int tx = kSizes[k / 2], ty = k & 1 ? (k > 1 ? kSizes[k / 2 - 1] : tx) : tx;
                TilePlan p{};
                const int t[3] = {tx < n[0] ? tx : n[0], ty < n[1] ? ty : n[1], depth[zi]};
                int64_t tiles = c->n_enc;
                for (int a = 0; a < 3; ++a) {
                    p.t[a] = t[a];
                    p.nt[a] = (int)ceil_div(n[a], t[a]);
                    p.m[a] = (uint32_t)(((1ull << 32) + t[a] - 1) / t[a]);
                    tiles *= p.nt[a];
                }
                int64_t cells = 0;
                for (int l = 0; l < boxed; ++l) {
                    p.off[l] = (int)cells;
                    int64_t nl = 1;
                    for (int a = 0; a < 3; ++a) {
                        // base cells of a tile's span, and the last one's neighbour
                        const int64_t span =
                            (int64_t)(t[a] - (vertices ? 1 : 0)) * (g.R[l][a] - 1) / (n[a] - 1) + 3;
                        p.box[l][a] = (int)(span < g.R[l][a] ? span : g.R[l][a]);
                        nl *= p.box[l][a];
                    }
                    cells += nl;
                }
                if (cells * kF * 4 > (int64_t)kTileLds) break;
                size_t list, hist;
                if (tiles > kMaxTiles || tile_scratch(rows, tiles, rows_wg, &list, &hist) > scratch)
                    continue;
                p.n_tiles = (int)(tiles / c->n_enc);
                p.cells = (int)cells;
                p.rows = rows_wg;
                p.boxed = boxed;
                const double per = nr / (double)tiles;
                const double wgs = (double)tiles * (double)ceil_div((int64_t)per + 1, rows_wg);
                const double chain = per < rows_wg ? per : rows_wg;
                const double box = 0.106 * chain * (wgs > 512.0 ? wgs / 512.0 + 0.5 : 1.0) +
                                   (double)cells * wgs / 32e3;
                const double us = 12.0 + 0.023e-3 * nr + (box > left ? box : left);
                if (us < cost) {
                    cost = us;
                    best = p;
                    found = true;
                }
            }
        }
    }
    return found;
}

// The grid gradient from dL/dh0; scratch: the FP32 latents' region, free by then.
static void scatter_grid(const ndf_net_config *c, const NetOffsets &o, const int64_t *pairs,
                         const float *pos, int64_t B, float *G, const float *dh0, void *scratch,
                         size_t scratch_bytes, hipStream_t st) {
    const GridGeom g = grid_geom(c);
    const GridOffs go = grid_offs(o);
    const int64_t rows = 2 * B;
    TilePlan tp;
    if (!tile_plan(c, g, rows, pos == nullptr, scratch_bytes, tp)) {
        scatter_direct(G, go, g, c->n_enc, pairs, pos, B, dh0, st);
        return;
    }
    const int tiles = c->n_enc * tp.n_tiles;
    const int64_t items = tiles + rows / tp.rows;  // at most
    size_t list_at, hist_at;
    tile_scratch(rows, tiles, tp.rows, &list_at, &hist_at);
    SortedRow *sorted = (SortedRow *)scratch;
    int4 *list = (int4 *)((char *)scratch + list_at);
    int *hist = (int *)((char *)scratch + hist_at);
    hipLaunchKernelGGL(grid_sort_count_kernel, dim3(kSortWgs), dim3(kSortThreads), 0, st, g, tp,
                       c->n_enc, pairs, pos, B, hist);
    hipLaunchKernelGGL(grid_sort_place_kernel, dim3(kSortWgs), dim3(kSortThreads), 0, st, g, tp,
                       c->n_enc, pairs, pos, B, hist, sorted, list);
    const size_t lds = tp.boxed * sizeof(TileStage) + (size_t)tp.cells * kF * sizeof(float);
    if (pos)
        hipLaunchKernelGGL(grid_tile_kernel<true>, dim3((unsigned)items), dim3(64 * kL), lds,
                           st, G, go, g, tp, sorted, list, dh0);
    else
        hipLaunchKernelGGL(grid_tile_kernel<false>, dim3((unsigned)items), dim3(64 * kL), lds,
                           st, G, go, g, tp, sorted, list, dh0);
}

// Workgroups per encoder of the encoder kernels (64 rows per wave): as fused_blocks, the
// two encoders sharing the CUs.
static unsigned enc_blocks(int64_t B) {
    const int64_t T2 = ceil_div(ceil_div(B, 32), 2);
    return (unsigned)(T2 < 128 ? T2 : T2 <= 128 * kTW ? 128 : 256);
}

static FusedArgs fused_args(const ndf_net_config *c, const NetOffsets &o, const float *P,
                            const int64_t *pairs, const float *pos, const float *targets,
                            int64_t B, const FusedWS &t, float *y) {
    FusedArgs a{};
    a.P = P;
    for (int l = 0; l < kL; ++l) a.grid[l] = o.grid[0][l];
    for (int L = 0; L < 5; ++L) {
        const int i = L < 3 ? L : 3 * (c->n_enc - 1) + L;
        a.wf[L] = t.fr.f[i];
        a.wt[L] = t.fr.t[i];
    }
    if (c->n_enc == 2) {
        for (int l = 0; l < kL; ++l) a.grid1[l] = o.grid[1][l];
        for (int L = 0; L < 3; ++L) {
            a.wf1[L] = t.fr.f[3 + L];
            a.wt1[L] = t.fr.t[3 + L];
        }
        a.b1[0] = P + o.b1[1];
        a.b1[1] = P + o.b2[1];
        a.b1[2] = P + o.b3[1];
    }
    a.b[0] = P + o.b1[0];
    a.b[1] = P + o.b2[0];
    a.b[2] = P + o.b3[0];
    a.b[3] = P + o.b4;
    a.b[4] = P + o.b5;
    a.w6 = P + o.w6;
    a.b6 = P + o.b6;
    a.g = grid_geom(c);
    a.pairs = pairs;
    a.pos = pos;
    a.targets = targets;
    a.B = B;
    a.h0 = t.h0; a.h1 = t.h1; a.h2 = t.h2; a.m = t.m; a.d1 = t.d1; a.d2 = t.d2;
    a.da5 = t.da5; a.da4 = t.da4; a.dlat = t.dlat; a.da2 = t.da2; a.da1 = t.da1;
    a.lat = t.lat;
    a.gy = t.gy;
    a.y = y;
    a.dh0 = t.dh0;
    a.partial = t.partial;
    return a;
}

// G, status: the gradient and the status word to clear first (null: neither).
static void fused_forward(const ndf_net_config *c, const NetOffsets &o, const FusedArgs &a,
                          const FusedWS &t, float *G, int32_t *status, hipStream_t st) {
    const float *P = a.P, *pos = a.pos;
    const int64_t B = a.B;
    const unsigned zero = G ? gs_blocks(o.total / 4) : 0;
    PackArgs pk{};
    pk.n_enc = c->n_enc;
    pk.kin1 = enc_in(c);
    pk.F = t.fr;
    for (int e = 0; e < c->n_enc; ++e) {
        pk.w[3 * e] = o.W1[e];
        pk.w[3 * e + 1] = o.W2[e];
        pk.w[3 * e + 2] = o.W3[e];
    }
    pk.w[3 * c->n_enc] = o.W4;
    pk.w[3 * c->n_enc + 1] = o.W5;
    hipLaunchKernelGGL(pack_train_kernel, dim3(kPackBlocks * n_mats(c) + zero), dim3(256), 0, st, P,
                       pk, G, o.total, status);
    if (c->n_enc == 2) {
        const dim3 ge(enc_blocks(B), 2);
        if (pos)
            hipLaunchKernelGGL(train_enc_fwd_kernel<true>, ge, dim3(kTThreads), 0, st, a);
        else
            hipLaunchKernelGGL(train_enc_fwd_kernel<false>, ge, dim3(kTThreads), 0, st, a);
        hipLaunchKernelGGL(train_dec_fwd_kernel, dim3(fused_blocks(B)), dim3(kTThreads), 0, st, a);
        return;
    }
    const dim3 g(fused_blocks(B)), b(kTThreads);
    if (c->fourier) {
        if (pos)
            hipLaunchKernelGGL((train_fwd_kernel<true, true>), g, b, 0, st, a);
        else
            hipLaunchKernelGGL((train_fwd_kernel<false, true>), g, b, 0, st, a);
    } else {
        if (pos)
            hipLaunchKernelGGL((train_fwd_kernel<true, false>), g, b, 0, st, a);
        else
            hipLaunchKernelGGL((train_fwd_kernel<false, false>), g, b, 0, st, a);
    }
}

static int fused_grad(const ndf_net_config *c, const float *P, const int64_t *pairs,
                      const float *pos, const float *targets, int64_t B, float *G, float *loss,
                      void *ws, hipStream_t st) {
    const NetOffsets o = net_offsets(c);
    const FusedWS t = carve_fused(c, ws, B);
    FusedArgs a = fused_args(c, o, P, pairs, pos, targets, B, t, nullptr);
    a.n_partial = (int)fused_blocks(B);
    a.loss = loss;
    a.status = t.status;
    fused_forward(c, o, a, t, G, t.status, st);
    const int n_enc = c->n_enc;
    if (n_enc == 2) {
        hipLaunchKernelGGL(train_dec_bwd_kernel, dim3(fused_blocks(B)), dim3(kTThreads), 0, st, a);
        hipLaunchKernelGGL(train_enc_bwd_kernel, dim3(enc_blocks(B), 2), dim3(kTThreads), 0, st, a);
    } else {
        hipLaunchKernelGGL(train_bwd_kernel, dim3(fused_blocks(B)), dim3(kTThreads), 0, st, a);
    }
    scatter_grid(c, o, pairs, pos, B, G, t.dh0, t.lat, (size_t)((char *)t.m - (char *)t.lat), st);
    WgradArgs w{};
    const int64_t T = ceil_div(B, 32);
    const int64_t te = n_enc == 2 ? T : 2 * T;  // slabs per encoder
    int acc_wg = 0, L = 0;
    // workgroups per layer in proportion to the bytes it reads (per decoder slab:
    // W1 20 KB, W2 and W3 32, W4 and W5 16, the head 8), 511 in all, one round at
    // two workgroups per CU; at most one per slab pair
    auto layer = [&](int share, const u32x4 *g, const u32x4 *x, int kin, int64_t nslab, float *dW,
                     float *db) {
        if (g) {
            w.g[L] = g;
            w.x[L] = x;
            w.kin[L] = kin;
        }
        w.nslab[L] = nslab;
        w.dW[L] = dW;
        w.db[L] = db;
        w.wg0[L] = acc_wg;
        const int64_t pairs_l = ceil_div(nslab, 2);
        acc_wg += (int)(pairs_l < share ? pairs_l : share);
        ++L;
    };
    const int64_t s8 = te * 8 * 64, s1 = te * (enc_in(c) / 16) * 64;  // chunks per encoder
    for (int e = 0; e < n_enc; ++e) {
        layer(82 / n_enc, t.da1 + e * s8, t.h0 + e * s1, enc_in(c), te, G + o.W1[e], G + o.b1[e]);
        layer(132 / n_enc, t.da2 + e * s8, t.h1 + e * s8, kH, te, G + o.W2[e], G + o.b2[e]);
        layer(132 / n_enc, t.dlat + e * s8, t.h2 + e * s8, kH, te, G + o.W3[e], G + o.b3[e]);
    }
    layer(66, t.da4, t.m, kH, T, G + o.W4, G + o.b4);
    layer(66, t.da5, t.d1, kH, T, G + o.W5, G + o.b5);
    layer(33, nullptr, nullptr, kH, T, G + o.w6, G + o.b6);
    w.n_mat = L - 1;
    w.wg0[L] = acc_wg;
    w.d2 = t.d2;
    w.gy = t.gy;
    hipLaunchKernelGGL(wgrad_all_kernel, dim3((unsigned)acc_wg), dim3(512), 0, st, w);
    return status_of_launch();
}

}  // namespace

size_t net_train_ws_bytes(const ndf_net_config *c, int64_t B) {
    return fused_path(c) ? carve_fused(c, nullptr, B).bytes : carve(nullptr, B).bytes;
}

size_t net_train_plan_bytes(const ndf_net_config *c, int64_t B, size_t avail) {
    const size_t asked = net_train_ws_bytes(c, B);
    if (avail >= asked) return asked;
    const size_t rows = carve(nullptr, B).bytes;
    return c->n_enc == 2 && avail >= rows ? rows : 0;
}

// Whether a call with net_train_plan_bytes = plan runs the fused step.
static bool runs_fused(const ndf_net_config *c, int64_t B, size_t plan) {
    return fused_path(c) && plan >= net_train_ws_bytes(c, B);
}

int launch_net_init(const ndf_net_config *c, float *params, float *opt, uint64_t seed,
                    hipStream_t st) {
    const NetOffsets o = net_offsets(c);
    hipLaunchKernelGGL(fill_kernel, dim3(gs_blocks(o.total)), dim3(kThreads), 0, st, params,
                       o.total, 0.f);
    if (opt)
        hipLaunchKernelGGL(fill_kernel, dim3(gs_blocks(2 * o.total)), dim3(kThreads), 0, st, opt,
                           2 * o.total, 0.f);
    auto uni = [&](int64_t off, int64_t n, float a) {
        hipLaunchKernelGGL(uniform_kernel, dim3(gs_blocks(n)), dim3(kThreads), 0, st, params + off,
                           n, a, seed, off);
    };
    for (int e = 0; e < c->n_enc; ++e) {
        for (int l = 0; l < kL; ++l) uni(o.grid[e][l], o.cells[l] * kF, 1e-4f);
        if (c->grid_only) continue;
        uni(o.W1[e], kH * enc_in(c), sqrtf(6.f / (float)enc_in(c)));
        uni(o.W2[e], kH * kH, sqrtf(6.f / kH));
        uni(o.W3[e], kH * kH, sqrtf(6.f / kH));
    }
    const int k4 = c->grid_only ? kK0 : kH;  // inputs of the first decoder layer
    uni(o.W4, kH * k4, sqrtf(6.f / k4));
    uni(o.W5, kH * kH, sqrtf(6.f / kH));
    uni(o.w6, kH, sqrtf(6.f / kH));
    return status_of_launch();
}

int launch_net_forward(const ndf_net_config *c, const float *params, const int64_t *pairs,
                       const float *pos, int64_t B, float *y, void *ws, size_t plan,
                       hipStream_t st) {
    const NetOffsets o = net_offsets(c);
    if (runs_fused(c, B, plan)) {
        const FusedWS t = carve_fused(c, ws, B);
        fused_forward(c, o, fused_args(c, o, params, pairs, pos, nullptr, B, t, y), t, nullptr,
                      nullptr, st);
        return status_of_launch();
    }
    TrainWS t = carve(ws, B);
    t.y = y;
    forward(c, o, params, pairs, pos, nullptr, B, t, st);
    return status_of_launch();
}

int launch_net_grad(const ndf_net_config *c, const float *P, const int64_t *pairs,
                    const float *pos, const float *targets, int64_t B, float *G, float *loss,
                    void *ws, size_t plan, hipStream_t st) {
    if (runs_fused(c, B, plan)) return fused_grad(c, P, pairs, pos, targets, B, G, loss, ws, st);
    const NetOffsets o = net_offsets(c);
    const TrainWS t = carve(ws, B);
    launch_status_clear(t.status, st);
    hipLaunchKernelGGL(fill_kernel, dim3(gs_blocks(o.total)), dim3(kThreads), 0, st, G, o.total,
                       0.f);
    forward(c, o, P, pairs, pos, targets, B, t, st);
    const int nparts = (int)ceil_div(B, kThreads);
    hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(64), 0, st, t.partial, nparts, B, loss,
                       t.status);
    // decoder adjoint
    {
        int64_t hb = ceil_div(B, 2);
        hipLaunchKernelGGL(head_bwd_kernel, dim3((unsigned)(hb < 1024 ? hb : 1024)), dim3(kThreads),
                           0, st, t.D2, t.gy, P + o.w6, B, t.dA, G + o.w6, G + o.b6);
    }
    rows_wgrad<kH>(t.dA, t.D1, B, G + o.W5, G + o.b5, st);
    rows_layer<kH, kH, EPI_MASK>(t.dA, B, P + o.W5, 1, kH, nullptr, t.D1, t.dB, st);
    const GridGeom g = grid_geom(c);
    const GridOffs go = grid_offs(o);
    if (c->grid_only) {
        // W4 [128][32] on the merged grid features; the product rule gives the
        // grid features' gradient directly
        rows_wgrad<kK0>(t.dB, t.M, B, G + o.W4, G + o.b4, st);
        rows_layer<kH, kK0, EPI_PLAIN>(t.dB, B, P + o.W4, 1, kK0, nullptr, nullptr, t.dA, st);
        hipLaunchKernelGGL(merge_bwd_kernel, dim3(gs_blocks(B * kK0 / 4)), dim3(kThreads), 0, st,
                           t.dA, t.H0, B, t.dH0, kK0);
    } else {
        rows_wgrad<kH>(t.dB, t.M, B, G + o.W4, G + o.b4, st);
        rows_layer<kH, kH, EPI_PLAIN>(t.dB, B, P + o.W4, 1, kH, nullptr, nullptr, t.dA, st);
        // product rule across the merge: dE[b] = dM[b] * E[B+b], dE[B+b] = dM[b] * E[b]
        hipLaunchKernelGGL(merge_bwd_kernel, dim3(gs_blocks(B * kH / 4)), dim3(kThreads), 0, st,
                           t.dA, t.E, B, t.dB, kH);
        for (int e = 0; e < 2; ++e) {  // encoder adjoints
            const int64_t r0 = e * B;
            float *dE = t.dB + r0 * kH, *dP2 = t.dA + r0 * kH, *dP1 = t.dB + r0 * kH;
            rows_wgrad<kH>(dE, t.H2 + r0 * kH, B, G + o.W3[e], G + o.b3[e], st);
            rows_layer<kH, kH, EPI_MASK>(dE, B, P + o.W3[e], 1, kH, nullptr, t.H2 + r0 * kH, dP2, st);
            rows_wgrad<kH>(dP2, t.H1 + r0 * kH, B, G + o.W2[e], G + o.b2[e], st);
            rows_layer<kH, kH, EPI_MASK>(dP2, B, P + o.W2[e], 1, kH, nullptr, t.H1 + r0 * kH, dP1, st);
            rows_wgrad<kK0>(dP1, t.H0 + r0 * kK0, B, G + o.W1[e], G + o.b1[e], st);
            rows_layer<kH, kK0, EPI_PLAIN>(dP1, B, P + o.W1[e], 1, kK0, nullptr, nullptr,
                                           t.dH0 + r0 * kK0, st);
        }
    }
    scatter_direct(G, go, g, c->n_enc, pairs, pos, B, t.dH0, st);
    return status_of_launch();
}

int launch_adam(const ndf_net_config *c, float *params, float *opt, const float *grad,
                int64_t step, float lr, const int32_t *status, hipStream_t st) {
    const NetOffsets o = net_offsets(c);
    const double c1 = 1.0 / (1.0 - pow(0.9, (double)step));
    const double c2 = 1.0 / (1.0 - pow(0.999, (double)step));
    hipLaunchKernelGGL(adam_kernel, dim3(gs_blocks(o.total)), dim3(kThreads), 0, st, params, opt,
                       opt + o.total, grad, o.total, lr, (float)c1, (float)c2, status);
    return status_of_launch();
}

// Phi_{nu mu} from Phi_{mu nu} (Sec. 6.4): the two encoder blocks [grid0..b3_0]
// and [grid1..b3_1] have the same layout and length, so out is in with the two
// ranges exchanged and the decoder copied.
__global__ void swap_encoders_kernel(const float *__restrict__ in, float *__restrict__ out,
                                     int64_t e0, int64_t e1, int64_t total) {
    const int64_t len = e1 - e0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kThreads) {
        int64_t src = i;
        if (i >= e0 && i < e1)
            src = i + len;
        else if (i >= e1 && i < e1 + len)
            src = i - len;
        out[i] = in[src];
    }
}

int launch_net_swap_encoders(const ndf_net_config *c, const float *in, float *out,
                             hipStream_t st) {
    const NetOffsets o = net_offsets(c);
    // encoder 1 starts where encoder 0 ends; both end before W4
    const int64_t e0 = o.grid[0][0], e1 = o.grid[1][0];
    hipLaunchKernelGGL(swap_encoders_kernel, dim3(gs_blocks(o.total)), dim3(kThreads), 0, st, in,
                       out, e0, e1, o.total);
    return status_of_launch();
}

}  // namespace ndf
