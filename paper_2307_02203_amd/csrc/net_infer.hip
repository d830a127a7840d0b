// Learned dependence field inference (Sec. 5): phi(p) = Phi(p_ref, p) at every
// grid vertex, in one fused kernel per reference.
//
// The reference latent is computed once (same kernel, latent-only mode).  Each
// wave then takes 64 query vertices at a time through
//   grid gather (4 levels x 8 corners of 8 bf16 features, FP32 trilinear weights)
//   -> L1 32->128 ReLU -> L2 128->128 ReLU -> L3 128->128 (latent)
//   -> product with the reference latent -> L4 ReLU -> L5 ReLU -> w6 . d2 + b6
// entirely in registers: every layer is MFMA 32x32x16 bf16 with FP32 accumulate,
// the weights of all layers (136 KB bf16) sit in LDS for the whole launch in
// MFMA operand order, and a layer's FP32 accumulators are rounded to bf16 and
// used directly as the next layer's B operand.  That works because the MFMA
// output layout (lane = query, 16 feature rows per lane) equals the operand
// layout up to a fixed permutation of the contraction index inside every
// 16-block, which is folded into the packed weights:
//   logical k = 16 kb + 8 h + e  <->  feature 16 kb + 8 (e / 4) + 4 h + e % 4.
// Latents are rounded to bf16 before the product, and the product of two bf16
// numbers is exact in FP32, so Phi(p, q) and Phi(q, p) of a self field are
// computed identically.
#include <type_traits>

#include "net.hpp"

namespace ndf {

constexpr int kInferWaves = 8;
constexpr int kInferThreads = 64 * kInferWaves;

// Byte offsets inside the packed inference parameters.
struct QLayout {
    int64_t grid[2][kL];           // bf16 [cells][8]
    int64_t w1[2], w2[2], w3[2];   // bf16 MFMA A fragments
    int64_t w4, w5;
    int64_t b1[2], b2[2], b3[2];   // fp32 [128]
    int64_t b4, b5, w6, b6;        // fp32
    // FP8 (OCP E4M3) copies of W2..W5 in 32x32x64 operand order + per-row scales
    int64_t q2[2], q3[2], q4, q5;  // fp8 fragments, 16 KB each
    int64_t s2[2], s3[2], s4, s5;  // int32 [128][4] E8M0 scale bytes per row and 32-k block
    int64_t amax;                  // int32 [4]: calibrated max |input| of layers 2..5
    int64_t total;
};

static QLayout qlayout(const ndf_net_config *c) {
    QLayout q{};
    int64_t pos = 0;
    auto take = [&](int64_t bytes) {
        int64_t at = pos;
        pos += (int64_t)align_up((size_t)bytes, 256);
        return at;
    };
    const NetOffsets o = net_offsets(c);
    for (int e = 0; e < c->n_enc; ++e) {
        for (int l = 0; l < kL; ++l) q.grid[e][l] = take(o.cells[l] * kF * 2);
        if (c->grid_only) continue;  // no encoder MLP
        q.w1[e] = take(kH * enc_in(c) * 2);
        q.w2[e] = take(kH * kH * 2);
        q.w3[e] = take(kH * kH * 2);
        q.b1[e] = take(kH * 4);
        q.b2[e] = take(kH * 4);
        q.b3[e] = take(kH * 4);
    }
    if (c->n_enc == 1) {
        for (int l = 0; l < kL; ++l) q.grid[1][l] = q.grid[0][l];
        q.w1[1] = q.w1[0]; q.w2[1] = q.w2[0]; q.w3[1] = q.w3[0];
        q.b1[1] = q.b1[0]; q.b2[1] = q.b2[0]; q.b3[1] = q.b3[0];
    }
    q.w4 = take(kH * (c->grid_only ? kK0 : kH) * 2);
    q.w5 = take(kH * kH * 2);
    q.b4 = take(kH * 4);
    q.b5 = take(kH * 4);
    q.w6 = take(kH * 4);
    q.b6 = take(4);
    if (c->grid_only) {  // BF16 only: no FP8 copies
        q.total = pos;
        return q;
    }
    for (int e = 0; e < c->n_enc; ++e) {
        q.q2[e] = take(kH * kH);
        q.q3[e] = take(kH * kH);
        q.s2[e] = take(kH * 4 * 4);
        q.s3[e] = take(kH * 4 * 4);
    }
    if (c->n_enc == 1) {
        q.q2[1] = q.q2[0]; q.q3[1] = q.q3[0]; q.s2[1] = q.s2[0]; q.s3[1] = q.s3[0];
    }
    q.q4 = take(kH * kH);
    q.q5 = take(kH * kH);
    q.s4 = take(kH * 4 * 4);
    q.s5 = take(kH * 4 * 4);
    q.amax = take(4 * 4);
    q.total = pos;
    return q;
}

size_t net_qparam_bytes(const ndf_net_config *c, int prec) {
    (void)prec;
    return (size_t)qlayout(c).total;
}

// Workspace of the calls that decode from given or cached query latents: the
// reference latents [n_ref][128] FP32, and room for a reference list that no kernel uses any
// more (the size stays what callers have laid out).
size_t net_infer_lat_ws_bytes(int64_t n_ref) {
    return align_up((size_t)n_ref * kH * sizeof(float), 256) +
           align_up((size_t)n_ref * sizeof(int64_t), 256);
}

size_t net_latent_cache_bytes(const ndf_net_config *c);

// ndf_infer_field: a BF16 call with several references also holds the query
// latents of every vertex (they are computed once and decoded per reference).
size_t net_infer_ws_bytes(const ndf_net_config *c, int64_t n_ref, int prec) {
    size_t b = net_infer_lat_ws_bytes(n_ref);
    // n_ref >= 2: the query latents are cached in the workspace (BF16 and FP8)
    if (n_ref >= 2 && !c->grid_only) b += align_up(net_latent_cache_bytes(c), 256);
    return b;
}

// ----------------------------------------------------------- quantize ----
// Exponent e of the E8M0 scale 2^e for a block whose largest magnitude is m >= 0:
// the smallest e with m / 2^e <= 448 (the largest E4M3 value, 1.75 * 2^8),
// read exactly from m's fields: with m = M * 2^E, M in [1, 2), e = E - 8 when
// M <= 1.75, else E - 7.  Zero and subnormal m give the smallest scale.
__device__ __forceinline__ int e4m3_block_exp(float m) {
    const uint32_t b = __float_as_uint(m);
    const int ex = (int)(b >> 23);
    const int e = ex - 135 + ((b & 0x7fffffu) > 0x600000u ? 1 : 0);
    return ex == 0 ? -126 : (e < -126 ? -126 : e);
}

__global__ void to_bf16_kernel(const float *__restrict__ src, int64_t n,
                               uint16_t *__restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = f2bf_bits(src[i]);
}

// A fragments of W[128][KIN] (row-major): frag[(ob*KB + kb)*64 + lane][e] =
// W[32 ob + lane%32][k], k natural (first layer) or permuted to match the
// previous layer's output layout.
__global__ void pack_frag_kernel(const float *__restrict__ W, int KIN, int permuted,
                                 uint16_t *__restrict__ frag) {
    const int KB = KIN / 16;
    const int n = kH * KIN;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        const int e = t & 7;
        const int lane = (t >> 3) & 63;
        const int fi = t >> 9;  // fragment index ob*KB + kb
        const int ob = fi / KB, kb = fi % KB;
        const int h = lane >> 5, il = lane & 31;
        const int k = permuted ? 16 * kb + 8 * (e >> 2) + 4 * h + (e & 3) : 16 * kb + 8 * h + e;
        frag[t] = f2bf_bits(W[(32 * ob + il) * KIN + k]);
    }
}

// The input that lane half h of k-block kb holds in byte t of the MFMA 32x32x64
// A and B operands (the previous layer's output layout):
//   f = 64 kb + 32 (t/16) + 8 ((t%16)/4) + 4 h + t%4.
// The hardware's K order puts bytes t < 16 of both lane halves in its first
// 32-element scale block and bytes t >= 16 in the second, so scale block b of
// k-block kb is inputs 64 kb + 32 b .. + 31, and its E8M0 scale comes from the
// lane half h = b.
__host__ __device__ inline int fp8_feature(int kb, int h, int t) {
    return 64 * kb + 32 * (t >> 4) + 8 * ((t & 15) >> 2) + 4 * h + (t & 3);
}

// E8M0 scale bytes of W[128][128]: se[o][2 kb + b] = 127 + e, 2^e the smallest
// power of two with max |W[o][f]| / 2^e <= 448 over the 32 inputs of scale
// block (kb, b).
// Thread o of a 128-thread block owns row o; fragment (ob, kb) lane l byte t holds
// W[32 ob + l%32][f] / 2^e (exact: a power of two), written 4 bytes at a time.
__device__ __forceinline__ void pack_row_fp8(const float *__restrict__ w, int o,
                                             uint32_t *__restrict__ frag, int *__restrict__ se) {
    const int ob = o >> 5, il = o & 31;
    for (int kb = 0; kb < 2; ++kb) {
        float inv[2];
        for (int b = 0; b < 2; ++b) {
            float m = 0.f;
            for (int f = 64 * kb + 32 * b; f < 64 * kb + 32 * b + 32; ++f)
                m = fmaxf(m, fabsf(w[f]));
            const int e = e4m3_block_exp(m);
            se[o * 4 + 2 * kb + b] = 127 + e;
            inv[b] = __uint_as_float((uint32_t)(127 - e) << 23);  // 2^-e
        }
        for (int h = 0; h < 2; ++h) {
            const int lane = 32 * h + il;
            for (int t = 0; t < 32; t += 4) {
                float v[4];
                for (int c = 0; c < 4; ++c) {
                    const int f = fp8_feature(kb, h, t + c);
                    v[c] = w[f] * inv[t >> 4];
                }
                int wd = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], 0, false);
                wd = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], wd, true);
                frag[((ob * 2 + kb) * 64 + lane) * 8 + (t >> 2)] = (uint32_t)wd;
            }
        }
    }
}

__global__ void pack_fp8_kernel(const float *__restrict__ W, uint32_t *__restrict__ frag,
                                int *__restrict__ se) {
    const int o = threadIdx.x;  // 128 threads
    pack_row_fp8(W + (int64_t)o * kH, o, frag, se);
}

static void launch_calibrate(const ndf_net_config *c, const QLayout &q, char *Q, hipStream_t st);

__global__ void zero_i32_kernel(int *__restrict__ p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

__global__ void copy_f32_kernel(const float *__restrict__ src, int n, float *__restrict__ dst) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        dst[i] = src[i];
}

int launch_net_quantize(const ndf_net_config *c, const float *P, int prec, void *qp,
                        hipStream_t st) {
    if (prec != NDF_PREC_BF16 && prec != NDF_PREC_FP8_E4M3) return NDF_E_UNSUPPORTED;
    const NetOffsets o = net_offsets(c);
    const QLayout q = qlayout(c);
    char *Q = (char *)qp;
    for (int e = 0; e < c->n_enc; ++e) {
        for (int l = 0; l < kL; ++l) {
            const int64_t n = o.cells[l] * kF;
            int64_t nb = ceil_div(n, 256);
            hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)(nb < 4096 ? nb : 4096)), dim3(256),
                               0, st, P + o.grid[e][l], n, (uint16_t *)(Q + q.grid[e][l]));
        }
        if (c->grid_only) continue;
        hipLaunchKernelGGL(pack_frag_kernel, dim3(16), dim3(256), 0, st, P + o.W1[e], enc_in(c), 0,
                           (uint16_t *)(Q + q.w1[e]));
        hipLaunchKernelGGL(pack_frag_kernel, dim3(64), dim3(256), 0, st, P + o.W2[e], kH, 1,
                           (uint16_t *)(Q + q.w2[e]));
        hipLaunchKernelGGL(pack_frag_kernel, dim3(64), dim3(256), 0, st, P + o.W3[e], kH, 1,
                           (uint16_t *)(Q + q.w3[e]));
        hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(128), 0, st, P + o.b1[e], kH,
                           (float *)(Q + q.b1[e]));
        hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(128), 0, st, P + o.b2[e], kH,
                           (float *)(Q + q.b2[e]));
        hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(128), 0, st, P + o.b3[e], kH,
                           (float *)(Q + q.b3[e]));
    }
    if (c->grid_only)  // W4 [128][32] on the merged grid features, natural input order
        hipLaunchKernelGGL(pack_frag_kernel, dim3(16), dim3(256), 0, st, P + o.W4, kK0, 0,
                           (uint16_t *)(Q + q.w4));
    else
        hipLaunchKernelGGL(pack_frag_kernel, dim3(64), dim3(256), 0, st, P + o.W4, kH, 1,
                           (uint16_t *)(Q + q.w4));
    hipLaunchKernelGGL(pack_frag_kernel, dim3(64), dim3(256), 0, st, P + o.W5, kH, 1,
                       (uint16_t *)(Q + q.w5));
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(128), 0, st, P + o.b4, kH,
                       (float *)(Q + q.b4));
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(128), 0, st, P + o.b5, kH,
                       (float *)(Q + q.b5));
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(128), 0, st, P + o.w6, kH,
                       (float *)(Q + q.w6));
    hipLaunchKernelGGL(copy_f32_kernel, dim3(1), dim3(1), 0, st, P + o.b6, 1, (float *)(Q + q.b6));
    if (c->grid_only) return status_of_launch();
    // FP8 copies of the 128x128 layers (both precisions share one packed blob)
    auto fp8 = [&](const float *W, int64_t qoff, int64_t soff) {
        hipLaunchKernelGGL(pack_fp8_kernel, dim3(1), dim3(kH), 0, st, W, (uint32_t *)(Q + qoff),
                           (int *)(Q + soff));
    };
    for (int e = 0; e < c->n_enc; ++e) {
        fp8(P + o.W2[e], q.q2[e], q.s2[e]);
        fp8(P + o.W3[e], q.q3[e], q.s3[e]);
    }
    fp8(P + o.W4, q.q4, q.s4);
    fp8(P + o.W5, q.q5, q.s5);
    // static activation scales: the largest |input| of layers 2..5 over the
    // calibration set, measured with the BF16 layers just packed
    launch_calibrate(c, q, Q, st);
    return status_of_launch();
}

// ------------------------------------------------------- fused kernel ----
// The vertices of the latent mode (MODE 1), 256 per launch, as a kernel argument (a list in
// device memory took a launch of its own, 5 us, in front of every call); the other modes
// take the vertices or positions in order.
constexpr int kLatRefs = 256;
struct RefVerts {
    int64_t v[kLatRefs];
};
struct NoVerts {};
template <int MODE>
using QueryList = std::conditional_t<MODE == 1, RefVerts, NoVerts>;

struct InferArgs {
    const uint16_t *grid[kL];   // bf16 [cells][8] of the query encoder
    const bf16x8 *w[5];         // A fragments W1..W5
    const float *b[5];          // b1..b5
    const float *w6;
    const float *b6;
    GridGeom g;
    int64_t V;
    int64_t fuse_ref;  // field modes: reference vertex whose latent the workgroup computes
                       // itself, or -1: read it from ref_lat
    // SEP (two encoders): the reference encoder's grids, W1..W3 and b1..b3
    const uint16_t *rgrid[kL];
    const bf16x8 *rw[3];
    const float *rb[3];
};

// LDS plan (bytes): W1 8K | W2..W5 4 x 32K | b1..b5 5 x 512 | w6 512 | ref latent 512
constexpr int kFragW1 = 4 * 2 * 64;   // bf16x8 elements
constexpr int kFragW = 4 * 8 * 64;

// Corner cells (int32) and weights of vertex v on a level of sizes R; same
// arithmetic as the training lookup.  HASH: the level may be hashed (hm != 0).
template <bool HASH>
__device__ __forceinline__ void corners32(const GridGeom &g, const int R[3], int64_t v, int idx[8],
                                          float w[8], uint32_t hm) {
    corners_R32<HASH>(g, R, v, idx, w, hm);
}

enum { LAY_RELU = 0, LAY_LATENT = 1, LAY_HEAD = 2, LAY_LATENT_OUT = 3, LAY_LATENT_CACHE = 4 };

// Query-latent cache: the bf16 latents of 64-vertex tiles in the B-operand
// register order of the fused kernel, [tile][k-block 8][query half 2][lane 64]
// 16-byte chunks (16 KB per tile), so a tile reloads with 16 coalesced loads.
__device__ __forceinline__ int64_t cache_chunk(int64_t tile, int kb, int q, int lane) {
    return ((tile * 8 + kb) * 2 + q) * 64 + lane;
}

// One 128-wide layer for the wave's 2 x 32 queries.  in: KB k-blocks of B
// operands.  The accumulators start at the bias, so the epilogue is only the
// bf16 packing (plus ReLU on the packed pairs, the latent product, or the head).
// NQ: query blocks computed (1: only block 0, for a single row such as the
// reference vertex in a prologue; its bits are those of block 0 with NQ = 2)
template <int KB, int KIND, int NQ = 2>
__device__ __forceinline__ void dense_layer(const bf16x8 *__restrict__ wf,
                                            const float *__restrict__ bias,
                                            const float *__restrict__ ref,
                                            const float *__restrict__ w6,
                                            const bf16x8 (&in)[8][2], bf16x8 (&out)[8][2],
                                            float (&part)[2], float *__restrict__ lat_out,
                                            int64_t row0, const bool (&ok)[2], int lane, int h4) {
    // per-lane row offset 4*(lane/32); rows of block ob are h4 + 32 ob + 8 (r/4) + r%4
    const float *bias_h = bias + h4;
    const float *ref_h = ref + h4;
    const float *w6_h = w6 + h4;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        // rows 8 g + 0..3 of block ob are contiguous: one 16-byte LDS read each
        f32x16 acc0, acc1;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias_h + 32 * ob + 8 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc0[4 * g + i] = acc1[4 * g + i] = bv[i];
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const bf16x8 a = wf[(ob * KB + kb) * 64 + lane];
            acc0 = mfma32(a, in[kb][0], acc0);
            if (NQ == 2) acc1 = mfma32(a, in[kb][1], acc1);
        }
        if (KIND == LAY_HEAD) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 wv = *reinterpret_cast<const f32x4 *>(w6_h + 32 * ob + 8 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    part[0] = fmaf(wv[i], relu_f32(acc0[4 * g + i]), part[0]);
                    if (NQ == 2) part[1] = fmaf(wv[i], relu_f32(acc1[4 * g + i]), part[1]);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                u32x4 t0, t1;  // built whole, so the previous contents of out[] die here
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) {
                    const int r = 8 * s + 2 * e2;  // rows r, r+1 (same 4-row group)
                    uint32_t p0 = pack_bf16x2(acc0[r], acc0[r + 1]);
                    uint32_t p1 = NQ == 2 ? pack_bf16x2(acc1[r], acc1[r + 1]) : 0u;
                    if (KIND == LAY_RELU) {
                        p0 = relu_bf16x2(p0);
                        if (NQ == 2) p1 = relu_bf16x2(p1);
                    } else if (KIND != LAY_LATENT_CACHE) {  // latent: bf16 values (exact
                                                            // products with the bf16 reference)
                        const int ic = 32 * ob + 8 * (r >> 2) + (r & 3);
                        if (KIND == LAY_LATENT_OUT) {
                            const int64_t n0 = row0 + (lane & 31), n1 = n0 + 32;
                            if (ok[0]) {
                                lat_out[n0 * kH + ic + h4] = bf_lo(p0);
                                lat_out[n0 * kH + ic + h4 + 1] = bf_hi(p0);
                            }
                            if (NQ == 2 && ok[1]) {
                                lat_out[n1 * kH + ic + h4] = bf_lo(p1);
                                lat_out[n1 * kH + ic + h4 + 1] = bf_hi(p1);
                            }
                        } else {
                            const f32x2 rv = *reinterpret_cast<const f32x2 *>(ref_h + ic);
                            const float ra = rv[0], rb = rv[1];
                            p0 = pack_bf16x2(bf_lo(p0) * ra, bf_hi(p0) * rb);
                            if (NQ == 2) p1 = pack_bf16x2(bf_lo(p1) * ra, bf_hi(p1) * rb);
                        }
                    }
                    t0[e2] = p0;
                    t1[e2] = p1;
                }
                if (KIND == LAY_RELU || KIND == LAY_LATENT) {
                    out[2 * ob + s][0] = __builtin_bit_cast(bf16x8, t0);
                    if (NQ == 2) out[2 * ob + s][1] = __builtin_bit_cast(bf16x8, t1);
                } else if (KIND == LAY_LATENT_CACHE) {
                    u32x4 *cache = reinterpret_cast<u32x4 *>(lat_out);
                    const int64_t tile = row0 / 64;
                    cache[cache_chunk(tile, 2 * ob + s, 0, lane)] = t0;
                    cache[cache_chunk(tile, 2 * ob + s, 1, lane)] = t1;
                }
            }
        }
    }
}

template <int MODE>
__device__ __forceinline__ int64_t query_vertex(const QueryList<MODE> &ql, int64_t n) {
    if constexpr (MODE == 1)
        return ql.v[n];
    else
        return n;
}

// Work of the field and latent kernels: workgroup b owns the contiguous tiles
// [ntiles b / G, ntiles (b + 1) / G) (neighbouring tiles share grid corners in
// L2), and its waves claim them one at a time from an LDS counter, so a wave that
// starts late (wave 0, after the reference latent) simply takes fewer.
__device__ __forceinline__ int64_t wg_tile_begin(int64_t ntiles, int64_t b) {
    return ntiles * b / gridDim.x;
}

__device__ __forceinline__ int64_t claim_tile(int *counter) {
    int c = 0;
    if ((threadIdx.x & 63) == 0) c = atomicAdd(counter, 1);
    return __builtin_amdgcn_readfirstlane(c);
}

// The reference latent computed in a field kernel's prologue is published with a
// workgroup-scope release (after its LDS stores) and awaited with an acquire just
// before its first use, so the other waves start their tiles meanwhile.
__device__ __forceinline__ void publish_flag(int *flag) {
    __hip_atomic_store(flag, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void await_flag(int *flag) {
    while (__hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0)
        __builtin_amdgcn_s_sleep(1);
}

// MODE 0: field (out[v] = Phi(ref, v) for v < nq); MODE 1: latents of the
// vertices in ql (lat_out[n][128], bf16-rounded values stored as FP32);
// MODE 2: latents of vertices 0 .. nq-1 into the query-latent cache (out);
// MODE 3: field at the continuous positions qpos[n][3] in [-1, 1]^3.
// HASH: some grid level is a hash table (compiled out when every level is dense).
// SEP: a field mode of a two-encoder network that computes the reference latent in
// the prologue: the reference encoder's layers are staged first, then replaced
// by the query encoder's.
// Calibration set of the FP8 activation scales (MODE 4): kCalRefs references and
// kCalQueries queries spread evenly over the vertex range, v = (2 i + 1) V / (2 n).
constexpr int kCalRefs = 32;
constexpr int kCalQueries = 2048;
__host__ __device__ inline int64_t cal_vertex(int64_t i, int64_t n, int64_t V) {
    return ((2 * i + 1) * V) / (2 * n);
}

// Largest |value| of a wave's bf16 operands (the rows of valid queries), folded
// into *dst with an integer max on the float bits (non-negative floats order
// like their bits).
template <int KB>
__device__ __forceinline__ void wave_max_into(const bf16x8 (&v)[8][2], const bool (&ok)[2],
                                              int *__restrict__ dst) {
    float m = 0.f;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (ok[q]) m = fmaxf(m, fabsf((float)v[kb][q][e]));
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(dst, __float_as_int(m));
}

// GO: a grid-only network (the encoder MLP omitted): the latent is the gathered
// grid features (32, in the gather's natural feature order 16 kb + 8 h + e), the
// product with the reference's feeds W4 [128][32] (held in s_w1) and W5 sits in
// s_w[3]; field modes only, shared grid or separate grids alike.
template <int MODE, bool HASH, bool SEP = false, bool GO = false, bool FF = false>
__global__ __launch_bounds__(kInferThreads) void infer_kernel(InferArgs A,
                                                              const QueryList<MODE> ql,
                                                              int64_t nq,
                                                              const float *__restrict__ ref_lat,
                                                              float *__restrict__ out,
                                                              const float *__restrict__ qpos) {
    // MODE 4: calibration of the FP8 activation scales: workgroup w takes reference
    // cal_vertex(w, gridDim.x) against the nq calibration queries and folds the
    // largest |input| of layers 2..5 into ((int *)out)[0..3]
    // FF: Fourier features after the grid features (k-blocks 2 .. KB1 - 1)
    constexpr bool kField = MODE == 0 || MODE == 3 || MODE == 4;
    constexpr int KB1 = FF ? kK0F / 16 : 2;
    constexpr int kW1 = 4 * KB1 * 64;
    __shared__ bf16x8 s_w1[kW1];
    __shared__ bf16x8 s_w[4][kFragW];
    __shared__ __attribute__((aligned(16))) float s_b[5][kH];
    __shared__ __attribute__((aligned(16))) float s_w6[kH];
    __shared__ __attribute__((aligned(16))) float s_ref[kH];
    __shared__ int s_sync[2];  // reference latent ready, next tile of the workgroup
    const int64_t fref = MODE == 4 ? cal_vertex(blockIdx.x, gridDim.x, A.V) : A.fuse_ref;
    // a field of the shared encoder overlaps the reference latent with the first
    // tiles (a two-encoder field swaps the encoder's weights after it: a barrier)
    constexpr bool kOverlap = (MODE == 0 || MODE == 3) && !SEP;

    const int tid = threadIdx.x;
    if (tid == 0) {
        s_sync[0] = 0;
        s_sync[1] = 0;
    }
    if (GO) {
        for (int i = tid; i < kFragW1; i += kInferThreads) s_w1[i] = A.w[3][i];
        for (int i = tid; i < kFragW; i += kInferThreads) s_w[3][i] = A.w[4][i];
        for (int i = tid; i < 2 * kH; i += kInferThreads)
            s_b[3 + i / kH][i % kH] = A.b[3 + i / kH][i % kH];
    } else {
        stage_lds<kW1, kInferThreads>(s_w1, SEP ? A.rw[0] : A.w[0], tid);
        constexpr int nlay = kField ? 4 : 2;  // latent modes need W2, W3 only
#pragma unroll
        for (int L = 0; L < nlay; ++L)
            stage_lds<kFragW, kInferThreads>(s_w[L], SEP && L < 2 ? A.rw[L + 1] : A.w[L + 1], tid);
        for (int i = tid; i < 5 * kH; i += kInferThreads)
            s_b[i / kH][i % kH] = (SEP && i < 3 * kH ? A.rb[i / kH] : A.b[i / kH])[i % kH];
    }
    const bool fuse = kField && A.fuse_ref >= 0;
    for (int i = tid; i < kH; i += kInferThreads) {
        s_w6[i] = A.w6[i];
        s_ref[i] = kField && !fuse ? ref_lat[i] : 0.f;
    }
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    if (fuse) {
        // The reference latent with the shared encoder (same layers, same packing
        // as the latent mode, so the same bits): wave 0 runs the reference as the
        // only valid row of one tile and leaves its 128 latents in s_ref.
        if (wave == 0) {
            int h4 = 4 * h;
            const bool ok[2] = {jl == 0, false};
            bf16x8 a[8][2], b[8][2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const uint16_t *const *G = SEP ? A.rgrid : A.grid;
                const uint16_t *grid = h ? G[2 * kb + 1] : G[2 * kb];
                int R[3];
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) R[ax] = h ? A.g.R[2 * kb + 1][ax] : A.g.R[2 * kb][ax];
                const uint32_t hm = HASH ? (h ? A.g.hmask[2 * kb + 1] : A.g.hmask[2 * kb]) : 0u;
                int idx[8];
                float w[8];
                corners32<HASH>(A.g, R, fref, idx, w, hm);
                float sf[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int cn = 0; cn < 8; ++cn) {
                    const i32x4 raw = *reinterpret_cast<const i32x4 *>(grid + (int64_t)idx[cn] * kF);
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t u = (uint32_t)raw[p];
                        sf[2 * p] = fmaf(w[cn], __uint_as_float(u << 16), sf[2 * p]);
                        sf[2 * p + 1] = fmaf(w[cn], __uint_as_float(u & 0xffff0000u), sf[2 * p + 1]);
                    }
                }
                bf16x8 t;
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = f2bf(sf[e]);
                a[kb][0] = a[kb][1] = t;
                if (GO && jl == 0) {  // the latent is the rounded grid features
#pragma unroll
                    for (int e = 0; e < 8; ++e) s_ref[16 * kb + 8 * h + e] = (float)t[e];
                }
            }
            if (FF) {
                float pp[3];
                vertex_p(A.g, fref, pp);
#pragma unroll
                for (int kb = 2; kb < KB1; ++kb) a[kb][0] = a[kb][1] = ff_chunk(kb, h, pp);
            }
            float part[2] = {0.f, 0.f};
            if (!GO) {
                // query block 0 only: the reference is its row 0
                dense_layer<KB1, LAY_RELU, 1>(s_w1, s_b[0], s_ref, s_w6, a, b, part, nullptr, 0,
                                              ok, lane, h4);
                dense_layer<8, LAY_RELU, 1>(s_w[0], s_b[1], s_ref, s_w6, b, a, part, nullptr, 0,
                                            ok, lane, h4);
                dense_layer<8, LAY_LATENT_OUT, 1>(s_w[1], s_b[2], s_ref, s_w6, a, b, part, s_ref,
                                                  0, ok, lane, h4);
            }
            if (kOverlap) publish_flag(&s_sync[0]);
        }
    }
    if (fuse && !kOverlap) {
        __syncthreads();
        if (SEP && !GO) {  // the query encoder's layers replace the reference encoder's
            for (int i = tid; i < kW1; i += kInferThreads) s_w1[i] = A.w[0][i];
            for (int L = 0; L < 2; ++L)
                for (int i = tid; i < kFragW; i += kInferThreads) s_w[L][i] = A.w[L + 1][i];
            for (int i = tid; i < 3 * kH; i += kInferThreads)
                s_b[i / kH][i % kH] = A.b[i / kH][i % kH];
            __syncthreads();
        }
    }
    const float b6 = A.b6[0];
    const int64_t ntiles = ceil_div(nq, 64);
    // MODE 4: every workgroup takes all calibration tiles (against its own reference)
    const int64_t t_lo = MODE == 4 ? 0 : wg_tile_begin(ntiles, blockIdx.x);
    const int64_t t_hi = MODE == 4 ? ntiles : wg_tile_begin(ntiles, blockIdx.x + 1);
    bool await_ref = kOverlap && fuse;
    for (int64_t k = 0;; ++k) {
        const int64_t tile = MODE == 4 ? wave + k * kInferWaves : t_lo + claim_tile(&s_sync[1]);
        if (tile >= t_hi) break;
        const int64_t row0 = tile * 64;
        // opaque per tile, so the per-lane LDS addresses derived from it are
        // formed inside the loop (base + immediate) instead of hoisted and spilled
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        bool ok[2];
        int64_t vq[2];
        float pq[2][3];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t n = row0 + q * 32 + jl;
            ok[q] = n < nq;
            vq[q] = ok[q] && MODE != 3 ? (MODE == 4 ? cal_vertex(n, nq, A.V)
                                                    : query_vertex<MODE>(ql, n))
                                      : 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) pq[q][a] = MODE == 3 && ok[q] ? qpos[3 * n + a] : 0.f;
        }
        // grid gather: k-block kb, half h -> level 2 kb + h (its 8 features)
        bf16x8 a[8][2], b[8][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            // both candidate levels are uniform; the lane half picks one
            const uint16_t *grid = h ? A.grid[2 * kb + 1] : A.grid[2 * kb];
            int R[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) R[ax] = h ? A.g.R[2 * kb + 1][ax] : A.g.R[2 * kb][ax];
            const uint32_t hm = HASH ? (h ? A.g.hmask[2 * kb + 1] : A.g.hmask[2 * kb]) : 0u;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                int idx[8];
                float w[8];
                if (MODE == 3)
                    corners_pos32<HASH>(R, pq[q], idx, w, hm);
                else
                    corners32<HASH>(A.g, R, vq[q], idx, w, hm);
                float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int cn = 0; cn < 8; ++cn) {
                    const i32x4 raw = *reinterpret_cast<const i32x4 *>(grid + (int64_t)idx[cn] * kF);
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t u = (uint32_t)raw[p];
                        s[2 * p] = fmaf(w[cn], __uint_as_float(u << 16), s[2 * p]);
                        s[2 * p + 1] = fmaf(w[cn], __uint_as_float(u & 0xffff0000u), s[2 * p + 1]);
                    }
                }
                bf16x8 t;
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = f2bf(s[e]);
                a[kb][q] = t;
            }
        }
        if (FF) {  // the raw position and its Fourier features
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float pp[3];
                if (MODE == 3)
                    clamp_p(pq[q], pp);
                else
                    vertex_p(A.g, vq[q], pp);
#pragma unroll
                for (int kb = 2; kb < KB1; ++kb) a[kb][q] = ff_chunk(kb, h, pp);
            }
        }
        float part[2] = {0.f, 0.f};
        if (GO) {
            if (await_ref) {
                await_flag(&s_sync[0]);
                await_ref = false;
            }
            // product of the query's and the reference's grid features (exact in
            // FP32 for bf16 values, then rounded to bf16), decoder on top
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        b[kb][q][e] = f2bf((float)a[kb][q][e] * s_ref[16 * kb + 8 * h + e]);
            dense_layer<2, LAY_RELU>(s_w1, s_b[3], s_ref, s_w6, b, a, part, nullptr, row0, ok, lane,
                                     h4);
            dense_layer<8, LAY_HEAD>(s_w[3], s_b[4], s_ref, s_w6, a, b, part, nullptr, row0, ok,
                                     lane, h4);
        } else if (MODE == 4) {
            int *amax = reinterpret_cast<int *>(out);
            dense_layer<KB1, LAY_RELU>(s_w1, s_b[0], s_ref, s_w6, a, b, part, nullptr, row0, ok,
                                       lane, h4);
            wave_max_into<8>(b, ok, amax + 0);
            dense_layer<8, LAY_RELU>(s_w[0], s_b[1], s_ref, s_w6, b, a, part, nullptr, row0, ok,
                                     lane, h4);
            wave_max_into<8>(a, ok, amax + 1);
            dense_layer<8, LAY_LATENT>(s_w[1], s_b[2], s_ref, s_w6, a, b, part, nullptr, row0, ok,
                                       lane, h4);
            wave_max_into<8>(b, ok, amax + 2);
            dense_layer<8, LAY_RELU>(s_w[2], s_b[3], s_ref, s_w6, b, a, part, nullptr, row0, ok,
                                     lane, h4);
            wave_max_into<8>(a, ok, amax + 3);
            continue;
        } else {
        dense_layer<KB1, LAY_RELU>(s_w1, s_b[0], s_ref, s_w6, a, b, part, nullptr, row0, ok, lane, h4);
        dense_layer<8, LAY_RELU>(s_w[0], s_b[1], s_ref, s_w6, b, a, part, nullptr, row0, ok, lane, h4);
        if (MODE == 1) {
            dense_layer<8, LAY_LATENT_OUT>(s_w[1], s_b[2], s_ref, s_w6, a, b, part, out, row0, ok,
                                           lane, h4);
            continue;
        }
        if (MODE == 2) {
            dense_layer<8, LAY_LATENT_CACHE>(s_w[1], s_b[2], s_ref, s_w6, a, b, part, out, row0,
                                             ok, lane, h4);
            continue;
        }
        if (await_ref) {  // layer 3's epilogue forms the product with the reference latent
            await_flag(&s_sync[0]);
            await_ref = false;
        }
        dense_layer<8, LAY_LATENT>(s_w[1], s_b[2], s_ref, s_w6, a, b, part, nullptr, row0, ok,
                                   lane, h4);
        dense_layer<8, LAY_RELU>(s_w[2], s_b[3], s_ref, s_w6, b, a, part, nullptr, row0, ok, lane, h4);
        dense_layer<8, LAY_HEAD>(s_w[3], s_b[4], s_ref, s_w6, a, b, part, nullptr, row0, ok, lane, h4);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float y = part[q] + __shfl_xor(part[q], 32, 64) + b6;
            if (h == 0 && ok[q]) out[row0 + q * 32 + jl] = y;
        }
    }
}


// ------------------------------------------------------------ FP8 path ----
// Layers 2..5 run as MFMA 32x32x64 on OCP E4M3 with microscaling (MX): every
// operand lane carries an E8M0 power-of-two scale for its 32 K-values, which
// the scaled MFMA applies in hardware.
//  * weights: per output row and block of 32 inputs, 2^e with max|W| / 2^e <=
//    448 over the block, so accumulators come out in true units and start at
//    the bias like the BF16 path;
//  * activations: per query and block of 32 features (one output block of the
//    previous layer, held 16 + 16 by lanes l and l ^ 32), 2^e with max|a| / 2^e
//    <= 448; the quantising conversion divides by the scale itself.
// The hardware groups K into scale blocks in its own order: bytes 0..15 of both
// lane halves form the first block of 32, bytes 16..31 the second, and lane half
// h carries the scale of block h (measured on gfx950 with half-dependent
// operand values and scales).
// The first layer (32 inputs, 6% of the work) stays BF16.  Block k = 64 kb +
// 32 h + t of a lane comes from output blocks 2 kb (t < 16) and 2 kb + 1
// (t >= 16) of the previous layer; the packed weights absorb that order (see
// pack_row_fp8).
typedef __attribute__((ext_vector_type(8))) int i32x8;

__device__ __forceinline__ f32x16 mfma_fp8(const i32x8 &a, int sa, const i32x8 &b, int sb,
                                           const f32x16 &c) {
    // A scaled by 2^(sa - 127), B by 2^(sb - 127)
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, sa, 0, sb);
}

// Two floats divided by the power of two s -> E4M3 pair into half HI of w.
template <bool HI>
__device__ __forceinline__ int cvt_fp8x2(int w, float a, float b, float s) {
    const s16x2 old = __builtin_bit_cast(s16x2, w);
    return __builtin_bit_cast(int, __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(old, a, b, s, HI));
}

// The 32 values of one lane (f(o, r) = output block 2 kb + o, row r of the lane;
// byte t = 16 o + r) -> E4M3 with the layer's static activation scale s (the
// conversion divides by s; the caller has clamped the values to [-448 s, 448 s],
// so none overflows).
template <typename F>
__device__ __forceinline__ void quant_static(F f, float s, i32x8 &out) {
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int o = d >> 2, r = 4 * (d & 3);
        const int w = cvt_fp8x2<false>(0, f(o, r), f(o, r + 1), s);
        out[d] = cvt_fp8x2<true>(w, f(o, r + 2), f(o, r + 3), s);
        // pinned here: left free, the conversions sink to their uses in the next
        // layer and keep all the FP32 accumulators alive until then
        asm volatile("" : "+v"(out[d]));
    }
}

// Static activation scales of the FP8 layers (inputs of layers 2..5): 2^e with e
// the smallest exponent for which twice the calibrated maximum |activation| stays
// within E4M3's 448 (ndf_net_quantize measures the maxima on a fixed calibration
// set; twice leaves headroom for inputs beyond it, which are clamped).
struct ActScales {
    float s[4];    // 2^e per layer input (layers 2, 3, 4, 5)
    float clip[4]; // 448 * s
    int sbyte[4];  // E8M0 byte 127 + e (the MFMA's B-operand scale)
};

__device__ __forceinline__ ActScales act_scales(const int *__restrict__ amax) {
    ActScales a;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int e = e4m3_block_exp(2.0f * __int_as_float(amax[l]));
        a.s[l] = __uint_as_float((uint32_t)(e + 127) << 23);
        a.clip[l] = 448.0f * a.s[l];
        a.sbyte[l] = e + 127;
    }
    return a;
}

struct InferArgs8 {
    const uint16_t *grid[kL];
    const bf16x8 *w1;
    const i32x8 *q[4];    // W2..W5 fp8 fragments
    const int *se[4];     // their E8M0 bytes [128][4] (row, 32-input block)
    const int *amax;      // calibrated max |input| of layers 2..5 (float bits)
    const float *b[5];
    const float *w6;
    const float *b6;
    GridGeom g;
    int64_t fuse_ref;  // as in InferArgs
};

constexpr int kFrag8 = 4 * 2 * 64;  // i32x8 per 128x128 fp8 layer

// NQ as in dense_layer
template <int KIND, bool BF16IN, int KB1, int NQ = 2>
__device__ __forceinline__ void dense_layer_fp8(
    const bf16x8 *__restrict__ w16, const i32x8 *__restrict__ w8, const int *__restrict__ se,
    const float *__restrict__ bias, const float *__restrict__ ref, const float *__restrict__ w6,
    const bf16x8 (&in16)[KB1][2], const i32x8 (&in8)[2][2], int sin, i32x8 (&out8)[2][2],
    float so, float clip, float (&part)[2], float *__restrict__ lat_out, int64_t row0,
    const bool (&ok)[2], int lane, int h4) {
    // sin: the E8M0 scale byte of this layer's inputs; so, clip: the scale of the
    // next layer's inputs and 448 so
    __builtin_amdgcn_sched_barrier(0);
    const float *bias_h = bias + h4;
    const float *ref_h = ref + h4;
    const float *w6_h = w6 + h4;
    const int il = lane & 31, hh = h4 >> 2;
    if (KIND == LAY_HEAD) {
        // last layer: one output block and query half at a time, straight into
        // the w6 dot product (keeps the register footprint of the head small)
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                f32x16 acc;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias_h + 32 * ob + 8 * g);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[4 * g + i] = bv[i];
                }
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    acc = mfma_fp8(w8[(ob * 2 + kb) * 64 + lane], se[(32 * ob + il) * 4 + 2 * kb + hh],
                                   in8[kb][q], sin, acc);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 wv = *reinterpret_cast<const f32x4 *>(w6_h + 32 * ob + 8 * g);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        part[q] = fmaf(wv[i], relu_f32(acc[4 * g + i]), part[q]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return;
    }
#pragma unroll
    for (int op = 0; op < 2; ++op) {
        f32x16 acc[2][2];
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 bv =
                    *reinterpret_cast<const f32x4 *>(bias_h + 32 * (2 * op + o) + 8 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[o][0][4 * g + i] = acc[o][1][4 * g + i] = bv[i];
            }
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const int ob = 2 * op + o;
            if (BF16IN) {
#pragma unroll
                for (int kb = 0; kb < KB1; ++kb) {
                    const bf16x8 a = w16[(ob * KB1 + kb) * 64 + lane];
                    acc[o][0] = mfma32(a, in16[kb][0], acc[o][0]);
                    if (NQ == 2) acc[o][1] = mfma32(a, in16[kb][1], acc[o][1]);
                }
            } else {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const i32x8 a = w8[(ob * 2 + kb) * 64 + lane];
                    const int sa = se[(32 * ob + il) * 4 + 2 * kb + hh];
                    acc[o][0] = mfma_fp8(a, sa, in8[kb][0], sin, acc[o][0]);
                    if (NQ == 2) acc[o][1] = mfma_fp8(a, sa, in8[kb][1], sin, acc[o][1]);
                }
            }
            // fetch one output block's weights at a time (32 registers, not 64)
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (KIND == LAY_LATENT_OUT) {
                if (ok[q]) {
                    float *dst = lat_out + (row0 + 32 * q + il) * kH + h4;
#pragma unroll
                    for (int o = 0; o < 2; ++o)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            dst[32 * (2 * op + o) + 8 * (r >> 2) + (r & 3)] = acc[o][q][r];
                }
            } else if (KIND == LAY_RELU) {
                // ReLU and the clamp to the E4M3 range in one median of three
                quant_static([&](int o, int r) {
                    return __builtin_amdgcn_fmed3f(acc[o][q][r], 0.f, clip);
                }, so, out8[op][q]);
            } else {  // LAY_LATENT: product with the reference latent
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 rv = *reinterpret_cast<const f32x4 *>(
                            ref_h + 32 * (2 * op + o) + 8 * g);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            acc[o][q][4 * g + i] = __builtin_amdgcn_fmed3f(
                                acc[o][q][4 * g + i] * rv[i], -clip, clip);
                    }
                quant_static([&](int o, int r) { return acc[o][q][r]; }, so, out8[op][q]);
            }
            // one query half at a time (keeps the epilogue's temporaries few)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// MODE 0: field (out[v] = Phi(ref, v)); MODE 1: latents of the vertices in
// ql (FP32); MODE 3: field at the continuous positions qpos[n][3].
template <int MODE, bool HASH, bool FF = false>
__global__ __launch_bounds__(kInferThreads) void infer_fp8_kernel(InferArgs8 A,
                                                                  const QueryList<MODE> ql,
                                                                  int64_t nq,
                                                                  const float *__restrict__ ref_lat,
                                                                  float *__restrict__ out,
                                                                  const float *__restrict__ qpos) {
    constexpr bool kField = MODE == 0 || MODE == 3;
    constexpr int KB1 = FF ? kK0F / 16 : 2;  // k-blocks of the encoder input
    __shared__ bf16x8 s_w1[4 * KB1 * 64];
    __shared__ i32x8 s_q[4][kFrag8];
    __shared__ int s_e[4][kH * 4];
    __shared__ __attribute__((aligned(16))) float s_b[5][kH];
    __shared__ __attribute__((aligned(16))) float s_w6[kH];
    __shared__ __attribute__((aligned(16))) float s_ref[kH];
    __shared__ int s_sync[2];  // reference latent ready, next tile of the workgroup

    const int tid = threadIdx.x;
    if (tid == 0) {
        s_sync[0] = 0;
        s_sync[1] = 0;
    }
    stage_lds<4 * KB1 * 64, kInferThreads>(s_w1, A.w1, tid);
    constexpr int nlay = kField ? 4 : 2;
#pragma unroll
    for (int L = 0; L < nlay; ++L) stage_lds<kFrag8, kInferThreads>(s_q[L], A.q[L], tid);
#pragma unroll
    for (int L = 0; L < 4; ++L) stage_lds<kH * 4, kInferThreads>(s_e[L], A.se[L], tid);
    for (int i = tid; i < 5 * kH; i += kInferThreads) s_b[i / kH][i % kH] = A.b[i / kH][i % kH];
    const bool fuse = kField && A.fuse_ref >= 0;
    for (int i = tid; i < kH; i += kInferThreads) {
        s_w6[i] = A.w6[i];
        s_ref[i] = kField && !fuse ? ref_lat[i] : 0.f;
    }
    const ActScales as = act_scales(A.amax);
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    if (fuse) {
        // the reference latent with the shared encoder, as the latent mode computes
        // it (the only valid row of one tile), left in s_ref by wave 0
        if (wave == 0) {
            const int h4 = 4 * h;
            const bool ok[2] = {jl == 0, false};
            bf16x8 g16[KB1][2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const uint16_t *grid = h ? A.grid[2 * kb + 1] : A.grid[2 * kb];
                int R[3];
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) R[ax] = h ? A.g.R[2 * kb + 1][ax] : A.g.R[2 * kb][ax];
                const uint32_t hm = HASH ? (h ? A.g.hmask[2 * kb + 1] : A.g.hmask[2 * kb]) : 0u;
                int idx[8];
                float w[8];
                corners32<HASH>(A.g, R, A.fuse_ref, idx, w, hm);
                float sf[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int cn = 0; cn < 8; ++cn) {
                    const i32x4 raw = *reinterpret_cast<const i32x4 *>(grid + (int64_t)idx[cn] * kF);
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t u = (uint32_t)raw[p];
                        sf[2 * p] = fmaf(w[cn], __uint_as_float(u << 16), sf[2 * p]);
                        sf[2 * p + 1] = fmaf(w[cn], __uint_as_float(u & 0xffff0000u), sf[2 * p + 1]);
                    }
                }
                bf16x8 t;
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = f2bf(sf[e]);
                g16[kb][0] = g16[kb][1] = t;
            }
            if (FF) {
                float pp[3];
                vertex_p(A.g, A.fuse_ref, pp);
#pragma unroll
                for (int kb = 2; kb < KB1; ++kb) g16[kb][0] = g16[kb][1] = ff_chunk(kb, h, pp);
            }
            i32x8 a8[2][2], b8[2][2];
            float part[2] = {0.f, 0.f};
            // query block 0 only: the reference is its row 0
            dense_layer_fp8<LAY_RELU, true, KB1, 1>(s_w1, nullptr, nullptr, s_b[0], s_ref, s_w6,
                                                    g16, b8, 0, a8, as.s[0], as.clip[0], part,
                                                    nullptr, 0, ok, lane, h4);
            dense_layer_fp8<LAY_RELU, false, KB1, 1>(nullptr, s_q[0], s_e[0], s_b[1], s_ref, s_w6,
                                                     g16, a8, as.sbyte[0], b8, as.s[1],
                                                     as.clip[1], part, nullptr, 0, ok, lane, h4);
            dense_layer_fp8<LAY_LATENT_OUT, false, KB1, 1>(nullptr, s_q[1], s_e[1], s_b[2], s_ref,
                                                           s_w6, g16, b8, as.sbyte[1], a8, 0.f,
                                                           0.f, part, s_ref, 0, ok, lane, h4);
            // the other waves start their tiles meanwhile (as in infer_kernel)
            publish_flag(&s_sync[0]);
        }
    }
    // uniform: a scalar register, not a VGPR held across the tile loop
    const float b6 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(A.b6[0])));
    const int64_t ntiles = ceil_div(nq, 64);
    const int64_t t_hi = wg_tile_begin(ntiles, blockIdx.x + 1);
    const int64_t t_lo = wg_tile_begin(ntiles, blockIdx.x);
    bool await_ref = fuse;
    for (int64_t k = 0;; ++k) {
        const int64_t tile = t_lo + claim_tile(&s_sync[1]);
        if (tile >= t_hi) break;
        const int64_t row0 = tile * 64;
        // opaque per tile, like h4: the lane-dependent selects and addresses below
        // are formed inside the loop instead of hoisted and spilled
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        int ln = lane;
        asm volatile("" : "+v"(ln));
        bool ok[2];
        int64_t vq[2];
        float pq[2][3];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t n = row0 + q * 32 + jl;
            ok[q] = n < nq;
            vq[q] = ok[q] && MODE != 3 ? query_vertex<MODE>(ql, n) : 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) pq[q][a] = MODE == 3 && ok[q] ? qpos[3 * n + a] : 0.f;
        }
        bf16x8 g16[KB1][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const uint16_t *grid = h4 ? A.grid[2 * kb + 1] : A.grid[2 * kb];
            int R[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) R[ax] = h4 ? A.g.R[2 * kb + 1][ax] : A.g.R[2 * kb][ax];
            const uint32_t hm = HASH ? (h4 ? A.g.hmask[2 * kb + 1] : A.g.hmask[2 * kb]) : 0u;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                int idx[8];
                float w[8];
                if (MODE == 3)
                    corners_pos32<HASH>(R, pq[q], idx, w, hm);
                else
                    corners32<HASH>(A.g, R, vq[q], idx, w, hm);
                float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int cn = 0; cn < 8; ++cn) {
                    const i32x4 raw = *reinterpret_cast<const i32x4 *>(grid + (int64_t)idx[cn] * kF);
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t u = (uint32_t)raw[p];
                        s[2 * p] = fmaf(w[cn], __uint_as_float(u << 16), s[2 * p]);
                        s[2 * p + 1] = fmaf(w[cn], __uint_as_float(u & 0xffff0000u), s[2 * p + 1]);
                    }
                }
                bf16x8 t;
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = f2bf(s[e]);
                g16[kb][q] = t;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (FF) {  // the raw position and its Fourier features
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float pp[3];
                if (MODE == 3)
                    clamp_p(pq[q], pp);
                else
                    vertex_p(A.g, vq[q], pp);
#pragma unroll
                for (int kb = 2; kb < KB1; ++kb) g16[kb][q] = ff_chunk(kb, h, pp);
            }
        }
        i32x8 a8[2][2], b8[2][2];
        float part[2] = {0.f, 0.f};
        dense_layer_fp8<LAY_RELU, true>(s_w1, nullptr, nullptr, s_b[0], s_ref, s_w6, g16, b8, 0,
                                        a8, as.s[0], as.clip[0], part, nullptr, row0, ok, ln,
                                        h4);
        if (MODE == 1) {
            dense_layer_fp8<LAY_RELU, false>(nullptr, s_q[0], s_e[0], s_b[1], s_ref, s_w6, g16,
                                             a8, as.sbyte[0], b8, as.s[1], as.clip[1], part,
                                             nullptr, row0, ok, ln, h4);
            dense_layer_fp8<LAY_LATENT_OUT, false>(nullptr, s_q[1], s_e[1], s_b[2], s_ref, s_w6,
                                                   g16, b8, as.sbyte[1], a8, 0.f, 0.f, part, out,
                                                   row0, ok, ln, h4);
            continue;
        }
        dense_layer_fp8<LAY_RELU, false>(nullptr, s_q[0], s_e[0], s_b[1], s_ref, s_w6, g16, a8,
                                         as.sbyte[0], b8, as.s[1], as.clip[1], part, nullptr, row0,
                                         ok, ln, h4);
        if (await_ref) {  // layer 3's epilogue forms the product with the reference latent
            await_flag(&s_sync[0]);
            await_ref = false;
        }
        dense_layer_fp8<LAY_LATENT, false>(nullptr, s_q[1], s_e[1], s_b[2], s_ref, s_w6, g16, b8,
                                           as.sbyte[1], a8, as.s[2], as.clip[2], part, nullptr,
                                           row0, ok, ln, h4);
        dense_layer_fp8<LAY_RELU, false>(nullptr, s_q[2], s_e[2], s_b[3], s_ref, s_w6, g16, a8,
                                         as.sbyte[2], b8, as.s[3], as.clip[3], part, nullptr, row0,
                                         ok, ln, h4);
        dense_layer_fp8<LAY_HEAD, false>(nullptr, s_q[3], s_e[3], s_b[4], s_ref, s_w6, g16, b8,
                                         as.sbyte[3], a8, 0.f, 0.f, part, nullptr, row0, ok, ln,
                                         h4);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float y = part[q] + __shfl_xor(part[q], 32, 64) + b6;
            if (h == 0 && ok[q]) out[row0 + q * 32 + jl] = y;
        }
    }
}

// Work of a launch that decodes several references per tile: whole rounds of
// tiles go to the waves workgroup by workgroup (a workgroup's waves take
// neighbouring tiles); the tiles of the last, partial round are split over the
// references (2, 4, ... parts while the parts still fit in one round, dealt in
// wave-major order), so that round takes a fraction of a tile's time instead of a
// whole tile's on a fraction of the waves.  Wave-uniform throughout.
struct RefSplit {
    int64_t w, wt, W, rounds, rem;  // wt: the wave's index in wave-major order (last round)
    int split;
};

__device__ __forceinline__ RefSplit ref_split(int64_t ntiles, int n_ref, bool allow) {
    RefSplit s;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s.W = (int64_t)gridDim.x * kInferWaves;
    s.w = (int64_t)blockIdx.x * kInferWaves + wave;
    s.wt = (int64_t)wave * gridDim.x + blockIdx.x;
    s.rounds = ntiles / s.W;
    s.rem = ntiles - s.rounds * s.W;
    s.split = 1;
    if (allow)
        while (2 * s.split <= n_ref && 2 * s.split * s.rem <= s.W) s.split *= 2;
    return s;
}

// item k of the calling wave: its tile and reference range [r0, r1); false once
// the wave has no more work
__device__ __forceinline__ bool ref_split_item(const RefSplit &s, int64_t k, int n_ref,
                                               int64_t &tile, int &r0, int &r1) {
    if (k < s.rounds) {
        tile = s.w + k * s.W;
        r0 = 0;
        r1 = n_ref;
        return true;
    }
    if (k > s.rounds || s.wt >= s.rem * s.split) return false;
    tile = s.rounds * s.W + s.wt / s.split;
    const int part = (int)(s.wt % s.split);
    r0 = part * n_ref / s.split;
    r1 = (part + 1) * n_ref / s.split;
    return true;
}

// Fields from cached query latents, several references per pass: per 64-vertex
// tile the wave loads the tile's bf16 latents once (16 loads, kept in LDS and
// registers),
// then for each reference of the launch forms the product with that reference's
// latent (the same packed arithmetic as the uncached kernel, so both give the
// same bits) and runs layers 4, 5 and w6.  A launch decodes up to kMultiRefs
// references; the cache is read once per launch instead of once per field.
// Only W4, W5 (64 KB) and the launch's reference latents live in LDS.
// DIFF: two references, out[v] = Phi(ref 0, v) - Phi(ref 1, v) (the difference
// of two fields, Sec. 6.4), both decoded from one read of the tile.
constexpr int kMultiRefs = 16;
constexpr int kLatLds = 5;  // k-blocks of the tile latents held in LDS

template <bool DIFF>
__global__ __launch_bounds__(kInferThreads) void infer_cached_kernel(InferArgs A,
                                                                      const u32x4 *__restrict__ cache,
                                                                      int64_t nq,
                                                                      const float *__restrict__ ref_lat,
                                                                      int n_ref,
                                                                      float *__restrict__ out,
                                                                      int64_t ld_out) {
    __shared__ bf16x8 s_w[2][kFragW];
    __shared__ __attribute__((aligned(16))) float s_b[2][kH];
    __shared__ __attribute__((aligned(16))) float s_w6[kH];
    __shared__ __attribute__((aligned(16))) float s_ref[kMultiRefs][kH];
    // k-blocks 0..kLatLds-1 of each wave's tile latents (the others stay in
    // registers: all eight plus layer 4's 128 accumulators would not fit in 256
    // VGPRs)
    __shared__ u32x4 s_lat[kInferWaves][kLatLds][2][64];
    const int tid = threadIdx.x;
    for (int L = 0; L < 2; ++L)
        for (int i = tid; i < kFragW; i += kInferThreads) s_w[L][i] = A.w[L + 3][i];
    for (int i = tid; i < 2 * kH; i += kInferThreads) s_b[i / kH][i % kH] = A.b[3 + i / kH][i % kH];
    for (int i = tid; i < kH; i += kInferThreads) s_w6[i] = A.w6[i];
    for (int i = tid; i < n_ref * kH; i += kInferThreads) s_ref[i / kH][i % kH] = ref_lat[i];
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    const float b6 = A.b6[0];
    const int64_t ntiles = ceil_div(nq, 64);
    const RefSplit rs = ref_split(ntiles, n_ref, !DIFF);
    for (int64_t k = 0;; ++k) {
        int64_t tile;
        int r0, r1;
        if (!ref_split_item(rs, k, n_ref, tile, r0, r1)) break;
        const int64_t row0 = tile * 64;
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        bool ok[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) ok[q] = row0 + q * 32 + jl < nq;
        // each lane writes and later reads only its own LDS entries (in order
        // within the wave), so no barrier is needed
        u32x4 lat[8 - kLatLds][2];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const u32x4 v = __builtin_nontemporal_load(cache + cache_chunk(tile, kb, q, lane));
                if (kb < kLatLds)
                    s_lat[wave][kb][q][lane] = v;
                else
                    lat[kb - kLatLds][q] = v;
            }
        float y0[2] = {0.f, 0.f};
#pragma unroll 1
        for (int r = r0; r < r1; ++r) {
            // opaque per reference, so the LDS reads of weights and biases stay
            // inside the loop instead of being hoisted out of it into registers
            asm volatile("" : "+v"(h4));
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const float *ref_h = &s_ref[r][0] + h4;
            // layer 4 with the k-blocks outermost, so each product operand is
            // formed once and used by all four output blocks (each accumulator
            // still sums its k-blocks in order: the bits of dense_layer)
            f32x16 acc[4][2];
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 bv = *reinterpret_cast<const f32x4 *>(&s_b[0][0] + h4 + 32 * ob + 8 * g);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[ob][0][4 * g + i] = acc[ob][1][4 * g + i] = bv[i];
                }
            // k-block kb = 2 ob + s holds rows r = 8 s + 2 e2, r + 1 of output block ob
            auto product = [&](int kb, bf16x8 (&bq)[2]) {
                const int obk = kb >> 1, sb = kb & 1;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const u32x4 lv = kb < kLatLds ? s_lat[wave][kb][q][ln] : lat[kb - kLatLds][q];
                    u32x4 t;
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {
                        const int rr = 8 * sb + 2 * e2;
                        const int ic = 32 * obk + 8 * (rr >> 2) + (rr & 3);
                        const f32x2 rv = *reinterpret_cast<const f32x2 *>(ref_h + ic);
                        t[e2] = pack_bf16x2(bf_lo(lv[e2]) * rv[0], bf_hi(lv[e2]) * rv[1]);
                    }
                    bq[q] = __builtin_bit_cast(bf16x8, t);
                }
            };
            // software pipeline: k-block kb + 1's products are formed in the same
            // scheduling region as k-block kb's MFMAs, so their VALU work issues
            // while the matrix core runs
            bf16x8 bq[2][2];
            product(0, bq[0]);
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) {
                if (kb + 1 < 8) product(kb + 1, bq[(kb + 1) & 1]);
#pragma unroll
                for (int ob = 0; ob < 4; ++ob) {
                    const bf16x8 w = s_w[0][(ob * 8 + kb) * 64 + ln];
                    acc[ob][0] = mfma32(w, bq[kb & 1][0], acc[ob][0]);
                    acc[ob][1] = mfma32(w, bq[kb & 1][1], acc[ob][1]);
                }
                // keep each k-block's weight reads with its MFMAs (128 accumulators
                // and 64 cached-latent registers are live here)
                __builtin_amdgcn_sched_barrier(0);
            }
            bf16x8 a[8][2], b[8][2];
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int sb = 0; sb < 2; ++sb) {
                    u32x4 t0, t1;
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {
                        const int rr = 8 * sb + 2 * e2;
                        t0[e2] = relu_bf16x2(pack_bf16x2(acc[ob][0][rr], acc[ob][0][rr + 1]));
                        t1[e2] = relu_bf16x2(pack_bf16x2(acc[ob][1][rr], acc[ob][1][rr + 1]));
                    }
                    a[2 * ob + sb][0] = __builtin_bit_cast(bf16x8, t0);
                    a[2 * ob + sb][1] = __builtin_bit_cast(bf16x8, t1);
                }
            float part[2] = {0.f, 0.f};
            dense_layer<8, LAY_HEAD>(s_w[1], s_b[1], &s_ref[r][0], s_w6, a, b, part, nullptr, row0,
                                     ok, ln, h4);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float y = part[q] + __shfl_xor(part[q], 32, 64) + b6;
                if (DIFF) {
                    if (r == 0) y0[q] = y;
                    else if (h == 0 && ok[q]) out[row0 + q * 32 + jl] = y0[q] - y;
                } else if (h == 0 && ok[q]) {
                    out[(int64_t)r * ld_out + row0 + q * 32 + jl] = y;
                }
            }
        }
    }
}

// E4M3 decoder on cached query latents (many fields of one network at FP8): per
// 64-vertex tile the wave loads its bf16 latents once; per reference it forms
// the product with the reference latent (exact in FP32 for two bf16 values),
// clamps and quantises it with layer 4's static input scale and runs layers 4
// and 5 on the scaled E4M3 MFMA (weights microscaled per row and 32 inputs) and
// the head; kMultiRefs references per launch, the cache read once per launch.
// The encoder ran in BF16 (the cache and the reference latents), so this is the
// BF16 network with its decoder in E4M3.
// The E4M3 operand of layer 4's k-block kb (inputs 64 kb .. 64 kb + 63) takes
// byte t of lane (l, h) from the same lane's bf16 chunk j = 4 kb + 2 (t / 16) +
// (t % 16) / 8, element 4 ((t / 4) % 2) + t % 4 (both hold input
// fp8_feature(kb, h, t)), so the product and its quantisation are lane-local.
__global__ __launch_bounds__(kInferThreads) void infer_cached_fp8_kernel(
    InferArgs8 A, const u32x4 *__restrict__ cache, int64_t nq, const float *__restrict__ ref_lat,
    int n_ref, float *__restrict__ out, int64_t ld_out) {
    __shared__ i32x8 s_q[2][kFrag8];
    __shared__ int s_e[2][kH * 4];
    __shared__ __attribute__((aligned(16))) float s_b[2][kH];
    __shared__ __attribute__((aligned(16))) float s_w6[kH];
    __shared__ __attribute__((aligned(16))) float s_ref[kMultiRefs][kH];
    // chunks 0..kLat8Lds-1 of each wave's tile latents (the rest in registers)
    constexpr int kLat8Lds = 7;
    __shared__ u32x4 s_lat[kInferWaves][kLat8Lds][2][64];
    const int tid = threadIdx.x;
    for (int L = 0; L < 2; ++L)
        for (int i = tid; i < kFrag8; i += kInferThreads) s_q[L][i] = A.q[L + 2][i];
    for (int i = tid; i < 2 * kH * 4; i += kInferThreads)
        s_e[i / (kH * 4)][i % (kH * 4)] = A.se[2 + i / (kH * 4)][i % (kH * 4)];
    for (int i = tid; i < 2 * kH; i += kInferThreads) s_b[i / kH][i % kH] = A.b[3 + i / kH][i % kH];
    for (int i = tid; i < kH; i += kInferThreads) s_w6[i] = A.w6[i];
    for (int i = tid; i < n_ref * kH; i += kInferThreads) s_ref[i / kH][i % kH] = ref_lat[i];
    const ActScales as = act_scales(A.amax);
    __syncthreads();

    const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, jl = lane & 31;
    const float b6 = A.b6[0];
    const int64_t ntiles = ceil_div(nq, 64);
    const bf16x8 unused16[2][2] = {};
    const RefSplit rs = ref_split(ntiles, n_ref, true);
    for (int64_t k = 0;; ++k) {
        int64_t tile;
        int r0, r1;
        if (!ref_split_item(rs, k, n_ref, tile, r0, r1)) break;
        const int64_t row0 = tile * 64;
        int h4 = 4 * h;
        asm volatile("" : "+v"(h4));
        bool ok[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) ok[q] = row0 + q * 32 + jl < nq;
        // each lane writes and later reads only its own LDS entries
        u32x4 lat[8 - kLat8Lds][2];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const u32x4 v = __builtin_nontemporal_load(cache + cache_chunk(tile, kb, q, lane));
                if (kb < kLat8Lds)
                    s_lat[wave][kb][q][lane] = v;
                else
                    lat[kb - kLat8Lds][q] = v;
            }
#pragma unroll 1
        for (int r = r0; r < r1; ++r) {
            // opaque per reference: LDS addresses are formed inside the loop
            asm volatile("" : "+v"(h4));
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const float *ref_h = &s_ref[r][0] + h4;
            const float clip = as.clip[2];
            i32x8 m8[2][2], d8[2][2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    quant_static([&](int o, int rr) {
                        const int j = 4 * kb + 2 * o + (rr >> 3), e = 4 * ((rr >> 2) & 1) + (rr & 3);
                        const uint32_t w2 = j < kLat8Lds ? s_lat[wave][j][q][ln][e >> 1]
                                                         : lat[j - kLat8Lds][q][e >> 1];
                        const float lv = (e & 1) ? bf_hi(w2) : bf_lo(w2);
                        const float rv = ref_h[64 * kb + 32 * o + 8 * (rr >> 2) + (rr & 3)];
                        return __builtin_amdgcn_fmed3f(lv * rv, -clip, clip);
                    }, as.s[2], m8[kb][q]);
            float part[2] = {0.f, 0.f};
            dense_layer_fp8<LAY_RELU, false>(nullptr, s_q[0], s_e[0], s_b[0], ref_h - h4, s_w6,
                                             unused16, m8, as.sbyte[2], d8, as.s[3], as.clip[3],
                                             part, nullptr, row0, ok, lane, h4);
            dense_layer_fp8<LAY_HEAD, false>(nullptr, s_q[1], s_e[1], s_b[1], ref_h - h4, s_w6,
                                             unused16, d8, as.sbyte[3], m8, 0.f, 0.f, part,
                                             nullptr, row0, ok, lane, h4);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float y = part[q] + __shfl_xor(part[q], 32, 64) + b6;
                if (h == 0 && ok[q]) out[(int64_t)r * ld_out + row0 + q * 32 + jl] = y;
            }
        }
    }
}

static InferArgs8 make_args8(const ndf_net_config *c, const QLayout &q, const char *Q, int e) {
    InferArgs8 a{};
    for (int l = 0; l < kL; ++l) a.grid[l] = (const uint16_t *)(Q + q.grid[e][l]);
    a.w1 = (const bf16x8 *)(Q + q.w1[e]);
    a.q[0] = (const i32x8 *)(Q + q.q2[e]);
    a.q[1] = (const i32x8 *)(Q + q.q3[e]);
    a.q[2] = (const i32x8 *)(Q + q.q4);
    a.q[3] = (const i32x8 *)(Q + q.q5);
    a.se[0] = (const int *)(Q + q.s2[e]);
    a.se[1] = (const int *)(Q + q.s3[e]);
    a.se[2] = (const int *)(Q + q.s4);
    a.se[3] = (const int *)(Q + q.s5);
    a.amax = (const int *)(Q + q.amax);
    a.b[0] = (const float *)(Q + q.b1[e]);
    a.b[1] = (const float *)(Q + q.b2[e]);
    a.b[2] = (const float *)(Q + q.b3[e]);
    a.b[3] = (const float *)(Q + q.b4);
    a.b[4] = (const float *)(Q + q.b5);
    a.w6 = (const float *)(Q + q.w6);
    a.b6 = (const float *)(Q + q.b6);
    a.g = grid_geom(c);
    a.fuse_ref = -1;
    return a;
}

static InferArgs make_args(const ndf_net_config *c, const QLayout &q, const char *Q, int e) {
    InferArgs a{};
    for (int l = 0; l < kL; ++l) a.grid[l] = (const uint16_t *)(Q + q.grid[e][l]);
    a.w[0] = (const bf16x8 *)(Q + q.w1[e]);
    a.w[1] = (const bf16x8 *)(Q + q.w2[e]);
    a.w[2] = (const bf16x8 *)(Q + q.w3[e]);
    a.w[3] = (const bf16x8 *)(Q + q.w4);
    a.w[4] = (const bf16x8 *)(Q + q.w5);
    a.b[0] = (const float *)(Q + q.b1[e]);
    a.b[1] = (const float *)(Q + q.b2[e]);
    a.b[2] = (const float *)(Q + q.b3[e]);
    a.b[3] = (const float *)(Q + q.b4);
    a.b[4] = (const float *)(Q + q.b5);
    a.w6 = (const float *)(Q + q.w6);
    a.b6 = (const float *)(Q + q.b6);
    a.g = grid_geom(c);
    a.V = (int64_t)c->nx * c->ny * c->nz;
    a.fuse_ref = -1;
    return a;
}

// Field arguments of the query encoder (the last one) with the reference vertex
// whose latent the kernel computes itself; with two encoders the reference
// encoder's (encoder 0's) grids and layers go along (SEP launches).
static InferArgs fused_args(const ndf_net_config *c, const QLayout &q, const char *Q,
                            int64_t ref) {
    InferArgs a = make_args(c, q, Q, c->n_enc - 1);
    a.fuse_ref = ref;
    if (c->n_enc == 2) {
        const InferArgs r = make_args(c, q, Q, 0);
        for (int l = 0; l < kL; ++l) a.rgrid[l] = r.grid[l];
        for (int i = 0; i < 3; ++i) {
            a.rw[i] = r.w[i];
            a.rb[i] = r.b[i];
        }
    }
    return a;
}

static bool any_hashed(const ndf_net_config *c) {
    for (int l = 0; l < kL; ++l)
        if (level_hashed(c, l)) return true;
    return false;
}

// Static activation scales of the E4M3 layers: the largest |input| of layers
// 2..5 over a fixed calibration set (kCalRefs references x kCalQueries
// queries spread evenly over the grid), run through the BF16 layers.
template <int MODE>
static void run_infer(const ndf_net_config *c, bool sep, dim3 g, const InferArgs &a,
                      const QueryList<MODE> &ql, int64_t nq, const float *rl, float *out,
                      const float *qpos, hipStream_t st);

static void launch_calibrate(const ndf_net_config *c, const QLayout &q, char *Q, hipStream_t st) {
    int *amax = (int *)(Q + q.amax);
    hipLaunchKernelGGL(zero_i32_kernel, dim3(1), dim3(64), 0, st, amax, 4);
    const InferArgs a = fused_args(c, q, Q, 0);
    const dim3 g(kCalRefs);
    run_infer<4>(c, c->n_enc == 2, g, a, {}, (int64_t)kCalQueries, nullptr, (float *)amax,
                 nullptr, st);
}

// Workgroups of a launch over nq queries, each for `refs` references that a tile can be
// split over: one per CU, and with little work one per tile (and reference), so that few
// tiles run on many CUs, though every workgroup then stages the weights (from L2) for one.
// Dealt eight to a workgroup's waves, 11803 vertices ran on 24 CUs: one BF16 field 17.4 ->
// 11.7 us, 16 of them 117 -> 46, 9 E4M3 cross fields 86 -> 45; no size measured slower.
static unsigned infer_blocks(int64_t nq, int refs = 1) {
    const int64_t items = ceil_div(nq, 64) * refs;
    return (unsigned)(items < 256 ? (items > 0 ? items : 1) : 256);
}

size_t net_latent_cache_bytes(const ndf_net_config *c) {
    const int64_t V = (int64_t)c->nx * c->ny * c->nz;
    return (size_t)ceil_div(V, 64) * 8 * 2 * 64 * 16;
}

// infer_kernel<MODE, ...> for the network's hashing, encoders (sep: a field mode
// whose reference latent comes from encoder 0) and input embedding.
template <int MODE>
static void run_infer(const ndf_net_config *c, bool sep, dim3 g, const InferArgs &a,
                      const QueryList<MODE> &ql, int64_t nq, const float *rl, float *out,
                      const float *qpos, hipStream_t st) {
    const dim3 b(kInferThreads);
    const bool hash = any_hashed(c);
#define NDF_IK(H, S, F) \
    hipLaunchKernelGGL((infer_kernel<MODE, H, S, false, F>), g, b, 0, st, a, ql, nq, rl, out, qpos)
    if (c->fourier) {
        if (hash) NDF_IK(true, false, true);
        else NDF_IK(false, false, true);
        return;
    }
    if constexpr (MODE == 0 || MODE == 3 || MODE == 4) {
        if (sep) {
            if (hash) NDF_IK(true, true, false);
            else NDF_IK(false, true, false);
            return;
        }
    }
    if (hash) NDF_IK(true, false, false);
    else NDF_IK(false, false, false);
#undef NDF_IK
}

template <int MODE>
static void run_infer8(const ndf_net_config *c, dim3 g, const InferArgs8 &a,
                       const QueryList<MODE> &ql, int64_t nq, const float *rl, float *out,
                       const float *qpos, hipStream_t st) {
    const dim3 b(kInferThreads);
    const bool hash = any_hashed(c);
#define NDF_IK8(H, F) \
    hipLaunchKernelGGL((infer_fp8_kernel<MODE, H, F>), g, b, 0, st, a, ql, nq, rl, out, qpos)
    if (c->fourier) {
        if (hash) NDF_IK8(true, true);
        else NDF_IK8(false, true);
    } else {
        if (hash) NDF_IK8(true, false);
        else NDF_IK8(false, false);
    }
#undef NDF_IK8
}

int launch_infer_latents(const ndf_net_config *c, const void *qp, void *cache, hipStream_t st) {
    const QLayout q = qlayout(c);
    const InferArgs a = make_args(c, q, (const char *)qp, c->n_enc - 1);
    run_infer<2>(c, false, dim3(infer_blocks(a.V)), a, {}, a.V, nullptr, (float *)cache,
                 nullptr, st);
    return status_of_launch();
}

// Fields of n_ref references (latents lat[n_ref][128]) from the query-latent
// cache, kMultiRefs per launch.
static void decode_cached(const ndf_net_config *c, const QLayout &q, const char *Q,
                          const void *cache, const float *lat, int n_ref, float *out,
                          hipStream_t st) {
    const InferArgs a1 = make_args(c, q, Q, c->n_enc - 1);
    for (int r0 = 0; r0 < n_ref; r0 += kMultiRefs) {
        const int n = n_ref - r0 < kMultiRefs ? n_ref - r0 : kMultiRefs;
        hipLaunchKernelGGL(infer_cached_kernel<false>, dim3(infer_blocks(a1.V, n)),
                           dim3(kInferThreads), 0, st, a1, (const u32x4 *)cache, a1.V,
                           lat + (int64_t)r0 * kH, n, out + (int64_t)r0 * a1.V, a1.V);
    }
}

// Reference latents lat[n_ref][128] of the vertices ref_v[n_ref] (host) with encoder 0:
// run(list, count, latents) per kLatRefs of them.
template <typename F>
static void each_ref_list(const int64_t *ref_v, int n_ref, float *lat, F run) {
    for (int r0 = 0; r0 < n_ref; r0 += kLatRefs) {
        const int n = n_ref - r0 < kLatRefs ? n_ref - r0 : kLatRefs;
        RefVerts list{};
        for (int i = 0; i < n; ++i) list.v[i] = ref_v[r0 + i];
        run(list, n, lat + (int64_t)r0 * kH);
    }
}

static void ref_latents(const ndf_net_config *c, const QLayout &q, const char *Q,
                        const int64_t *ref_v, int n_ref, float *lat, hipStream_t st) {
    const InferArgs a0 = make_args(c, q, Q, 0);
    each_ref_list(ref_v, n_ref, lat, [&](const RefVerts &list, int n, float *l) {
        run_infer<1>(c, false, dim3(infer_blocks(n)), a0, list, (int64_t)n, nullptr, l, nullptr, st);
    });
}

static void ref_latents8(const ndf_net_config *c, const QLayout &q, const char *Q,
                         const int64_t *ref_v, int n_ref, float *lat, hipStream_t st) {
    const InferArgs8 a0 = make_args8(c, q, Q, 0);
    each_ref_list(ref_v, n_ref, lat, [&](const RefVerts &list, int n, float *l) {
        run_infer8<1>(c, dim3(infer_blocks(n)), a0, list, (int64_t)n, nullptr, l, nullptr, st);
    });
}

int launch_infer_field_cached(const ndf_net_config *c, const void *qp, const int64_t *ref_v,
                              int n_ref, const void *cache, float *out, void *ws, hipStream_t st) {
    const QLayout q = qlayout(c);
    const char *Q = (const char *)qp;
    float *lat = (float *)ws;
    ref_latents(c, q, Q, ref_v, n_ref, lat, st);
    decode_cached(c, q, Q, cache, lat, n_ref, out, st);
    return status_of_launch();
}

int launch_infer_field(const ndf_net_config *c, const void *qp, int prec, const int64_t *ref_v,
                       int n_ref, float *out, void *ws, hipStream_t st) {
    const bool hash = any_hashed(c);
    if (prec != NDF_PREC_BF16 && prec != NDF_PREC_FP8_E4M3) return NDF_E_UNSUPPORTED;
    const QLayout q = qlayout(c);
    const char *Q = (const char *)qp;
    float *lat = (float *)ws;
    const int64_t V = (int64_t)c->nx * c->ny * c->nz;
    if (prec == NDF_PREC_FP8_E4M3 && n_ref >= 2 && !c->grid_only) {
        // the BF16 query latents once into the workspace, then every reference's
        // decoder in E4M3, kMultiRefs references per pass over the cache
        void *cache = (char *)ws + net_infer_lat_ws_bytes(n_ref);
        ref_latents(c, q, Q, ref_v, n_ref, lat, st);
        if (launch_infer_latents(c, qp, cache, st) != NDF_OK) return NDF_E_HIP;
        const InferArgs8 a8 = make_args8(c, q, Q, c->n_enc - 1);
        for (int r0 = 0; r0 < n_ref; r0 += kMultiRefs) {
            const int n = n_ref - r0 < kMultiRefs ? n_ref - r0 : kMultiRefs;
            hipLaunchKernelGGL(infer_cached_fp8_kernel, dim3(infer_blocks(V, n)),
                               dim3(kInferThreads), 0, st, a8, (const u32x4 *)cache, V,
                               lat + (int64_t)r0 * kH, n, out + (int64_t)r0 * V, V);
        }
        return status_of_launch();
    }
    if (prec == NDF_PREC_FP8_E4M3 && c->n_enc == 1) {
        // shared encoder: each workgroup computes the reference latent itself
        InferArgs8 a = make_args8(c, q, Q, 0);
        for (int r = 0; r < n_ref; ++r) {
            a.fuse_ref = ref_v[r];
            run_infer8<0>(c, dim3(infer_blocks(V)), a, {}, V, nullptr, out + (int64_t)r * V,
                          nullptr, st);
        }
        return status_of_launch();
    }
    if (c->grid_only) {
        // grid-only network: one fused pass per reference (BF16; the reference's
        // grid features gathered in each workgroup's prologue)
        if (prec != NDF_PREC_BF16) return NDF_E_UNSUPPORTED;
        const bool sep = c->n_enc == 2;
        for (int r = 0; r < n_ref; ++r) {
            const InferArgs a = fused_args(c, q, Q, ref_v[r]);
            const dim3 g(infer_blocks(a.V)), b(kInferThreads);
            float *o = out + (int64_t)r * a.V;
#define NDF_GO_FIELD(H, S) \
    hipLaunchKernelGGL((infer_kernel<0, H, S, true>), g, b, 0, st, a, NoVerts{}, a.V, nullptr, o, nullptr)
            if (hash && sep) NDF_GO_FIELD(true, true);
            else if (hash) NDF_GO_FIELD(true, false);
            else if (sep) NDF_GO_FIELD(false, true);
            else NDF_GO_FIELD(false, false);
#undef NDF_GO_FIELD
        }
        return status_of_launch();
    }
    if (prec == NDF_PREC_BF16 && n_ref >= 2) {
        // the query latents once into the workspace, then every reference decoded
        // from them, kMultiRefs references per pass over the cache (bit for bit
        // the fused single-reference field)
        void *cache = (char *)ws + net_infer_lat_ws_bytes(n_ref);
        ref_latents(c, q, Q, ref_v, n_ref, lat, st);
        if (launch_infer_latents(c, qp, cache, st) != NDF_OK) return NDF_E_HIP;
        decode_cached(c, q, Q, cache, lat, n_ref, out, st);
        return status_of_launch();
    }
    if (prec == NDF_PREC_BF16) {
        // each workgroup computes the reference latent itself (SEP: with encoder 0)
        const bool sep = c->n_enc == 2;
        for (int r = 0; r < n_ref; ++r) {
            const InferArgs a = fused_args(c, q, Q, ref_v[r]);
            run_infer<0>(c, sep, dim3(infer_blocks(a.V)), a, {}, a.V, nullptr,
                         out + (int64_t)r * a.V, nullptr, st);
        }
        return status_of_launch();
    }
    // FP8 with two encoders: reference latents with encoder 0 (p1), then one pass
    // per reference with the query encoder (p2)
    ref_latents8(c, q, Q, ref_v, n_ref, lat, st);
    const InferArgs8 a1 = make_args8(c, q, Q, c->n_enc - 1);
    for (int r = 0; r < n_ref; ++r)
        run_infer8<0>(c, dim3(infer_blocks(V)), a1, {}, V, lat + (int64_t)r * kH,
                      out + (int64_t)r * V, nullptr, st);
    return status_of_launch();
}

int launch_infer_points(const ndf_net_config *c, const void *qp, int prec, const int64_t *ref_v,
                        int n_ref, const float *pos, int64_t n, float *out, void *ws,
                        hipStream_t st) {
    const bool hash = any_hashed(c);
    if (prec != NDF_PREC_BF16 && prec != NDF_PREC_FP8_E4M3) return NDF_E_UNSUPPORTED;
    const QLayout q = qlayout(c);
    const char *Q = (const char *)qp;
    float *lat = (float *)ws;
    if (c->grid_only) {  // BF16, one fused pass per reference
        if (prec != NDF_PREC_BF16) return NDF_E_UNSUPPORTED;
        const bool sep = c->n_enc == 2;
        for (int r = 0; r < n_ref; ++r) {
            const InferArgs a = fused_args(c, q, Q, ref_v[r]);
            const dim3 g(infer_blocks(n)), b(kInferThreads);
            float *o = out + (int64_t)r * n;
#define NDF_GO_POINTS(H, S) \
    hipLaunchKernelGGL((infer_kernel<3, H, S, true>), g, b, 0, st, a, NoVerts{}, n, nullptr, o, pos)
            if (hash && sep) NDF_GO_POINTS(true, true);
            else if (hash) NDF_GO_POINTS(true, false);
            else if (sep) NDF_GO_POINTS(false, true);
            else NDF_GO_POINTS(false, false);
#undef NDF_GO_POINTS
        }
        return status_of_launch();
    }
    if (c->n_enc == 1) {  // shared encoder: the reference latent in each workgroup
        if (prec == NDF_PREC_FP8_E4M3) {
            InferArgs8 a = make_args8(c, q, Q, 0);
            for (int r = 0; r < n_ref; ++r) {
                a.fuse_ref = ref_v[r];
                run_infer8<3>(c, dim3(infer_blocks(n)), a, {}, n, nullptr,
                              out + (int64_t)r * n, pos, st);
            }
        } else {
            for (int r = 0; r < n_ref; ++r) {
                const InferArgs a = fused_args(c, q, Q, ref_v[r]);
                run_infer<3>(c, false, dim3(infer_blocks(n)), a, {}, n, nullptr,
                             out + (int64_t)r * n, pos, st);
            }
        }
        return status_of_launch();
    }
    if (prec == NDF_PREC_FP8_E4M3) {
        ref_latents8(c, q, Q, ref_v, n_ref, lat, st);
        const InferArgs8 a1 = make_args8(c, q, Q, c->n_enc - 1);
        for (int r = 0; r < n_ref; ++r)
            run_infer8<3>(c, dim3(infer_blocks(n)), a1, {}, n, lat + (int64_t)r * kH,
                          out + (int64_t)r * n, pos, st);
        return status_of_launch();
    }
    ref_latents(c, q, Q, ref_v, n_ref, lat, st);
    const InferArgs a1 = make_args(c, q, Q, c->n_enc - 1);
    for (int r = 0; r < n_ref; ++r)
        run_infer<3>(c, false, dim3(infer_blocks(n)), a1, {}, n, lat + (int64_t)r * kH,
                     out + (int64_t)r * n, pos, st);
    return status_of_launch();
}

int launch_infer_difference(const ndf_net_config *c, const void *qp, int64_t ref_a, int64_t ref_b,
                            const void *cache, float *out, void *ws, hipStream_t st) {
    const QLayout q = qlayout(c);
    const char *Q = (const char *)qp;
    float *lat = (float *)ws;
    const int64_t both[2] = {ref_a, ref_b};
    ref_latents(c, q, Q, both, 2, lat, st);
    const InferArgs a1 = make_args(c, q, Q, c->n_enc - 1);
    hipLaunchKernelGGL(infer_cached_kernel<true>, dim3(infer_blocks(a1.V)), dim3(kInferThreads), 0,
                       st, a1, (const u32x4 *)cache, a1.V, lat, 2, out, a1.V);
    return status_of_launch();
}

}  // namespace ndf
