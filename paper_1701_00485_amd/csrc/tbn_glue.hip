// tbn_glue.hip -- the layers the workloads put around the two-bit convolutions
// (Sec. 4 uses ResNet-18 with batch normalisation; the smaller workloads add max pooling,
// ReLU and a softmax cross-entropy loss).  All HBM-bound, NHWC bf16 activations.
//   * max pooling forward (argmax kept for the backward pass; ties go to the first
//     maximum in row-major window order) and backward (gather, deterministic);
//   * global average pooling;
//   * batch normalisation in training form (batch statistics) forward and backward,
//     with ReLU fused on both sides;
//   * softmax cross-entropy over fp32 logits (loss and gradient).
#include <type_traits>

#include "tbn_device.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

__device__ __forceinline__ void st_act(void* p, int64_t i, float v, int f32) {
    if (f32)
        reinterpret_cast<float*>(p)[i] = v;
    else
        reinterpret_cast<uint16_t*>(p)[i] = (uint16_t)f32_to_bf16_bits(v);
}

// Element index -> (image, row, column, channel) of an N x H x W x C tensor: by 32-bit multiply-shift
// divisions where it has fewer than 2^31 elements, else by 64-bit ones (which took most of the time
// of the kernels of one channel per thread).
struct PoolSplit {
    FastDiv c, w, h;
    int32_t C, W, H, small;
};

PoolSplit make_pool_split(int64_t N, int32_t H, int32_t W, int32_t C) {
    return {make_fastdiv((uint32_t)C), make_fastdiv((uint32_t)W), make_fastdiv((uint32_t)H), C, W, H,
            N * H * W * C < 0x7FFFFFFFll};
}

__device__ __forceinline__ void split_index(const PoolSplit& s, int64_t i, int64_t* n, int* h, int* w, int* c) {
    if (s.small) {
        const uint32_t pix = fdiv((uint32_t)i, s.c), row = fdiv(pix, s.w), img = fdiv(row, s.h);
        *c = (int)((uint32_t)i - pix * (uint32_t)s.C);
        *w = (int)(pix - row * (uint32_t)s.W);
        *h = (int)(row - img * (uint32_t)s.H);
        *n = img;
    } else {
        const int64_t pix = i / s.C, row = pix / s.W;
        *c = (int)(i - pix * s.C);
        *w = (int)(pix - row * s.W);
        *n = row / s.H;
        *h = (int)(row - *n * s.H);
    }
}

// NV channels per thread (8 = one 16-byte access when C % 8 == 0).  bf16 values compare
// as their fp32 widening; ties keep the first window position in row-major order.
template <int NV>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const PoolArgs a, const PoolSplit s,
                                                          const uint16_t* __restrict__ x, uint16_t* __restrict__ y,
                                                          int32_t* __restrict__ arg) {
    const int64_t total = (int64_t)a.N * a.P * a.Q * a.C;
    const int64_t o = ((int64_t)blockIdx.x * 256 + threadIdx.x) * NV;
    if (o >= total) return;
    int64_t n;
    int p, q, c;
    split_index(s, o, &n, &p, &q, &c);
    float best[NV];
    int bi[NV];
#pragma unroll
    for (int e = 0; e < NV; ++e) {
        best[e] = 0.0f;
        bi[e] = -1;
    }
    for (int r = 0; r < a.k; ++r) {
        const int h = p * a.s - a.pad + r;
        if ((unsigned)h >= (unsigned)a.H) continue;
        for (int t = 0; t < a.k; ++t) {
            const int w = q * a.s - a.pad + t;
            if ((unsigned)w >= (unsigned)a.W) continue;
            const int64_t xi = ((n * a.H + h) * a.W + w) * a.C + c;
            uint32_t b[NV];
            if constexpr (NV == 8) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(x + xi);
#pragma unroll
                for (int e = 0; e < 8; ++e) b[e] = (e & 1) ? (v[e / 2] >> 16) : (v[e / 2] & 0xFFFFu);
            } else {
                b[0] = x[xi];
            }
#pragma unroll
            for (int e = 0; e < NV; ++e) {
                const float v = bf16_bits_to_f32(b[e]);
                if (bi[e] < 0 || v > best[e]) {
                    best[e] = v;
                    bi[e] = h * a.W + w;
                }
            }
        }
    }
    // exact: each maximum is a bf16 value
    if constexpr (NV == 8) {
        *reinterpret_cast<u32x4*>(y + o) = u32x4{pack_bf16x2(best[0], best[1]), pack_bf16x2(best[2], best[3]),
                                                  pack_bf16x2(best[4], best[5]), pack_bf16x2(best[6], best[7])};
        if (arg) {
            *reinterpret_cast<u32x4*>(arg + o) = u32x4{(uint32_t)bi[0], (uint32_t)bi[1], (uint32_t)bi[2], (uint32_t)bi[3]};
            *reinterpret_cast<u32x4*>(arg + o + 4) =
                u32x4{(uint32_t)bi[4], (uint32_t)bi[5], (uint32_t)bi[6], (uint32_t)bi[7]};
        }
    } else {
        y[o] = (uint16_t)f32_to_bf16_bits(best[0]);
        if (arg) arg[o] = bi[0];
    }
}

// The same for a compile-time K x K window, 8 channels per thread (C % 8 == 0) and 32-bit
// indices (the host checks the sizes): the K*K 16-byte loads of a thread are all issued
// before the first comparison, and the pixel index is split with multiply-shift divisions.
template <int K>
__global__ __launch_bounds__(256) void maxpool_fwd8_kernel(const PoolArgs a, const FastDiv div_g, const FastDiv div_q,
                                                           const FastDiv div_p, const uint32_t groups,
                                                           const uint16_t* __restrict__ x, uint16_t* __restrict__ y,
                                                           int32_t* __restrict__ arg) {
    const uint32_t gi = blockIdx.x * 256u + threadIdx.x;  // (output pixel, 8-channel group)
    if (gi >= groups) return;
    const uint32_t pix = fdiv(gi, div_g);
    const uint32_t c = (gi - pix * (uint32_t)(a.C / 8)) * 8u;
    const uint32_t nq = fdiv(pix, div_q);
    const int q = (int)(pix - nq * (uint32_t)a.Q);
    const uint32_t n = fdiv(nq, div_p);
    const int p = (int)(nq - n * (uint32_t)a.P);
    const int h0 = p * a.s - a.pad, w0 = q * a.s - a.pad;
    u32x4 v[K * K];
    bool ok[K * K];
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int h = h0 + r, w = w0 + t;
            ok[r * K + t] = (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
            const uint32_t xi = (((n * (uint32_t)a.H + (uint32_t)h) * (uint32_t)a.W + (uint32_t)w) * (uint32_t)a.C + c);
            v[r * K + t] = ok[r * K + t] ? *reinterpret_cast<const u32x4*>(x + xi) : u32x4{0u, 0u, 0u, 0u};
        }
    float best[8];
    int bi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        best[e] = 0.0f;
        bi[e] = -1;
    }
#pragma unroll
    for (int j = 0; j < K * K; ++j) {
        if (!ok[j]) continue;
        const int pos = (h0 + j / K) * a.W + (w0 + j % K);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float f = bf16_bits_to_f32((e & 1) ? (v[j][e / 2] >> 16) : (v[j][e / 2] & 0xFFFFu));
            if (bi[e] < 0 || f > best[e]) {
                best[e] = f;
                bi[e] = pos;
            }
        }
    }
    const uint32_t o = gi * 8u;
    *reinterpret_cast<u32x4*>(y + o) = u32x4{pack_bf16x2(best[0], best[1]), pack_bf16x2(best[2], best[3]),
                                              pack_bf16x2(best[4], best[5]), pack_bf16x2(best[6], best[7])};
    if (arg) {
        *reinterpret_cast<u32x4*>(arg + o) = u32x4{(uint32_t)bi[0], (uint32_t)bi[1], (uint32_t)bi[2], (uint32_t)bi[3]};
        *reinterpret_cast<u32x4*>(arg + o + 4) = u32x4{(uint32_t)bi[4], (uint32_t)bi[5], (uint32_t)bi[6], (uint32_t)bi[7]};
    }
}

// dx[n,h,w,c] = sum of dy over the windows that chose (h, w); NV channels per thread
template <int NV>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const PoolArgs a, const PoolSplit s,
                                                          const uint16_t* __restrict__ dy,
                                                          const int32_t* __restrict__ arg, void* __restrict__ dx,
                                                          int dx_f32) {
    const int64_t total = (int64_t)a.N * a.H * a.W * a.C;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * NV;
    if (i >= total) return;
    int64_t n;
    int h, w, c;
    split_index(s, i, &n, &h, &w, &c);
    const int me = h * a.W + w;
    // windows p with p*s - pad <= h <= p*s - pad + k - 1
    const int p_lo = max(0, (h + a.pad - a.k + a.s) / a.s), p_hi = min(a.P - 1, (h + a.pad) / a.s);
    const int q_lo = max(0, (w + a.pad - a.k + a.s) / a.s), q_hi = min(a.Q - 1, (w + a.pad) / a.s);
    float acc[NV];
#pragma unroll
    for (int e = 0; e < NV; ++e) acc[e] = 0.0f;
    for (int p = p_lo; p <= p_hi; ++p)
        for (int q = q_lo; q <= q_hi; ++q) {
            const int64_t o = ((n * a.P + p) * a.Q + q) * a.C + c;
            if constexpr (NV == 8) {
                const u32x4 a0 = *reinterpret_cast<const u32x4*>(arg + o);
                const u32x4 a1 = *reinterpret_cast<const u32x4*>(arg + o + 4);
                const u32x4 d = *reinterpret_cast<const u32x4*>(dy + o);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t ae = e < 4 ? a0[e] : a1[e - 4];
                    const uint32_t db = (e & 1) ? (d[e / 2] >> 16) : (d[e / 2] & 0xFFFFu);
                    if ((int)ae == me) acc[e] += bf16_bits_to_f32(db);
                }
            } else {
                if (arg[o] == me) acc[0] += bf16_bits_to_f32(dy[o]);
            }
        }
    if constexpr (NV == 8) {
        if (dx_f32) {
            float* dp = reinterpret_cast<float*>(dx) + i;
            *reinterpret_cast<f32x4*>(dp) = f32x4{acc[0], acc[1], acc[2], acc[3]};
            *reinterpret_cast<f32x4*>(dp + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
        } else {
            *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(dx) + i) =
                u32x4{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]), pack_bf16x2(acc[4], acc[5]),
                      pack_bf16x2(acc[6], acc[7])};
        }
    } else {
        st_act(dx, i, acc[0], dx_f32);
    }
}

// The same gather over 8-channel groups with 32-bit multiply-shift index splits (sizes below
// 2^31): the kernel above spends most of its instructions on 64-bit divisions.
__global__ __launch_bounds__(256) void maxpool_bwd8_kernel(const PoolArgs a, const FastDiv div_g, const FastDiv div_w,
                                                           const FastDiv div_h, const uint32_t groups,
                                                           const uint16_t* __restrict__ dy,
                                                           const int32_t* __restrict__ arg, void* __restrict__ dx,
                                                           int dx_f32) {
    const uint32_t gi = blockIdx.x * 256u + threadIdx.x;  // (input pixel, 8-channel group)
    if (gi >= groups) return;
    const uint32_t pix = fdiv(gi, div_g);
    const uint32_t c = (gi - pix * (uint32_t)(a.C / 8)) * 8u;
    const uint32_t nh = fdiv(pix, div_w);
    const int w = (int)(pix - nh * (uint32_t)a.W);
    const uint32_t n = fdiv(nh, div_h);
    const int h = (int)(nh - n * (uint32_t)a.H);
    const int me = h * a.W + w;
    const int p_lo = max(0, (h + a.pad - a.k + a.s) / a.s), p_hi = min(a.P - 1, (h + a.pad) / a.s);
    const int q_lo = max(0, (w + a.pad - a.k + a.s) / a.s), q_hi = min(a.Q - 1, (w + a.pad) / a.s);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    for (int p = p_lo; p <= p_hi; ++p)
        for (int q = q_lo; q <= q_hi; ++q) {
            const uint32_t o = ((n * (uint32_t)a.P + (uint32_t)p) * (uint32_t)a.Q + (uint32_t)q) * (uint32_t)a.C + c;
            const u32x4 a0 = *reinterpret_cast<const u32x4*>(arg + o);
            const u32x4 a1 = *reinterpret_cast<const u32x4*>(arg + o + 4);
            const u32x4 d = *reinterpret_cast<const u32x4*>(dy + o);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t ae = e < 4 ? a0[e] : a1[e - 4];
                const uint32_t db = (e & 1) ? (d[e / 2] >> 16) : (d[e / 2] & 0xFFFFu);
                if ((int)ae == me) acc[e] += bf16_bits_to_f32(db);
            }
        }
    const uint32_t i = gi * 8u;
    if (dx_f32) {
        float* dp = reinterpret_cast<float*>(dx) + i;
        *reinterpret_cast<f32x4*>(dp) = f32x4{acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<f32x4*>(dp + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
    } else {
        *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(dx) + i) =
            u32x4{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]), pack_bf16x2(acc[4], acc[5]),
                  pack_bf16x2(acc[6], acc[7])};
    }
}

// Windows that do not overlap (k = stride, no padding): a thread takes one window's argmax and gradient
// (8 channels) and writes its k x k inputs, where the gather above reads them k x k times (32 x 32 x 128 at
// batch 128: 15.2 -> 10.2 us).  The grid covers the input in cells of k x k; cells cut off by its edge
// and cells past the last window write zeros.
template <int KW>
__global__ __launch_bounds__(256) void maxpool_bwd_cells_kernel(const PoolArgs a, const FastDiv div_g, const FastDiv div_q,
                                                                const FastDiv div_p, const uint32_t cells_p,
                                                                const uint32_t cells_q, const uint32_t groups,
                                                                const uint16_t* __restrict__ dy,
                                                                const int32_t* __restrict__ arg, void* __restrict__ dx,
                                                                int dx_f32) {
    const uint32_t gi = blockIdx.x * 256u + threadIdx.x;  // (cell, 8-channel group)
    if (gi >= groups) return;
    const uint32_t cell = fdiv(gi, div_g);
    const uint32_t c = (gi - cell * (uint32_t)(a.C / 8)) * 8u;
    const uint32_t np = fdiv(cell, div_q);
    const uint32_t q = cell - np * cells_q;
    const uint32_t n = fdiv(np, div_p);
    const uint32_t p = np - n * cells_p;
    u32x4 a0 = {~0u, ~0u, ~0u, ~0u}, a1 = a0, d = {0u, 0u, 0u, 0u};
    if (p < (uint32_t)a.P && q < (uint32_t)a.Q) {
        const uint32_t o = ((n * (uint32_t)a.P + p) * (uint32_t)a.Q + q) * (uint32_t)a.C + c;
        a0 = *reinterpret_cast<const u32x4*>(arg + o);
        a1 = *reinterpret_cast<const u32x4*>(arg + o + 4);
        d = *reinterpret_cast<const u32x4*>(dy + o);
    }
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int j = 0; j < KW; ++j) {
            const uint32_t h = p * KW + i, w = q * KW + j;
            if (h >= (uint32_t)a.H || w >= (uint32_t)a.W) continue;
            const uint32_t me = h * (uint32_t)a.W + w;
            const uint32_t o = ((n * (uint32_t)a.H + h) * (uint32_t)a.W + w) * (uint32_t)a.C + c;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t ae = e < 4 ? a0[e] : a1[e - 4];
                const uint32_t db = (e & 1) ? (d[e / 2] >> 16) : (d[e / 2] & 0xFFFFu);
                v[e] = ae == me ? 0.0f + bf16_bits_to_f32(db) : 0.0f;
            }
            if (dx_f32) {
                float* dp = reinterpret_cast<float*>(dx) + o;
                *reinterpret_cast<f32x4*>(dp) = f32x4{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<f32x4*>(dp + 4) = f32x4{v[4], v[5], v[6], v[7]};
            } else {
                *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(dx) + o) =
                    u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                          pack_bf16x2(v[6], v[7])};
            }
        }
}

// y[n][c] = mean over h, w of x[n][h][w][c]; one thread per (n, c)
__global__ __launch_bounds__(256) void avgpool_kernel(int32_t N, int32_t HW, int32_t C, const uint16_t* __restrict__ x,
                                                      void* __restrict__ y, int y_f32) {
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= (int64_t)N * C) return;
    const int c = (int)(o % C);
    const int64_t n = o / C;
    float acc = 0.0f;
    for (int i = 0; i < HW; ++i) acc += bf16_bits_to_f32(x[(n * HW + i) * C + c]);
    st_act(y, o, acc / (float)HW, y_f32);
}

// C % 8 == 0: eight lanes per group of 8 channels of one image; lane j sums positions
// j, j + 8, ... with 16-byte loads, then the eight partial sums are combined by a fixed
// butterfly (the result does not depend on scheduling).
__global__ __launch_bounds__(256) void avgpool8_kernel(int32_t N, int32_t HW, int32_t C, const uint16_t* __restrict__ x,
                                                       void* __restrict__ y, int y_f32) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t grp = t >> 3;  // (n, channel group), N * C / 8 of them
    const int j = (int)(t & 7);
    const int G = C / 8;
    const bool ok = grp < (int64_t)N * G;
    const int64_t n = ok ? grp / G : 0;
    const int c0 = ok ? (int)(grp - n * G) * 8 : 0;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (ok) {
        for (int i = j; i < HW; i += 8) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(x + (n * HW + i) * C + c0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[2 * e] += bf16_bits_to_f32(v[e] & 0xFFFFu);
                acc[2 * e + 1] += bf16_bits_to_f32(v[e] >> 16);
            }
        }
    }
    // every lane of the wave takes part in the shuffles (groups of 8 lanes never straddle
    // a wave; lanes past the end carry zeros)
#pragma unroll
    for (int m = 1; m < 8; m <<= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], m, 8);
    if (!ok || j != 0) return;
    const float inv = 1.0f / (float)HW;
    const int64_t o = n * C + c0;
    if (y_f32) {
        float* yp = reinterpret_cast<float*>(y) + o;
        *reinterpret_cast<f32x4*>(yp) = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
        *reinterpret_cast<f32x4*>(yp + 4) = f32x4{acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv};
    } else {
        *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(y) + o) =
            u32x4{pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv),
                  pack_bf16x2(acc[4] * inv, acc[5] * inv), pack_bf16x2(acc[6] * inv, acc[7] * inv)};
    }
}

// ---- batch normalisation, training form ----
// Per-channel sums over rows = N*H*W in two deterministic levels:
//   * partial: block (b, slice) sums a chunk of rows for up to 256 groups of 8 channels (one 16-byte
//     load per row each); the 256 threads cover tpr = 256 / groups rows at a time, four such steps'
//     loads issued together, then combine their row lanes through LDS in a fixed order and write
//     partial[b][c];
//   * finalize: 16 or 64 threads per channel add partial[0..chunks)[c] in a fixed order.
// Then the element-wise passes, with the same thread layout, so that a thread keeps the factors of
// its 8 channels in registers over its rows.  (A thread per 16 bytes, loading them for every 8 values,
// issued three to ten loads of factors per load of data: 28.5 us for the backward pass over 131072 x 128
// against 21.0, 14.4 for the forward pass against 11.1.)  Small tensors take one row a thread, for more blocks.
//
// C % 8 != 0 (up to 256 channels, large tensors): eight consecutive rows are C groups of 8 values whose channels
// (8 g + e) % C repeat every eight rows, so the same code runs over "rows" of 8 C values (FLAT); the last
// rows % 8 rows are added value by value.  Other uneven channel counts take one channel per thread.
// Modes: BN_STATS sums d and d^2 with d = x - x[0][c] (one pass for both statistics: the
// first row's value of each channel is a shift common to every chunk, so the chunk sums
// add, and the variance S2/n - (S1/n)^2 of the shifted values does not cancel against a
// large mean); BN_BWD sums g and g * xhat, with g = dy masked by y > 0 when ReLU followed
// the normalisation.
enum { BN_BWD = 2, BN_STATS = 3 };
enum { BN_VEC = 0, BN_FLAT = 1, BN_SCALAR = 2 };

template <int NV>
__device__ __forceinline__ void load_values(const uint16_t* __restrict__ p, float (&v)[NV]) {
    if constexpr (NV == 8) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = bf16_bits_to_f32(w[e] & 0xFFFFu);
            v[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
        }
    } else {
        v[0] = bf16_bits_to_f32(*p);
    }
}

// Thread layout of a pass over rows of `width` values (C, or 8 C with FLAT): NV values per thread.
template <int KIND>
struct BnLane {
    static constexpr int NV = KIND == BN_SCALAR ? 1 : 8;
    int Gs, tpr, r0, g;  // groups of this slice, rows per step, this thread's row and group
    int64_t col;         // its first value in the row
    int width, base;     // ... and that value's channel (FLAT)
    bool active;
    __device__ BnLane(int32_t C) {
        width = KIND == BN_FLAT ? 8 * C : C;
        const int G = width / NV, gbase = (int)blockIdx.y * 256;
        Gs = min(256, G - gbase);
        tpr = 256 / Gs;
        r0 = (int)threadIdx.x / Gs;
        g = (int)threadIdx.x - r0 * Gs;
        active = r0 < tpr;
        col = (int64_t)(gbase + g) * NV;
        base = KIND == BN_FLAT ? (int)((uint32_t)col % (uint32_t)C) : 0;
    }
    __device__ int channel(int e, int32_t C) const {
        if (KIND != BN_FLAT) return (int)col + e;
        int c = base + e;
        while (c >= C) c -= C;  // once at most from 8 channels on
        return c;
    }
};

// The factors of a thread's NV channels in the element-wise passes: f[j][e] = src[j][channel e].  FLAT: through
// LDS, as a thread's channels follow no vector load and 32 to 40 gathered loads of 4 bytes bound the pass
// (10039 x 252: 10.9 and 14.6 us forward and backward with them).  All threads of the block call it.
template <int KIND, int NF>
__device__ __forceinline__ void bn_factors(const BnLane<KIND>& l, int32_t C, const float* const (&src)[NF],
                                           float (&f)[NF][BnLane<KIND>::NV]) {
    if constexpr (KIND == BN_FLAT) {
        constexpr int PITCH = 33;  // channel c at 33 (c % 8) + c / 8: neighbours' channels, 8 apart, in different banks
        __shared__ float sh[NF][8 * PITCH];
        if ((int)threadIdx.x < C)
#pragma unroll
            for (int j = 0; j < NF; ++j) sh[j][(threadIdx.x & 7) * PITCH + (threadIdx.x >> 3)] = src[j][threadIdx.x];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = l.channel(e, C);
#pragma unroll
            for (int j = 0; j < NF; ++j) f[j][e] = sh[j][(c & 7) * PITCH + (c >> 3)];
        }
    } else if (l.active) {
#pragma unroll
        for (int e = 0; e < BnLane<KIND>::NV; ++e)
#pragma unroll
            for (int j = 0; j < NF; ++j) f[j][e] = src[j][l.channel(e, C)];
    }
}

template <int MODE, int KIND>
__global__ __launch_bounds__(256) void bn_partial_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ y,
                                                         const uint16_t* __restrict__ dy, int64_t rows, int32_t C,
                                                         int64_t rpc, int relu, const float* __restrict__ mean,
                                                         const float* __restrict__ inv_std, float* __restrict__ p1,
                                                         float* __restrict__ p2) {
    using Lane = BnLane<KIND>;
    constexpr int NV = Lane::NV;
    constexpr int UN = 4;  // steps whose loads are issued together
    __shared__ float s1[256 * NV], s2[256 * NV];
    const Lane l(C);
    const int64_t srows = KIND == BN_FLAT ? rows / 8 : rows;
    const int64_t rbeg = (int64_t)blockIdx.x * rpc;
    const int64_t rend = min(srows, rbeg + rpc);
    float a1[NV], a2[NV], m[NV], is[NV];
#pragma unroll
    for (int e = 0; e < NV; ++e) {
        const int c = l.channel(e, C);
        a1[e] = a2[e] = 0.0f;
        m[e] = MODE == BN_BWD ? mean[c] : bf16_bits_to_f32(x[c]);  // BN_STATS: the shift, row 0
        is[e] = MODE == BN_BWD ? inv_std[c] : 0.0f;
    }
    auto add = [&](const float (&xv)[NV], const float (&dv)[NV], const float (&yv)[NV]) {
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            if constexpr (MODE == BN_STATS) {
                const float d = xv[e] - m[e];
                a1[e] += d;
                a2[e] += d * d;
            } else {
                const float gv = (relu && !(yv[e] > 0.0f)) ? 0.0f : dv[e];
                a1[e] += gv;
                a2[e] += gv * (xv[e] - m[e]) * is[e];
            }
        }
    };
    if (l.active) {
        int64_t r = rbeg + l.r0;
        for (; r + (UN - 1) * l.tpr < rend; r += UN * l.tpr) {
            float xv[UN][NV], dv[UN][NV], yv[UN][NV];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int64_t i = (r + u * l.tpr) * l.width + l.col;
                load_values<NV>(x + i, xv[u]);
                if constexpr (MODE == BN_BWD) {
                    load_values<NV>(dy + i, dv[u]);
                    load_values<NV>(y + i, yv[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) add(xv[u], dv[u], yv[u]);
        }
        if (r < rend) {  // the rest together, past the end the last row again and not added
            float xv[UN - 1][NV], dv[UN - 1][NV], yv[UN - 1][NV];
#pragma unroll
            for (int u = 0; u < UN - 1; ++u) {
                const int64_t i = min(r + u * l.tpr, rend - 1) * l.width + l.col;
                load_values<NV>(x + i, xv[u]);
                if constexpr (MODE == BN_BWD) {
                    load_values<NV>(dy + i, dv[u]);
                    load_values<NV>(y + i, yv[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < UN - 1; ++u)
                if (r + u * l.tpr < rend) add(xv[u], dv[u], yv[u]);
        }
    }
    const int W = l.Gs * NV;  // values of this slice
    if (l.active) {
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            s1[l.r0 * W + l.g * NV + e] = a1[e];
            s2[l.r0 * W + l.g * NV + e] = a2[e];
        }
    }
    __syncthreads();
    // The row lanes of each value, FLAT: and a channel's eight places in the 8 C values; in fixed order.
    // One loop over them by as many threads as there are channels is a chain of up to 256 LDS reads
    // (5 us for 17 channels): with FLAT, and where four threads or more share a value, the row lanes are
    // first reduced to at most 16 parts.  Elsewhere that would only add barriers (109 x 1952: 4.5 us without,
    // 7.1 with; 9000 x 128, two threads a value: 3.8 and 4.1).
    const int parts = W < 256 ? min(256 / W, 16) : 1;
    const bool reduce = parts < l.tpr && (KIND == BN_FLAT || parts >= 4);
    const int lanes = reduce ? parts : l.tpr;
    for (int q0 = 0; reduce && q0 < W; q0 += 256) {
        const int q = q0 + (parts > 1 ? (int)threadIdx.x % W : (int)threadIdx.x);
        const int part = parts > 1 ? (int)threadIdx.x / W : 0;
        float u1 = 0.0f, u2 = 0.0f;
        if (q < W && part < parts) {
#pragma unroll 4
            for (int rr = part; rr < l.tpr; rr += parts) {
                u1 += s1[rr * W + q];
                u2 += s2[rr * W + q];
            }
        }
        __syncthreads();
        if (q < W && part < parts) {
            s1[part * W + q] = u1;
            s2[part * W + q] = u2;
        }
        __syncthreads();
    }
    const int channels = KIND == BN_FLAT ? C : W;
    for (int c = threadIdx.x; c < channels; c += 256) {
        float u1 = 0.0f, u2 = 0.0f;
        for (int q = c; q < W; q += channels)
#pragma unroll 4
            for (int rr = 0; rr < lanes; ++rr) {
                u1 += s1[rr * W + q];
                u2 += s2[rr * W + q];
            }
        if (KIND == BN_FLAT && blockIdx.x == gridDim.x - 1) {  // the rows past the last eight
            for (int64_t r = srows * 8; r < rows; ++r) {
                const int64_t i = r * C + c;
                const float xv = bf16_bits_to_f32(x[i]);
                if constexpr (MODE == BN_STATS) {
                    const float d = xv - bf16_bits_to_f32(x[c]);
                    u1 += d;
                    u2 += d * d;
                } else {
                    const float gv = (relu && !(bf16_bits_to_f32(y[i]) > 0.0f)) ? 0.0f : bf16_bits_to_f32(dy[i]);
                    u1 += gv;
                    u2 += gv * (xv - mean[c]) * inv_std[c];
                }
            }
        }
        const int64_t o = (int64_t)blockIdx.x * C + (KIND == BN_FLAT ? 0 : (int64_t)blockIdx.y * 256 * NV) + c;
        p1[o] = u1;
        p2[o] = u2;
    }
}

// Sums over the chunks of 16 channels: LANES chunk lanes per channel (each adds every LANES-th chunk in
// order, eight loads in flight), combined in a fixed order: within the waves by a butterfly over their
// four chunk lanes, then over the waves four by four.  T: the sums' type.
template <typename T>
__device__ __forceinline__ T four_lanes(T u) {  // over the wave's four chunk lanes of a channel
    u += __shfl_xor(u, 16, kWave);
    return u + __shfl_xor(u, 32, kWave);
}

template <int LANES, typename T>
__device__ __forceinline__ bool bn_chunk_sums(const float* __restrict__ p1, const float* __restrict__ p2, int64_t chunks,
                                              int32_t C, int* channel, T* t1, T* t2) {
    __shared__ T s1[LANES / 4][16], s2[LANES / 4][16];
    const int cl = threadIdx.x & 15, part = threadIdx.x >> 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = (int)blockIdx.x * 16 + cl;
    T u1 = 0, u2 = 0;
    if (c < C) {
        if (chunks <= LANES) {
            if (part < chunks) {
                u1 = (T)p1[part * C + c];
                u2 = (T)p2[part * C + c];
            }
        } else {
            for (int64_t b = part; b < chunks; b += 8 * LANES) {
                float v1[8], v2[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    // (the last chunk's again past the end, not added below: a load under a condition
                    // waits for the one before it)
                    const int64_t at = min(b + LANES * k, chunks - 1) * C + c;
                    v1[k] = p1[at];
                    v2[k] = p2[at];
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool in = b + LANES * k < chunks;
                    u1 += in ? (T)v1[k] : (T)0;
                    u2 += in ? (T)v2[k] : (T)0;
                }
            }
        }
    }
    u1 = four_lanes(u1);
    u2 = four_lanes(u2);
    if (lane < 16) {
        s1[wave][cl] = u1;
        s2[wave][cl] = u2;
    }
    __syncthreads();
    if (wave > 0) return false;
    if constexpr (LANES == 16) {
        *t1 = (s1[0][cl] + s1[1][cl]) + (s1[2][cl] + s1[3][cl]);
        *t2 = (s2[0][cl] + s2[1][cl]) + (s2[2][cl] + s2[3][cl]);
    } else {
        static_assert(LANES == 64, "sixteen waves");
        const int w4 = 4 * (lane >> 4);
        *t1 = four_lanes((s1[w4][cl] + s1[w4 + 1][cl]) + (s1[w4 + 2][cl] + s1[w4 + 3][cl]));
        *t2 = four_lanes((s2[w4][cl] + s2[w4 + 1][cl]) + (s2[w4 + 2][cl] + s2[w4 + 3][cl]));
    }
    *channel = c;
    return lane < 16 && c < C;
}

// Backward sums dbeta = sum g and dgamma = sum g * xhat.
template <int LANES>
__global__ __launch_bounds__(16 * LANES) void bn_bwd_finalize_kernel(const float* __restrict__ p1,
                                                                     const float* __restrict__ p2, int64_t chunks,
                                                                     int32_t C, float* __restrict__ out1,
                                                                     float* __restrict__ out2) {
    int c;
    float t1, t2;
    if (!bn_chunk_sums<LANES>(p1, p2, chunks, C, &c, &t1, &t2)) return;
    out1[c] = t1;  // dbeta
    out2[c] = t2;  // dgamma
}

// One-pass statistics: the chunk sums S1 = sum d, S2 = sum d^2 (d = x - x[0][c]) added in fp64, then
// mean = x[0][c] + S1 / n and inv_std = 1 / sqrt(S2 / n - (S1 / n)^2 + eps) (biased variance,
// clamped at zero).
template <int LANES>
__global__ __launch_bounds__(16 * LANES) void bn_stats_finalize_kernel(const float* __restrict__ p1,
                                                                       const float* __restrict__ p2, int64_t chunks,
                                                                       int32_t C, int64_t rows, float eps,
                                                                       const uint16_t* __restrict__ x,
                                                                       float* __restrict__ mean,
                                                                       float* __restrict__ inv_std) {
    int c;
    double t1, t2;
    if (!bn_chunk_sums<LANES>(p1, p2, chunks, C, &c, &t1, &t2)) return;
    const double n = (double)rows;
    const double d1 = t1 / n;
    double var = t2 / n - d1 * d1;
    if (var < 0.0) var = 0.0;
    mean[c] = (float)((double)bf16_bits_to_f32(x[c]) + d1);
    inv_std[c] = 1.0f / sqrtf((float)var + eps);
}


// y = act(gamma * (x - mean) * inv_std + beta)
template <int KIND, int ROWS>
__global__ __launch_bounds__(256) void bn_apply_kernel(const uint16_t* __restrict__ x, int64_t rows, int32_t C,
                                                       const float* __restrict__ mean, const float* __restrict__ inv_std,
                                                       const float* __restrict__ gamma, const float* __restrict__ beta,
                                                       int relu, uint16_t* __restrict__ y) {
    using Lane = BnLane<KIND>;
    constexpr int NV = Lane::NV;
    const Lane l(C);
    auto act = [&](float v, float m, float is, float ga, float be) {
        const float o = ga * (v - m) * is + be;
        return relu ? fmaxf(o, 0.0f) : o;
    };
    if (KIND == BN_FLAT && blockIdx.x == gridDim.x - 1) {  // the rows past the last eight
        for (int64_t i = rows / 8 * 8 * C + threadIdx.x; i < rows * C; i += 256) {
            const int c = (int)(i % C);
            y[i] = (uint16_t)f32_to_bf16_bits(act(bf16_bits_to_f32(x[i]), mean[c], inv_std[c], gamma[c], beta[c]));
        }
    }
    const int64_t srows = KIND == BN_FLAT ? rows / 8 : rows;
    const int64_t r = (int64_t)blockIdx.x * (ROWS * l.tpr) + l.r0;
    float v[ROWS][NV];
    // (past the end the last row again: a load under a condition waits for the one before it)
#pragma unroll
    for (int u = 0; u < ROWS; ++u) load_values<NV>(x + min(r + u * l.tpr, srows - 1) * l.width + l.col, v[u]);
    float f[4][NV];
    bn_factors<KIND, 4>(l, C, {mean, inv_std, gamma, beta}, f);
    if (!l.active) return;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        if (r + u * l.tpr >= srows) break;
        uint16_t* const o = y + (r + u * l.tpr) * l.width + l.col;
#pragma unroll
        for (int e = 0; e < NV; ++e) v[u][e] = act(v[u][e], f[0][e], f[1][e], f[2][e], f[3][e]);
        if constexpr (NV == 8)
            *reinterpret_cast<u32x4*>(o) = u32x4{pack_bf16x2(v[u][0], v[u][1]), pack_bf16x2(v[u][2], v[u][3]),
                                                 pack_bf16x2(v[u][4], v[u][5]), pack_bf16x2(v[u][6], v[u][7])};
        else
            *o = (uint16_t)f32_to_bf16_bits(v[u][0]);
    }
}

// dx = gamma * inv_std * (g - dbeta / rows - xhat * dgamma / rows)
template <int KIND, int ROWS>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ y,
                                                           const uint16_t* __restrict__ dy, int64_t rows, int32_t C,
                                                           int relu, const float* __restrict__ mean,
                                                           const float* __restrict__ inv_std,
                                                           const float* __restrict__ gamma,
                                                           const float* __restrict__ dgamma,
                                                           const float* __restrict__ dbeta, uint16_t* __restrict__ dx) {
    using Lane = BnLane<KIND>;
    constexpr int NV = Lane::NV;
    const Lane l(C);
    const float inv_rows = 1.0f / (float)rows;
    auto grad = [&](float xv, float yv, float dv, float m, float is, float ga, float db, float dg) {
        const float g = relu && !(yv > 0.0f) ? 0.0f : dv;
        const float xh = (xv - m) * is;
        return ga * is * (g - db * inv_rows - xh * dg * inv_rows);
    };
    if (KIND == BN_FLAT && blockIdx.x == gridDim.x - 1) {  // the rows past the last eight
        for (int64_t i = rows / 8 * 8 * C + threadIdx.x; i < rows * C; i += 256) {
            const int c = (int)(i % C);
            dx[i] = (uint16_t)f32_to_bf16_bits(grad(bf16_bits_to_f32(x[i]), bf16_bits_to_f32(y[i]),
                                                    bf16_bits_to_f32(dy[i]), mean[c], inv_std[c], gamma[c], dbeta[c],
                                                    dgamma[c]));
        }
    }
    const int64_t srows = KIND == BN_FLAT ? rows / 8 : rows;
    const int64_t r = (int64_t)blockIdx.x * (ROWS * l.tpr) + l.r0;
    float xv[ROWS][NV], yv[ROWS][NV], dv[ROWS][NV];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int64_t i = min(r + u * l.tpr, srows - 1) * l.width + l.col;
        load_values<NV>(x + i, xv[u]);
        load_values<NV>(y + i, yv[u]);
        load_values<NV>(dy + i, dv[u]);
    }
    float f[5][NV];
    bn_factors<KIND, 5>(l, C, {mean, inv_std, gamma, dbeta, dgamma}, f);
    if (!l.active) return;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        if (r + u * l.tpr >= srows) break;
        uint16_t* const o = dx + (r + u * l.tpr) * l.width + l.col;
        float v[NV];
#pragma unroll
        for (int e = 0; e < NV; ++e)
            v[e] = grad(xv[u][e], yv[u][e], dv[u][e], f[0][e], f[1][e], f[2][e], f[3][e], f[4][e]);
        if constexpr (NV == 8)
            *reinterpret_cast<u32x4*>(o) = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                 pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
        else
            *o = (uint16_t)f32_to_bf16_bits(v[0]);
    }
}

// gradient of ReLU applied after the fact: g = dy * [y > 0]
// 8 elements (16 bytes of each tensor) per thread; the last thread takes the ragged tail
// element by element
__global__ __launch_bounds__(256) void relu_bwd_kernel(const uint16_t* __restrict__ y, const uint16_t* __restrict__ dy,
                                                       int64_t total, uint16_t* __restrict__ dx) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= total) return;
    if (i + 8 <= total) {
        const u32x4 yv = *reinterpret_cast<const u32x4*>(y + i);
        const u32x4 gv = *reinterpret_cast<const u32x4*>(dy + i);
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = bf16_bits_to_f32(yv[e] & 0xFFFFu) > 0.0f ? (gv[e] & 0xFFFFu) : 0u;
            const uint32_t hi = bf16_bits_to_f32(yv[e] >> 16) > 0.0f ? (gv[e] & 0xFFFF0000u) : 0u;
            o[e] = lo | hi;
        }
        *reinterpret_cast<u32x4*>(dx + i) = o;
    } else {
        for (int64_t j = i; j < total; ++j) dx[j] = bf16_bits_to_f32(y[j]) > 0.0f ? dy[j] : (uint16_t)0;
    }
}

// softmax cross-entropy, mean over the batch: one wave per sample (classes <= 64 * 32)
__global__ __launch_bounds__(64) void softmax_xent_kernel(const float* __restrict__ z, const int32_t* __restrict__ labels,
                                                          int32_t N, int32_t K, float* __restrict__ loss_per_sample,
                                                          uint16_t* __restrict__ dz) {
    const int n = blockIdx.x, lane = threadIdx.x;
    const float* zn = z + (int64_t)n * K;
    float mx = -INFINITY;
    for (int j = lane; j < K; j += 64) mx = fmaxf(mx, zn[j]);
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float se = 0.0f;
    for (int j = lane; j < K; j += 64) se += expf(zn[j] - mx);
    for (int off = 32; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
    const float lse = mx + logf(se);
    // a label outside [0, K) selects no logit: its loss is NaN and its gradient has no -1
    // term, so the row is never read out of bounds
    const int lab = labels[n];
    const bool lab_ok = lab >= 0 && lab < K;
    for (int j = lane; j < K; j += 64) {
        const float pj = expf(zn[j] - lse);
        dz[(int64_t)n * K + j] = (uint16_t)f32_to_bf16_bits((pj - (j == lab ? 1.0f : 0.0f)) / (float)N);
    }
    if (lane == 0) loss_per_sample[n] = lab_ok ? lse - zn[lab] : __builtin_nanf("");
}

// mean of the per-sample losses, summed in index order by one thread; the block first
// stages the values in LDS in chunks (parallel, coalesced loads), so that the serial sum
// reads LDS instead of waiting on one global load per element
__global__ __launch_bounds__(256) void mean_kernel(const float* __restrict__ v, int32_t n, float* __restrict__ out) {
    constexpr int kChunk = 4096;
    __shared__ float buf[kChunk];
    float acc = 0.0f;
    for (int base = 0; base < n; base += kChunk) {
        const int len = n - base < kChunk ? n - base : kChunk;
        for (int i = threadIdx.x; i < len; i += 256) buf[i] = v[base + i];
        __syncthreads();
        if (threadIdx.x == 0)
            for (int i = 0; i < len; ++i) acc += buf[i];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = acc / (float)n;
}

unsigned blocks_for(int64_t total) { return (unsigned)((total + 255) / 256); }

}  // namespace

hipError_t launch_maxpool_fwd(const PoolArgs& a, const uint16_t* x, uint16_t* y, int32_t* arg, hipStream_t s) {
    const int64_t total = (int64_t)a.N * a.P * a.Q * a.C;
    const int64_t in_total = (int64_t)a.N * a.H * a.W * a.C;
    if (a.C % 8 == 0 && (a.k == 2 || a.k == 3) && total < 0x7FFFFFFFll && in_total < 0x7FFFFFFFll) {
        const uint32_t groups = (uint32_t)(total / 8);
        const FastDiv dg = make_fastdiv((uint32_t)(a.C / 8)), dq = make_fastdiv((uint32_t)a.Q),
                      dp = make_fastdiv((uint32_t)a.P);
        if (a.k == 3)
            hipLaunchKernelGGL(maxpool_fwd8_kernel<3>, dim3(blocks_for(groups)), dim3(256), 0, s, a, dg, dq, dp, groups,
                               x, y, arg);
        else
            hipLaunchKernelGGL(maxpool_fwd8_kernel<2>, dim3(blocks_for(groups)), dim3(256), 0, s, a, dg, dq, dp, groups,
                               x, y, arg);
    } else if (a.C % 8 == 0)
        hipLaunchKernelGGL(maxpool_fwd_kernel<8>, dim3(blocks_for(total / 8)), dim3(256), 0, s, a,
                           make_pool_split(a.N, a.P, a.Q, a.C), x, y, arg);
    else
        hipLaunchKernelGGL(maxpool_fwd_kernel<1>, dim3(blocks_for(total)), dim3(256), 0, s, a,
                           make_pool_split(a.N, a.P, a.Q, a.C), x, y, arg);
    return hipGetLastError();
}

hipError_t launch_maxpool_bwd(const PoolArgs& a, const uint16_t* dy, const int32_t* arg, void* dx, int dx_f32,
                              hipStream_t s) {
    const int64_t total = (int64_t)a.N * a.H * a.W * a.C;
    const int64_t out_total = (int64_t)a.N * a.P * a.Q * a.C;
    const int64_t cp = ((int64_t)a.H + a.k - 1) / a.k, cq = ((int64_t)a.W + a.k - 1) / a.k;
    const int64_t cells = a.N * cp * cq * (a.C / 8);
    // by cells from 32768 threads on (k = 2 / 3, of the gather's time: 32 k to 48 k threads 0.91 / 0.96, 100 k to
    // 150 k 0.76 / 0.71); below, its k x k stores one after the other are a longer chain than the gather's
    // two loads (16 k to 32 k 1.02 / 1.10, below 16 k 1.05 / 1.30)
    if (a.C % 8 == 0 && a.k == a.s && a.pad == 0 && (a.k == 2 || a.k == 3) && total < 0x7FFFFFFFll &&
        cells >= 32768 && cells < 0x7FFFFFFFll) {
        const uint32_t groups = (uint32_t)cells;
        const FastDiv dg = make_fastdiv((uint32_t)(a.C / 8)), dq = make_fastdiv((uint32_t)cq),
                      dp = make_fastdiv((uint32_t)cp);
        if (a.k == 2)
            hipLaunchKernelGGL(maxpool_bwd_cells_kernel<2>, dim3(blocks_for(groups)), dim3(256), 0, s, a, dg, dq, dp,
                               (uint32_t)cp, (uint32_t)cq, groups, dy, arg, dx, dx_f32);
        else
            hipLaunchKernelGGL(maxpool_bwd_cells_kernel<3>, dim3(blocks_for(groups)), dim3(256), 0, s, a, dg, dq, dp,
                               (uint32_t)cp, (uint32_t)cq, groups, dy, arg, dx, dx_f32);
    } else if (a.C % 8 == 0 && total < 0x7FFFFFFFll && out_total < 0x7FFFFFFFll) {
        const uint32_t groups = (uint32_t)(total / 8);
        hipLaunchKernelGGL(maxpool_bwd8_kernel, dim3(blocks_for(groups)), dim3(256), 0, s, a,
                           make_fastdiv((uint32_t)(a.C / 8)), make_fastdiv((uint32_t)a.W), make_fastdiv((uint32_t)a.H),
                           groups, dy, arg, dx, dx_f32);
    } else if (a.C % 8 == 0)
        hipLaunchKernelGGL(maxpool_bwd_kernel<8>, dim3(blocks_for(total / 8)), dim3(256), 0, s, a,
                           make_pool_split(a.N, a.H, a.W, a.C), dy, arg, dx, dx_f32);
    else
        hipLaunchKernelGGL(maxpool_bwd_kernel<1>, dim3(blocks_for(total)), dim3(256), 0, s, a,
                           make_pool_split(a.N, a.H, a.W, a.C), dy, arg, dx, dx_f32);
    return hipGetLastError();
}

hipError_t launch_avgpool(int32_t N, int32_t HW, int32_t C, const uint16_t* x, void* y, int y_f32, hipStream_t s) {
    if (C % 8 == 0)  // 16-byte rows (the caller guarantees 16-byte aligned buffers)
        hipLaunchKernelGGL(avgpool8_kernel, dim3(blocks_for((int64_t)N * C)), dim3(256), 0, s, N, HW, C, x, y, y_f32);
    else
        hipLaunchKernelGGL(avgpool_kernel, dim3(blocks_for((int64_t)N * C)), dim3(256), 0, s, N, HW, C, x, y, y_f32);
    return hipGetLastError();
}

// FLAT from this many values on: its 16-byte loads win by size (sums of the three kernels, forward and
// backward, us: 4.3 M values of 31 channels 16.2 and 19.7, one value at a time 17.6 and 20.3; 4.3 M of 226 16.7
// and 21.0 against 19.7 and 22.6; 81 M of 226 102 and 209 against 207 and 299); below, its few blocks and longer
// LDS combination lose (2.1 M of 226 equal, 14.4 and 16.5; 1.4 M 13.0 and 14.7 against 12.0 and 13.9; 0.6 M
// of 17 12.8 and 13.7 against 10.3 and 11.0).
constexpr int64_t kBnFlatMin = (int64_t)1 << 21;
BnPlan plan_bn(int64_t rows, int32_t C) {
    BnPlan p;
    p.kind = C % 8 == 0 ? BN_VEC : C <= 256 && rows * C >= kBnFlatMin ? BN_FLAT : BN_SCALAR;
    const int64_t srows = p.kind == BN_FLAT ? rows / 8 : rows;  // rows of C (FLAT: 8 C) values
    const int G = p.kind == BN_VEC ? C / 8 : C;
    const int gs = G < 256 ? G : 256;
    p.tpr = 256 / gs;
    // about 512 row chunks (FLAT: 256, which take no more workspace than single rows would)
    const int64_t most = p.kind == BN_FLAT ? 256 : 512;
    int64_t rpc = (srows + most - 1) / most;
    const int64_t least = (p.kind == BN_FLAT ? 2 : 8) * (int64_t)p.tpr;  // rows per thread, times tpr
    if (rpc < least) rpc = least;
    p.rpc = rpc;
    p.chunks = (srows + rpc - 1) / rpc;
    p.slices = (G + 255) / 256;
    // Rows per thread of the element-wise passes: four where that leaves enough blocks, so that its factors serve
    // more values, else one.  Measured forward / backward, us, with four and with one: 8 channels a thread, 392
    // blocks of four rows (25088 x 128) 4.7 / 6.3 and 5.0 / 6.4, 196 (12544 x 128) 3.7 / 5.1 and 3.6 / 4.9, 98
    // (12544 x 64) 3.6 / 4.6 and 3.0 / 3.5; one channel a thread, 1250 blocks (10000 x 100) 3.5 / 4.2 and 3.9 /
    // 5.5, 560 (1117 x 260) 3.0 / 3.9 and 2.7 / 3.1.  FLAT always has them.
    const int64_t blocks4 = (srows + 4 * p.tpr - 1) / (4 * p.tpr) * p.slices;
    p.apply_rows = p.kind == BN_FLAT || blocks4 >= (p.kind == BN_VEC ? 256 : 768) ? 4 : 1;
    p.blocks = (srows + p.apply_rows * p.tpr - 1) / (p.apply_rows * p.tpr);
    p.ws_bytes = (size_t)2 * p.chunks * C * 4;
    return p;
}

namespace {

// f(kind, rows) with the plan's kind and rows per thread of the element-wise passes as compile-time
// constants, and g(lanes) with the finalize passes' chunk lanes
template <typename F>
void bn_dispatch(const BnPlan& p, F f) {
    const auto with_rows = [&](auto kind) {
        if (p.apply_rows == 1)
            f(kind, std::integral_constant<int, 1>{});
        else
            f(kind, std::integral_constant<int, 4>{});
    };
    switch (p.kind) {
        case BN_VEC: with_rows(std::integral_constant<int, BN_VEC>{}); break;
        case BN_FLAT: with_rows(std::integral_constant<int, BN_FLAT>{}); break;
        default: with_rows(std::integral_constant<int, BN_SCALAR>{}); break;
    }
}

// 16 chunk lanes (256 threads) up to 208 chunks, 64 beyond (forward / backward, us, with 16 and with 64: 12 chunks
// of 64 channels 2.4 / 1.9 and 2.6 / 2.2, 196 of 128 3.2 / 3.0 and 4.1 / 3.2, 250 of 250 4.8 / 4.7 and 4.0 / 3.2, 512
// of 128 4.8 / 4.7 and 3.9 / 3.9).
template <typename G>
void bn_lanes(const BnPlan& p, G g) {
    if (p.chunks <= 208)
        g(std::integral_constant<int, 16>{});
    else
        g(std::integral_constant<int, 64>{});
}

}  // namespace

hipError_t launch_bn_train_fwd(const uint16_t* x, int64_t rows, int32_t C, const float* gamma, const float* beta,
                               float eps, int relu, uint16_t* y, float* mean, float* inv_std, float* ws,
                               hipStream_t s) {
    const BnPlan p = plan_bn(rows, C);
    if (p.blocks > 0x7FFFFFFF || p.chunks > 0x7FFFFFFF || p.slices > 65535) return hipErrorInvalidValue;
    float* p1 = ws;
    float* p2 = ws + p.chunks * C;
    const unsigned cb = (unsigned)((C + 15) / 16);
    const uint16_t* none = nullptr;
    const float* nof = nullptr;
    bn_dispatch(p, [&](auto kind, auto per_thread) {
        constexpr int KIND = decltype(kind)::value, ROWS = decltype(per_thread)::value;
        // one pass over x for both statistics (shifted sums), then the per-channel finalize
        hipLaunchKernelGGL((bn_partial_kernel<BN_STATS, KIND>), dim3((unsigned)p.chunks, (unsigned)p.slices),
                           dim3(256), 0, s, x, none, none, rows, C, p.rpc, 0, nof, nof, p1, p2);
        bn_lanes(p, [&](auto lanes) {
            constexpr int L = decltype(lanes)::value;
            hipLaunchKernelGGL(bn_stats_finalize_kernel<L>, dim3(cb), dim3(16 * L), 0, s, p1, p2, p.chunks, C, rows, eps, x,
                               mean, inv_std);
        });
        hipLaunchKernelGGL((bn_apply_kernel<KIND, ROWS>), dim3((unsigned)p.blocks, (unsigned)p.slices), dim3(256),
                           0, s, x, rows, C, mean, inv_std, gamma, beta, relu, y);
    });
    return hipGetLastError();
}

hipError_t launch_bn_train_bwd(const uint16_t* x, const uint16_t* y, const uint16_t* dy, int64_t rows, int32_t C,
                               int relu, const float* mean, const float* inv_std, const float* gamma, float* dgamma,
                               float* dbeta, uint16_t* dx, float* ws, hipStream_t s) {
    const BnPlan p = plan_bn(rows, C);
    if (p.blocks > 0x7FFFFFFF || p.chunks > 0x7FFFFFFF || p.slices > 65535) return hipErrorInvalidValue;
    float* p1 = ws;
    float* p2 = ws + p.chunks * C;
    bn_dispatch(p, [&](auto kind, auto per_thread) {
        constexpr int KIND = decltype(kind)::value, ROWS = decltype(per_thread)::value;
        hipLaunchKernelGGL((bn_partial_kernel<BN_BWD, KIND>), dim3((unsigned)p.chunks, (unsigned)p.slices),
                           dim3(256), 0, s, x, y, dy, rows, C, p.rpc, relu, mean, inv_std, p1, p2);
        bn_lanes(p, [&](auto lanes) {
            constexpr int L = decltype(lanes)::value;
            hipLaunchKernelGGL(bn_bwd_finalize_kernel<L>, dim3((unsigned)((C + 15) / 16)), dim3(16 * L), 0, s, p1, p2, p.chunks,
                               C, dbeta, dgamma);
        });
        hipLaunchKernelGGL((bn_bwd_apply_kernel<KIND, ROWS>), dim3((unsigned)p.blocks, (unsigned)p.slices),
                           dim3(256), 0, s, x, y, dy, rows, C, relu, mean, inv_std, gamma, dgamma, dbeta, dx);
    });
    return hipGetLastError();
}

hipError_t launch_relu_bwd(const uint16_t* y, const uint16_t* dy, int64_t total, uint16_t* dx, hipStream_t s) {
    hipLaunchKernelGGL(relu_bwd_kernel, dim3(blocks_for((total + 7) / 8)), dim3(256), 0, s, y, dy, total, dx);
    return hipGetLastError();
}

hipError_t launch_softmax_xent(const float* z, const int32_t* labels, int32_t N, int32_t K, float* loss,
                               float* loss_per_sample, uint16_t* dz, hipStream_t s) {
    hipLaunchKernelGGL(softmax_xent_kernel, dim3((unsigned)N), dim3(64), 0, s, z, labels, N, K, loss_per_sample, dz);
    hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, s, loss_per_sample, N, loss);
    return hipGetLastError();
}

}  // namespace tbn
