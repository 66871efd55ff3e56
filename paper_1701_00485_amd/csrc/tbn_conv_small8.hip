// tbn_conv_small8.hip -- the int8- and fp8-activation forward passes (tbn_conv_i8.hip, tbn_conv_fp8.hip)
// for layers with few output rows: the small-layer kernel of tbn_conv_small.hip on 8-bit operands.
// A block owns 32 pixels x 32 TN filters; its W waves split the reduction (stages of 128 elements,
// wave w takes w, w + W, ..), each from its own LDS ring without barriers, and add their sums through
// LDS in wave order: int32 sums for int8 (exact), fp32 for fp8.
//   * int8: lane-half h of v_mfma_i32_32x32x32_i8 takes segments u + 4 h of a row in step u, so its filter
//     operand over the stage is code chunk h;
//   * fp8: step t of v_mfma_scale_f32_32x32x64_f8f6f4 takes segments 4 t + h and 4 t + 2 + h of a row and
//     words 2 h, 2 h + 1 of the filter's chunk t (repacked E2M1 layout).
#include <type_traits>

#include "tbn_codes8.h"
#include "tbn_device.h"
#include "tbn_dma.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

constexpr int BK = 128;

struct Small8Args {
    const void* x;
    const uint32_t* codes;
    const float* alpha;
    void* y;
    float x_scale;
    int32_t N, H, W, C, K, R, S, sh, sw, ph, pw, P, Q;
    int32_t relu, y_f32;
    FastDiv div_q, div_pq, div_tilesN, div_c, div_s;
    uint32_t rep_lo, rep_hi;
};

// UNI: C % 128 == 0, a stage lies in one tap.
template <bool FP8, int TN, int W, int S, bool UNI>
__global__ __launch_bounds__(64 * W) void conv_small8_kernel(const Small8Args a) {
    constexpr int BN = 32 * TN;
    constexpr int PITCH = BN + 4;          // sums per pixel
    constexpr int XB = 32 * 128;           // a stage: 32 rows of 128 bytes, ..
    constexpr int STAGE = XB + TN * 1024;  // .. two code chunks of BN filters
    constexpr int RING = S * STAGE;
    constexpr int SUMS = W * 32 * PITCH * 4;
    using Acc = typename std::conditional<FP8, f32x16, i32x16>::type;
    using Sum = typename std::conditional<FP8, f32x4, i32x4>::type;
    using Scalar = typename std::conditional<FP8, float, int>::type;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[W * RING > SUMS ? W * RING : SUMS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;

    const uint32_t PQ = (uint32_t)a.P * (uint32_t)a.Q;
    const uint32_t M = (uint32_t)a.N * PQ;
    const int C = a.C, K = a.K;
    const int n = a.R * a.S * C;
    const int nst = (n + BK - 1) / BK, nch = (n + 63) / 64;
    const int KB = (K + 63) / 64;
    const uint32_t tilesN = (uint32_t)(K + BN - 1) / BN;
    const uint32_t tile = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t mt = fdiv(tile, a.div_tilesN);
    const uint32_t m0 = mt * 32;
    const int n0 = (int)(tile - mt * tilesN) * BN;

    const v4i rs_x = make_rsrc(a.x, (uint32_t)a.N * (uint32_t)a.H * (uint32_t)a.W * (uint32_t)C);
    const v4i rs_c = make_rsrc(a.codes, (uint32_t)KB * (uint32_t)nch * 1024u);
    uint8_t* const ring = smem + wave * RING;
    const uint32_t ring_base = lds_addr(ring);

    // ---- copies, as in the bf16 kernel (rows 8 j + lane / 8, segments swizzled by (row / 2) % 8) ----
    uint32_t rbase[4], rmask[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t m = m0 + (uint32_t)(8 * j + (lane >> 3));
        uint64_t mask = 0;
        rbase[j] = 0;
        if (m < M) {
            const uint32_t img = fdiv(m, a.div_pq);
            const uint32_t pq = m - img * PQ;
            const uint32_t p = fdiv(pq, a.div_q);
            const int h0 = (int)p * a.sh - a.ph, w0 = (int)(pq - p * (uint32_t)a.Q) * a.sw - a.pw;
            rbase[j] = (uint32_t)((((int32_t)img * a.H + h0) * a.W + w0) * C);
            const int slo = max(0, -w0), shi = min(a.S, a.W - w0);
            const int rlo = max(0, -h0), rhi = min(a.R, a.H - h0);
            if (shi > slo && rhi > rlo) {
                const uint64_t wbits = (1ull << shi) - (1ull << slo);
                const uint64_t rowsel = (1ull << (rhi * a.S)) - (1ull << (rlo * a.S));
                mask = wbits * ((((uint64_t)a.rep_hi << 32) | a.rep_lo) & rowsel);
            }
        }
        rmask[j][0] = (uint32_t)mask;
        rmask[j][1] = (uint32_t)(mask >> 32);
    }
    const int lseg = (lane & 7) ^ ((lane >> 4) & 3);  // of the even instructions (odd: ^ 4)
    // code copy t: chunk 2 st + half of filter n0 + 32 t + l32
    uint32_t c_lane[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int f = n0 + 32 * t + l32;
        c_lane[t] = (f >> 6) < KB ? (uint32_t)((f >> 6) * nch + half) * 1024u + (uint32_t)(f & 63) * 16u : 0x80000000u;
    }
    auto issue = [&](int st, int slot) {
        const uint32_t base = ring_base + (uint32_t)(slot * STAGE);
        uint32_t toff[2];
        int tap[2];
        if constexpr (UNI) {
            const uint32_t e0 = (uint32_t)st * BK;  // scalar
            tap[0] = tap[1] = (int)fdiv(e0, a.div_c);
            const int r = (int)fdiv((uint32_t)tap[0], a.div_s);
            const uint32_t t0 = (uint32_t)((r * a.W + tap[0] - r * a.S) * C) + (e0 - (uint32_t)(tap[0] * C));
            toff[0] = t0 + 16u * (uint32_t)lseg;
            toff[1] = t0 + 16u * (uint32_t)(lseg ^ 4);
        } else {
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const uint32_t e = (uint32_t)st * BK + 16u * (uint32_t)(lseg ^ (4 * o));
                const uint32_t t = fdiv(e, a.div_c);
                const uint32_t r = fdiv(t, a.div_s);
                tap[o] = (int)min(t, 63u);  // past the filter: bit 63, clear in rmask (R*S <= 63)
                toff[o] = (r * (uint32_t)a.W + t - r * (uint32_t)a.S) * (uint32_t)C + (e - t * (uint32_t)C);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = UNI ? min(tap[0], 63) : tap[j & 1];
            const uint32_t bits = t >= 32 ? rmask[j][1] : rmask[j][0];
            const bool ok = (bits >> (t & 31)) & 1u;
            dma_b128(rs_x, base + (uint32_t)(1024 * j), ok ? rbase[j] + toff[j & 1] : 0x80000000u);
        }
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const bool ok = 2 * st + half < nch;  // an odd chunk count: the last stage has one
            dma_b128(rs_c, base + (uint32_t)(XB + 1024 * t), ok ? c_lane[t] + (uint32_t)st * 2048u : 0x80000000u);
        }
    };
    constexpr int DMAS = 4 + TN;

    // ---- the scale of this thread's outputs (4 channels of one pixel), requested now ----
    constexpr int GROUPS = BN / 4;
    constexpr int EPT = (32 * GROUPS + 64 * W - 1) / (64 * W);
    float cs[EPT][4];
#pragma unroll
    for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + 4 * ((tid + 64 * W * e) % GROUPS) + j;
            cs[e][j] = a.alpha[col < K ? col : K - 1] * a.x_scale;  // past K: never stored
        }

    Acc acc[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0;
    const uint32_t two22 = __builtin_amdgcn_readfirstlane(0x22222222u);
    const int cnt = nst > wave ? (nst - wave + W - 1) / W : 0;  // this wave's stages
#pragma unroll
    for (int i = 0; i < S; ++i)
        if (i < cnt) issue(wave + W * i, i);
    const uint8_t* const arow = ring + l32 * 128;
    const int sw = (l32 >> 1) & 7;
    int slot = 0;
    for (int i = 0; i < cnt; ++i) {
        if (i + S <= cnt)  // stages up to i + S - 1 are in flight
            wait_vmcnt((S - 1) * DMAS);
        else
            wait_vmcnt(0);
        asm volatile("" ::: "memory");
        const int so = slot * STAGE;
        i32x4 x[4];
        u32x4 c[TN];  // int8: the words of chunk `half`; fp8: words 2 h, 2 h + 1 of both chunks
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s16 = FP8 ? 4 * (u >> 1) + 2 * (u & 1) + half : u + 4 * half;
            x[u] = *reinterpret_cast<const i32x4*>(arow + so + 16 * (s16 ^ sw));
        }
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const uint8_t* const cp = ring + so + XB + 1024 * t + 16 * l32;
            if constexpr (FP8) {
                const u32x2 lo = *reinterpret_cast<const u32x2*>(cp + 8 * half);
                const u32x2 hi = *reinterpret_cast<const u32x2*>(cp + 512 + 8 * half);
                c[t] = u32x4{lo.x, lo.y, hi.x, hi.y};
            } else {
                c[t] = *reinterpret_cast<const u32x4*>(cp + 512 * half);
            }
        }
        if (i + S < cnt) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the slot is read before it is refilled
            issue(wave + W * (i + S), slot);
        }
        slot = slot + 1 == S ? 0 : slot + 1;
        if constexpr (FP8) {
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const i32x8 act = __builtin_shufflevector(x[2 * s2], x[2 * s2 + 1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[t] = mfma_f4f8(decode_f4(c[t][2 * s2], c[t][2 * s2 + 1], two22), act, acc[t]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[t] = mfma_i8(decode_i8(c[t][u]), x[u], acc[t]);
        }
    }

    // ---- the waves' sums: lane holds pixel l32 and, per v / 4, four consecutive filters ----
    __syncthreads();  // the sums lie over the rings
    Scalar* const sums = reinterpret_cast<Scalar*>(smem);
    Scalar* const mine = sums + (wave * 32 + l32) * PITCH;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<Sum*>(mine + 32 * t + 8 * g + 4 * half) =
                Sum{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int gi = tid + 64 * W * e;
        const int pix = gi / GROUPS;
        const uint32_t row = m0 + (uint32_t)pix;
        const int col0 = n0 + 4 * (gi % GROUPS);
        if (gi >= 32 * GROUPS || row >= M || col0 >= K) continue;
        Sum s = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < W; ++w)
            s += *reinterpret_cast<const Sum*>(sums + (w * 32 + pix) * PITCH + 4 * (gi % GROUPS));
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = (float)s[j] * cs[e][j];
            if (a.relu) v[j] = fmaxf(v[j], 0.0f);
        }
        const int64_t o = (int64_t)row * K + col0;
        if (K % 4 == 0) {
            if (a.y_f32)
                *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.y) + o) = f32x4{v[0], v[1], v[2], v[3]};
            else
                *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(a.y) + o) =
                    u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (col0 + j >= K) break;
                if (a.y_f32)
                    reinterpret_cast<float*>(a.y)[o + j] = v[j];
                else
                    reinterpret_cast<uint16_t*>(a.y)[o + j] = (uint16_t)f32_to_bf16_bits(v[j]);
            }
        }
    }
}

template <bool FP8, int TN, int W, int S>
hipError_t launch_cfg(const Small8Args& args, hipStream_t stream) {
    Small8Args a = args;
    const int64_t M = (int64_t)a.N * a.P * a.Q;
    const int64_t tilesN = (a.K + 32 * TN - 1) / (32 * TN);
    const int64_t tiles = ((M + 31) / 32) * tilesN;
    if (tiles >= 0x7FFFFFFFll) return hipErrorInvalidValue;
    a.div_tilesN = make_fastdiv((uint32_t)tilesN);
    const dim3 grid((unsigned)tiles), block(64 * W);
    if (a.C % 128 == 0)
        hipLaunchKernelGGL((conv_small8_kernel<FP8, TN, W, S, true>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((conv_small8_kernel<FP8, TN, W, S, false>), grid, block, 0, stream, a);
    return hipGetLastError();
}

template <bool FP8, typename Args>
hipError_t launch_small8(const Args& g, int cfg, hipStream_t stream) {
    Small8Args a;
    a.x = g.x;
    a.codes = g.codes;
    a.alpha = g.alpha;
    a.y = g.y;
    a.x_scale = g.x_scale;
    a.N = g.N; a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K; a.R = g.R; a.S = g.S;
    a.sh = g.sh; a.sw = g.sw; a.ph = g.ph; a.pw = g.pw; a.P = g.P; a.Q = g.Q;
    a.relu = g.relu;
    a.y_f32 = g.y_f32;
    a.div_q = make_fastdiv((uint32_t)g.Q);
    a.div_pq = make_fastdiv((uint32_t)g.P * (uint32_t)g.Q);
    a.div_c = make_fastdiv((uint32_t)g.C);
    a.div_s = make_fastdiv((uint32_t)g.S);
    uint64_t rep = 0;
    for (int r = 0; r < g.R; ++r) rep |= 1ull << (r * g.S);
    a.rep_lo = (uint32_t)rep;
    a.rep_hi = (uint32_t)(rep >> 32);
    switch (cfg) {
        case 5: return launch_cfg<FP8, 1, 4, 3>(a, stream);
        case 6: return launch_cfg<FP8, 1, 8, 3>(a, stream);
        default: return launch_cfg<FP8, 2, 8, 3>(a, stream);
    }
}

}  // namespace

int conv_code8_tile(int32_t N, int32_t P, int32_t Q, int32_t K, int64_t n) {
    const int64_t M = (int64_t)N * P * Q;
    // few output rows: the small-layer kernel.  Measured against the tiles below (graph-replayed, us,
    // int8 / fp8; b1 and b2 are its blocks with tiles of 32 and 64 filters): a block per CU at most,
    // 7 x 7 x 512 at batch 8 19.3 / 15.4 -> 6.0 / 5.0, 21 x 21 x 64 -> 224 at batch 2 6.6 / 6.0 -> 3.9 / 3.7
    // (four waves where eight have a stage or less each); two blocks per CU, 14 x 14 x 256 at batch 8
    // 11.6 / 9.6 -> 5.8 / 4.8; beyond that no gain (28 x 28 x 128 at batch 8 7.7 / 6.7 against 8.1 / 7.0)
    const int64_t rows = (M + 31) / 32, b1 = rows * ((K + 31) / 32), b2 = rows * ((K + 63) / 64);
    const int64_t nst = (n + 127) / 128;
    if (b1 <= 256) return nst <= 8 ? 5 : 6;
    if (b1 <= 512) return nst >= 12 && b2 <= 256 ? 7 : 5;
    int cfg = K > 128 ? 1 : (K > 64 ? 2 : 3);
    const int bm = 128, bn = cfg == 1 ? 256 : (cfg == 2 ? 128 : 64);
    // too few tiles for one wave of blocks: 64-pixel x 128-filter tiles.  Measured against the tile above, over
    // reductions of 64 to 10000: 72 to 120 filters, 18 k to 48 k rows 0.88-1.01 (int8) and 0.83-0.93 (fp8) of its
    // time (3 x 3 over 128 channels, 32 k rows, 96 filters 11.5 / 10.3 -> 10.8 / 9.1 us).  Up to 64 filters half of
    // the waves work on filters that do not exist, which is faster only while a CU has one block: 33 to 64 filters
    // 0.86-0.97 and 0.86-0.96 at 9 k to 15 k rows (3 x 3 over 256 channels, 64 filters 13.0 / 11.0 -> 12.3 / 10.2),
    // 0.97-1.24 and 0.96-1.10 at 17 k to 25 k (13.0 / 11.0 -> 15.9 / 12.0); 16 to 64 1.06-1.30 and 1.01-1.28 beyond
    if (((M + bm - 1) / bm) * ((K + bn - 1) / bn) < 384 && (K > 64 || M <= 256 * 64)) cfg = 4;
    return cfg;
}

hipError_t launch_conv_i8_small(const ConvI8Args& a, int cfg, hipStream_t stream) {
    return launch_small8<false>(a, cfg, stream);
}

hipError_t launch_conv_fp8_small(const ConvFp8Args& a, int cfg, hipStream_t stream) {
    return launch_small8<true>(a, cfg, stream);
}

}  // namespace tbn
