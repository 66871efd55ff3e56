// tbn_conv_small.hip -- the same GEMM as tbn_conv_dma.hip (forward pass, Sec. 2 Eq. 1, and
// backward-data, Sec. 3) for layers with few output rows: one image, a small batch, a
// fully-connected layer.  Such a layer is a chain of latencies, not of work: on the tiled kernel
// a 14 x 14 x 256 layer at batch 1 is 8 tiles, so 8 of 256 CUs multiply nine stages one after the
// other, each behind a barrier, and a layer split over the grid adds a second launch.
//
//   * the block owns a tile of 32 pixels x 32 TN filters, small enough that even one image gives
//     tens of blocks; its W waves split the reduction (wave w takes stages w, w + W, ..), so
//     that a wave multiplies only a few 64-element stages;
//   * nothing is shared between waves: each has its own ring of S stages in LDS, filled by
//     LDS-DMA copies of whole 128-byte runs and waited for by that wave alone, so the loop has no
//     barrier.  (The same loop with operands loaded straight to registers, 32 bytes of 32 rows per
//     instruction, touched four times as many cache lines: 7.7 against 5.9 us on a 14 x 14 x 256 layer
//     at batch 1.)
//   * the waves' sums are added through LDS in wave order (deterministic), the epilogue's column
//     factors and residual having been requested before the loop.
#include "tbn_device.h"
#include "tbn_dma.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

constexpr int BK = 64;

struct SmallArgs {
    ConvGemmArgs g;
    FastDiv div_c, div_s;
};

// UNI: C % 64 == 0, a stage lies in one tap.
template <int TN, int W, int S, bool BWD, bool UNI>
__global__ __launch_bounds__(64 * W) void conv_small_kernel(const SmallArgs sa) {
    const ConvGemmArgs& a = sa.g;
    constexpr int BN = 32 * TN;
    constexpr int PITCH = BN + 4;                 // floats per pixel of a wave's sums
    constexpr int XB = 32 * 128;                  // a stage: 32 rows of 64 bf16, ..
    constexpr int CB = BN * 16;                   // .. the code words of BN filters, ..
    constexpr int STAGE = XB + 1024 + (BWD ? 256 : 0);  // .. and 32 scale pairs
    constexpr int RING = S * STAGE;
    constexpr int SUMS = W * 32 * PITCH * 4;
    static_assert(CB <= 1024, "one copy of codes per stage");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[W * RING > SUMS ? W * RING : SUMS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;

    const uint32_t PQ = (uint32_t)a.P * (uint32_t)a.Q;
    const uint32_t M = (uint32_t)a.N * PQ;
    const int C = a.C, Kf = a.Kf;
    const int n = a.R * a.S * C;
    const int nst = (n + BK - 1) / BK;
    const int KB = (Kf + 63) / 64;
    const uint32_t tilesN = (uint32_t)(Kf + BN - 1) / BN;
    const uint32_t tile = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t mt = fdiv(tile, a.div_tilesN);
    const uint32_t m0 = mt * 32;
    const int n0 = (int)(tile - mt * tilesN) * BN;

    const v4i rs_x = make_rsrc(a.x, (uint32_t)a.N * (uint32_t)a.H * (uint32_t)a.W * (uint32_t)C * 2u);
    const v4i rs_c = make_rsrc(a.codes, (uint32_t)KB * (uint32_t)nst * 1024u);
    v4i rs_p = rs_c;
    if constexpr (BWD) rs_p = make_rsrc(a.apair, (uint32_t)nst * 128u);
    uint8_t* const ring = smem + wave * RING;
    const uint32_t ring_base = lds_addr(ring);

    // ---- copies.  Instruction j fills rows 8 j + lane / 8 of a stage; a row's 16-byte segments are
    //      swizzled by (row / 2) % 8 (the operand reads of 16 rows then use every bank once) ----
    uint32_t rbase[4], rmask[4][2];  // as in the tiled kernel: (h0, w0) in x, taps inside the image
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
    // segment of the even (odd: ^ 4) instructions
    const int lseg = (lane & 7) ^ ((lane >> 4) & 3);
    const int f = n0 + (lane < BN ? lane : 0);
    const uint32_t c_lane = lane < BN && (f >> 6) < KB
                                ? (uint32_t)((f >> 6) * nst) * 1024u + (uint32_t)(f & 63) * 16u : 0x80000000u;

    auto issue = [&](int st, int slot) {
        const uint32_t base = ring_base + (uint32_t)(slot * STAGE);
        uint32_t toff[2];
        int tap[2];
        if constexpr (UNI) {
            const uint32_t e0 = (uint32_t)st * BK;  // scalar
            tap[0] = tap[1] = (int)fdiv(e0, sa.div_c);
            const int r = (int)fdiv((uint32_t)tap[0], sa.div_s);
            const uint32_t t0 = (uint32_t)((r * a.W + tap[0] - r * a.S) * C) + (e0 - (uint32_t)(tap[0] * C));
            toff[0] = t0 + 8u * (uint32_t)lseg;
            toff[1] = t0 + 8u * (uint32_t)(lseg ^ 4);
        } else {
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const uint32_t e = (uint32_t)st * BK + 8u * (uint32_t)(lseg ^ (4 * o));
                const uint32_t t = fdiv(e, sa.div_c);
                const uint32_t r = fdiv(t, sa.div_s);
                // taps past the filter clamp to bit 63, clear in rmask (R*S <= 63)
                tap[o] = (int)min(t, 63u);
                toff[o] = (r * (uint32_t)a.W + t - r * (uint32_t)a.S) * (uint32_t)C + (e - t * (uint32_t)C);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = UNI ? min(tap[0], 63) : tap[j & 1];
            const uint32_t bits = t >= 32 ? rmask[j][1] : rmask[j][0];
            const bool ok = (bits >> (t & 31)) & 1u;
            dma_b128(rs_x, base + (uint32_t)(1024 * j), ok ? (rbase[j] + toff[j & 1]) << 1 : 0x80000000u);
        }
        dma_b128(rs_c, base + XB, c_lane + (uint32_t)st * 1024u);
        if constexpr (BWD) dma_b32(rs_p, base + XB + 1024, lane < 32 ? (uint32_t)(st * 128 + lane * 4) : 0x80000000u);
    };
    constexpr int DMAS = 4 + 1 + (BWD ? 1 : 0);

    // ---- epilogue operands of this thread (4 channels of one pixel), requested now ----
    constexpr int GROUPS = BN / 4;             // per pixel
    constexpr int EPT = (32 * GROUPS + 64 * W - 1) / (64 * W);  // groups per thread
    float cs[EPT][4], bi[EPT][4], rs[EPT][4];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int gi = tid + 64 * W * e;
        const int col0 = n0 + 4 * (gi % GROUPS);
        const uint32_t row = m0 + (uint32_t)(gi / GROUPS);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = col0 + j < Kf ? col0 + j : Kf - 1;  // past Kf: never stored
            cs[e][j] = a.colscale ? a.colscale[col] : 1.0f;
            if (a.scale) cs[e][j] *= a.scale[col];
            bi[e][j] = a.bias ? a.bias[col] : 0.0f;
            rs[e][j] = 0.0f;
        }
        if (a.residual && gi < 32 * GROUPS && row < M) {
            const int64_t o = (int64_t)row * Kf + col0;
            if (!a.y_f32 && Kf % 4 == 0) {
                if (col0 < Kf) {
                    const u32x2 r = *reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(a.residual) + o);
                    rs[e][0] = bf16_bits_to_f32(r.x & 0xFFFFu);
                    rs[e][1] = bf16_bits_to_f32(r.x >> 16);
                    rs[e][2] = bf16_bits_to_f32(r.y & 0xFFFFu);
                    rs[e][3] = bf16_bits_to_f32(r.y >> 16);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (col0 + j < Kf)
                        rs[e][j] = a.y_f32 ? reinterpret_cast<const float*>(a.residual)[o + j]
                                           : bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(a.residual)[o + j]);
            }
        }
    }

    f32x16 acc[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
    const int cnt = nst > wave ? (nst - wave + W - 1) / W : 0;  // this wave's stages
#pragma unroll
    for (int i = 0; i < S; ++i)
        if (i < cnt) issue(wave + W * i, i);
    const uint8_t* const arow = ring + l32 * 128;
    const int sw = (l32 >> 1) & 7;
    int slot = 0;
    for (int i = 0; i < cnt; ++i) {
        // stages up to i + S - 1 are in flight
        if (i + S <= cnt)
            wait_vmcnt((S - 1) * DMAS);
        else
            wait_vmcnt(0);
        asm volatile("" ::: "memory");
        const int so = slot * STAGE;
        u32x4 x[4], c[TN], sc[BWD ? 4 : 1];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const u32x4*>(arow + so + 16 * ((2 * u + half) ^ sw));
#pragma unroll
        for (int t = 0; t < TN; ++t) c[t] = *reinterpret_cast<const u32x4*>(ring + so + XB + 16 * (32 * t + l32));
        if constexpr (BWD) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                sc[u] = *reinterpret_cast<const u32x4*>(ring + so + XB + 1024 + 32 * u + 16 * half);
        }
        if (i + S < cnt) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the slot is read before it is refilled
            issue(wave + W * (i + S), slot);
        }
        slot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            u32x4 base = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
            if constexpr (BWD) base = sc[u];
#pragma unroll
            for (int t = 0; t < TN; ++t)
                acc[t] = mfma32(as_bf16x8(decode8(c[t][u] >> (4 * half), base)), as_bf16x8(x[u]), acc[t]);
        }
    }

    // ---- the waves' sums: lane holds pixel l32 and, per v / 4, four consecutive filters ----
    __syncthreads();  // the sums lie over the rings
    float* const sums = reinterpret_cast<float*>(smem);
    float* const mine = sums + (wave * 32 + l32) * PITCH;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4*>(mine + 32 * t + 8 * g + 4 * half) =
                f32x4{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int gi = tid + 64 * W * e;
        const int pix = gi / GROUPS;
        const uint32_t row = m0 + (uint32_t)pix;
        const int col0 = n0 + 4 * (gi % GROUPS);
        if (gi >= 32 * GROUPS || row >= M || col0 >= Kf) continue;
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < W; ++w)
            s += *reinterpret_cast<const f32x4*>(sums + (w * 32 + pix) * PITCH + 4 * (gi % GROUPS));
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = s[j] * cs[e][j] + bi[e][j] + rs[e][j];
            if (a.relu) v[j] = fmaxf(v[j], 0.0f);
        }
        const int64_t o = (int64_t)row * Kf + col0;
        if (Kf % 4 == 0) {
            if (a.y_f32)
                *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.y) + o) = f32x4{v[0], v[1], v[2], v[3]};
            else
                *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(a.y) + o) =
                    u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (col0 + j >= Kf) break;
                if (a.y_f32)
                    reinterpret_cast<float*>(a.y)[o + j] = v[j];
                else
                    reinterpret_cast<uint16_t*>(a.y)[o + j] = (uint16_t)f32_to_bf16_bits(v[j]);
            }
        }
    }
}

template <int TN, int W, int S>
hipError_t launch_cfg(const SmallArgs& args, hipStream_t stream) {
    SmallArgs a = args;
    const int64_t M = (int64_t)a.g.N * a.g.P * a.g.Q;
    const int64_t tilesN = (a.g.Kf + 32 * TN - 1) / (32 * TN);
    const int64_t tiles = ((M + 31) / 32) * tilesN;
    if (tiles >= 0x7FFFFFFFll) return hipErrorInvalidValue;
    a.g.div_tilesN = make_fastdiv((uint32_t)tilesN);
    const dim3 grid((unsigned)tiles), block(64 * W);
    const bool uni = a.g.C % 64 == 0;
    if (a.g.apair) {
        if (uni)
            hipLaunchKernelGGL((conv_small_kernel<TN, W, S, true, true>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((conv_small_kernel<TN, W, S, true, false>), grid, block, 0, stream, a);
    } else {
        if (uni)
            hipLaunchKernelGGL((conv_small_kernel<TN, W, S, false, true>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((conv_small_kernel<TN, W, S, false, false>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace

// Measured against the tiled kernel (forward with the whole epilogue, graph-replayed, us; b1 and b2
// are the blocks with tiles of 32 and 64 filters):
//   b1 <= 256 (a block per CU): 56 x 56 x 64 at batch 1 7.3 -> 4.7, 28 x 28 x 128 9.0 -> 5.0, 14 x 14 x 256
//     12.5 -> 5.9, 7 x 7 x 512 12.6 -> 7.8, 64 rows of 512 -> 1000 8.4 -> 4.3, 128 rows of 8192 -> 10 12.5 ->
//     10.5.  Eight waves, four where eight would have a stage or less each, sixteen (whose rings hold one
//     stage) from 72 stages on: 48 stages 7.1 with eight, 7.4 with sixteen, 64 to 90 equal, 126 (14 x 14 x 896)
//     11.2 and 10.6, 200 14.2 and 12.5.
//   b1 <= 512: four waves, two blocks per CU: 56 x 56 x 64 at batch 2 7.3 -> 5.4, 40 x 40 x 16 5 x 5 at
//     batch 9 10.1 -> 5.0; from 24 stages on 64 filters and eight waves if that is at most a block
//     per CU (7 x 7 x 512 at batch 16: 18.7 -> 10.8, against 12.0).
//   b1 <= 1024: only where the tiled kernel splits its reduction over the grid (an epilogue pass of
//     its own): 16 x 16 x 96 at batch 25 16.2 -> 8.8, 52 x 78 x 96 at batch 2 17.2 -> 8.8; otherwise the
//     tiled kernel is as fast or faster (28 x 28 x 128 at batch 6 9.3 against 9.4, 56 x 56 x 64 at batch
//     4 7.5 against 7.9).  Four waves, 64 filters a tile from 24 stages on: 14 stages (the two above) 9.2 with
//     32 filters, 9.5 with 64, 24 (1 x 1 x 1536 -> 72) equal, 36 (14 x 14 x 256 -> 96 at batch 30) 12.8 and 12.4,
//     128 (100 rows of 8192 -> 8000) 36.3 and 30.4.
// Reductions beyond 200 stages stay on the tiled kernel, which spreads them over the grid.
int conv_small_cfg(const ConvGemmArgs& a, int cfg) {
    if (cfg >= 51 && cfg <= 55) return cfg;
    if (cfg >= 0 || conv_splits_override() > 0) return 0;
    const int64_t M = (int64_t)a.N * a.P * a.Q, rows = (M + 31) / 32;
    const int64_t b1 = rows * ((a.Kf + 31) / 32), b2 = rows * ((a.Kf + 63) / 64);
    const int64_t nst = ((int64_t)a.R * a.S * a.C + BK - 1) / BK;
    if (b1 > 1024 || nst > 200) return 0;
    if (b1 <= 256) return nst <= 8 ? 51 : nst < 72 ? 52 : 53;
    if (b1 <= 512) return nst >= 24 && b2 <= 256 ? 55 : 51;
    if (plan_conv_dma(a, cfg).splits <= 1) return 0;
    return nst >= 24 ? 54 : 51;
}

hipError_t launch_conv_small(const ConvGemmArgs& g, int cfg, hipStream_t stream) {
    SmallArgs a;
    a.g = g;
    a.div_c = make_fastdiv((uint32_t)g.C);
    a.div_s = make_fastdiv((uint32_t)g.S);
    uint64_t rep = 0;
    for (int r = 0; r < g.R; ++r) rep |= 1ull << (r * g.S);
    a.g.rep_lo = (uint32_t)rep;
    a.g.rep_hi = (uint32_t)(rep >> 32);
    switch (cfg) {
        case 51: return launch_cfg<1, 4, 3>(a, stream);
        case 52: return launch_cfg<1, 8, 3>(a, stream);
        case 53: return launch_cfg<1, 16, 1>(a, stream);
        case 54: return launch_cfg<2, 4, 3>(a, stream);
        default: return launch_cfg<2, 8, 3>(a, stream);
    }
}

}  // namespace tbn
