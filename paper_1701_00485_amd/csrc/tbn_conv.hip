// tbn_conv.hip -- implicit-GEMM convolution on bf16 MFMA with the two-bit filters decoded
// in registers.  One kernel template serves
//   * the forward pass (Sec. 2 Eq. 1; Algorithm 1 forward step): rows = output pixels
//     (n,p,q), columns = filters k, reduction = filter elements (r,s,c); every code is
//     decoded to an exact bf16 +-1/+-2 and alpha_k is applied to the fp32 sum; and
//   * the backward-data pass (Sec. 3, backward through the approximate filters): the
//     same GEMM over dy with the transposed, spatially flipped filter, whose codes are
//     decoded straight into bf16(alpha_k) * W~ (sign flip / exponent + 1 of the scale).
//
// Work split (256 threads = 4 waves of 64, CDNA4):
//   * the block owns a BM x BN output tile; each wave a WM x WN sub-tile made of 32x32
//     v_mfma_f32_32x32x16_bf16 tiles with fp32 accumulators;
//   * the reduction advances 64 elements per stage, which is exactly one 1 KiB block of
//     packed codes per 64 filters;
//   * the activation tile (BM rows x 64 elements, bf16) is gathered from NHWC memory
//     (zero padding by predication) into LDS, double buffered, rows padded by 8 bf16 so
//     the 16-byte MFMA operand reads do not conflict;
//   * the filter operand never touches LDS: lane l of a wave loads the four words of
//     filter (l % 32) of its 32-column group (one coalesced 16-byte load per lane, 512
//     bytes per wave) and decodes at each 16-element MFMA step the 8 elements the MFMA
//     B layout gives it (elements 8*(l/32)..+7 of the step) with 2 integer ops per pair.
#include <cstdlib>

#include "tbn_device.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

constexpr int BK = 64;       // reduction elements per stage
constexpr int LDA = BK + 8;  // LDS row pitch (bf16 elements)

enum { A_VEC8 = 0, A_SCALAR = 1 };

template <int BM, int BN, int WM, int WN, int AM, bool BWD>
__global__ __launch_bounds__(256) void conv_gemm_kernel(const ConvGemmArgs a) {
    constexpr int WAVES_N = BN / WN;
    static_assert((BM / WM) * (BN / WN) == 4, "four waves per block");
    constexpr int TM = WM / 32, TN = WN / 32;

    __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * LDA];
    // Row table of the scalar gather: image offset and top-left input coordinate.
    __shared__ int64_t row_img[AM == A_SCALAR ? BM : 1];
    __shared__ int32_t row_h[AM == A_SCALAR ? BM : 1];
    __shared__ int32_t row_w[AM == A_SCALAR ? BM : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WAVES_N;
    const int wn = wave % WAVES_N;
    const int half = lane >> 5;  // which 8 of a 16-element MFMA step this lane holds
    const int l32 = lane & 31;

    const int64_t PQ = (int64_t)a.P * a.Q;
    const int64_t M = (int64_t)a.N * PQ;
    const int C = a.C;
    const int n = a.R * a.S * C;
    const int nchunks = (n + BK - 1) / BK;
    const int KB = (a.Kf + 63) / 64;
    const int tilesN = (a.Kf + BN - 1) / BN;
    // XCD-aware order: each XCD runs a contiguous range of tiles (column tiles of one row
    // tile first), so the activation rows and halos a tile re-reads stay in one L2.
    const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t tm = tile / tilesN;
    const int tn = (int)(tile % tilesN);
    const int64_t m0 = tm * BM;
    const int n0 = tn * BN;
    const int64_t HWC = (int64_t)a.H * a.W * C;

    // ---------------- activation gather state ----------------
    constexpr int AR = (AM == A_VEC8) ? BM / 32 : BM / 4;  // rows per thread
    const int seg = tid & 7;        // A_VEC8: 16-byte segment of the 64-element row
    const int vrow = tid >> 3;      // A_VEC8: first row
    const int sel = tid & 63;       // A_SCALAR: element of the chunk
    const int srow = tid >> 6;      // A_SCALAR: first row
    int32_t rh[AM == A_VEC8 ? AR : 1], rw[AM == A_VEC8 ? AR : 1];
    int64_t rimg[AM == A_VEC8 ? AR : 1];
    if constexpr (AM == A_VEC8) {
#pragma unroll
        for (int j = 0; j < AR; ++j) {
            const int64_t m = m0 + vrow + 32 * j;
            if (m < M) {
                const int64_t img = m / PQ;
                const int pq = (int)(m - img * PQ);
                const int p = pq / a.Q, q = pq - (pq / a.Q) * a.Q;
                rimg[j] = img * HWC;
                rh[j] = p * a.sh - a.ph;
                rw[j] = q * a.sw - a.pw;
            } else {
                rimg[j] = 0;
                rh[j] = -0x40000000;  // never inside the image
                rw[j] = -0x40000000;
            }
        }
    } else {
        for (int r = tid; r < BM; r += 256) {
            const int64_t m = m0 + r;
            if (m < M) {
                const int64_t img = m / PQ;
                const int pq = (int)(m - img * PQ);
                const int p = pq / a.Q, q = pq - (pq / a.Q) * a.Q;
                row_img[r] = img * HWC;
                row_h[r] = p * a.sh - a.ph;
                row_w[r] = q * a.sw - a.pw;
            } else {
                row_img[r] = 0;
                row_h[r] = -0x40000000;
                row_w[r] = -0x40000000;
            }
        }
        __syncthreads();
    }
    // (r, s, c) of this thread's first element in the current chunk (A_VEC8)
    int er = 0, es = 0, ec = 0;
    if constexpr (AM == A_VEC8) {
        const int e0 = seg * 8;
        const int rs = e0 / C;
        ec = e0 - rs * C;
        er = rs / a.S;
        es = rs - er * a.S;
    }

    u32x4 areg[AM == A_VEC8 ? AR : 1];
    uint16_t sreg[AM == A_SCALAR ? AR : 1];

    auto load_a = [&](int chunk) {
        if constexpr (AM == A_VEC8) {
            const uint16_t* x = reinterpret_cast<const uint16_t*>(a.x);
#pragma unroll
            for (int j = 0; j < AR; ++j) {
                u32x4 v = {0u, 0u, 0u, 0u};
                const int h = rh[j] + er, w = rw[j] + es;
                if (er < a.R && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W)
                    v = *reinterpret_cast<const u32x4*>(x + rimg[j] + ((int64_t)h * a.W + w) * C + ec);
                areg[j] = v;
            }
        } else {
            const int e = chunk * BK + sel;
            int r = 0, s = 0, c = 0;
            const bool ok = e < n;
            if (ok) {
                const int rs = e / C;
                c = e - rs * C;
                r = rs / a.S;
                s = rs - r * a.S;
            }
#pragma unroll 4
            for (int j = 0; j < AR; ++j) {
                const int row = srow + 4 * j;
                uint16_t v = 0;
                const int h = row_h[row] + r, w = row_w[row] + s;
                if (ok && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W) {
                    const int64_t off = row_img[row] + ((int64_t)h * a.W + w) * C + c;
                    if (a.x_f32)
                        v = (uint16_t)f32_to_bf16_bits(reinterpret_cast<const float*>(a.x)[off]);
                    else
                        v = reinterpret_cast<const uint16_t*>(a.x)[off];
                }
                sreg[j] = v;
            }
        }
    };
    auto advance_a = [&]() {
        if constexpr (AM == A_VEC8) {
            ec += BK;
            while (ec >= C) {
                ec -= C;
                if (++es == a.S) {
                    es = 0;
                    ++er;
                }
            }
        }
    };
    auto store_a = [&](int buf) {
        if constexpr (AM == A_VEC8) {
#pragma unroll
            for (int j = 0; j < AR; ++j)
                *reinterpret_cast<u32x4*>(&As[buf][(vrow + 32 * j) * LDA + seg * 8]) = areg[j];
        } else {
#pragma unroll
            for (int j = 0; j < AR; ++j) As[buf][(srow + 4 * j) * LDA + sel] = sreg[j];
        }
    };

    // ---------------- filter operand state ----------------
    u32x4 braw[TN];
    u32x4 bnext[TN];
    u32x4 base[4];
    u32x4 base_next[4];
    auto load_b = [&](int chunk, u32x4* dst, u32x4* bdst) {
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const int f = n0 + wn * WN + 32 * t + l32;
            const int fb = f >> 6;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (fb < KB)
                v = *reinterpret_cast<const u32x4*>(a.codes + (((int64_t)fb * nchunks + chunk) * 64 + (f & 63)) * 4);
            dst[t] = v;
        }
        if constexpr (BWD) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                bdst[u] = *reinterpret_cast<const u32x4*>(a.apair + (int64_t)chunk * 32 + 8 * u + 4 * half);
        }
    };
    if constexpr (!BWD) {
#pragma unroll
        for (int u = 0; u < 4; ++u) base[u] = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.0f;

    // ---------------- main loop ----------------
    load_a(0);
    load_b(0, braw, base);
    store_a(0);
    __syncthreads();
    for (int chunk = 0; chunk < nchunks; ++chunk) {
        const int cur = chunk & 1;
        const bool more = chunk + 1 < nchunks;
        if (more) {
            advance_a();
            load_a(chunk + 1);
            load_b(chunk + 1, bnext, base_next);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bf16x8 af[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *reinterpret_cast<const bf16x8*>(
                    &As[cur][(wm * WM + 32 * i + l32) * LDA + 16 * u + 8 * half]);
            bf16x8 bfr[TN];
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const uint32_t wd = braw[t][u] >> (4 * half);
                bfr[t] = as_bf16x8(decode8(wd, base[u]));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[i][t] = mfma32(af[i], bfr[t], acc[i][t]);
        }
        if (more) {
            store_a(cur ^ 1);
#pragma unroll
            for (int t = 0; t < TN; ++t) braw[t] = bnext[t];
            if constexpr (BWD) {
#pragma unroll
                for (int u = 0; u < 4; ++u) base[u] = base_next[u];
            }
        }
        __syncthreads();
    }

    // ---------------- epilogue ----------------
    const int Kf = a.Kf;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int col = n0 + wn * WN + 32 * t + l32;
        if (col >= Kf) continue;
        float cs = a.colscale ? a.colscale[col] : 1.0f;
        if (a.scale) cs *= a.scale[col];
        const float bi = a.bias ? a.bias[col] : 0.0f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t row = m0 + wm * WM + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row >= M) continue;
                const int64_t o = row * Kf + col;
                float val = acc[i][t][v] * cs + bi;
                if (a.residual) {
                    val += a.y_f32 ? reinterpret_cast<const float*>(a.residual)[o]
                                   : bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(a.residual)[o]);
                }
                if (a.relu) val = fmaxf(val, 0.0f);
                if (a.y_f32)
                    reinterpret_cast<float*>(a.y)[o] = val;
                else
                    reinterpret_cast<uint16_t*>(a.y)[o] = (uint16_t)f32_to_bf16_bits(val);
            }
        }
    }
}

template <int BM, int BN, int WM, int WN, int AM, bool BWD>
hipError_t launch_cfg(const ConvGemmArgs& a, hipStream_t stream) {
    const int64_t M = (int64_t)a.N * a.P * a.Q;
    const int64_t tiles = ((M + BM - 1) / BM) * ((a.Kf + BN - 1) / BN);
    if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL((conv_gemm_kernel<BM, BN, WM, WN, AM, BWD>), dim3((unsigned)tiles), dim3(256), 0,
                       stream, a);
    return hipGetLastError();
}


template <int AM, bool BWD>
hipError_t launch_mode(const ConvGemmArgs& a, int cfg, hipStream_t stream) {
    if (cfg == 1 || (cfg < 0 && a.Kf <= 64)) return launch_cfg<256, 64, 64, 64, AM, BWD>(a, stream);
    return launch_cfg<128, 128, 64, 64, AM, BWD>(a, stream);
}

}  // namespace

// Tile-shape and split overrides for tuning and for the tests that cover every shape (the
// knobs of tbn_tuning.h; -1 = the built-in choice).
int conv_tile_override() { return knob(KNOB_CONV_TILE); }

int conv_splits_override() { return knob(KNOB_CONV_SPLITS); }

// Which kernel runs a forward / backward-data GEMM: the weight-streaming kernel for a
// fully-connected layer of at most 16 rows, for C % 8 == 0 the small-layer kernel where there
// are few output tiles and the LDS-DMA implicit GEMM elsewhere, the direct kernel for small
// few-channel layers, the thin-input kernel for other few-channel ones, else the general one.
// cfg (the tile knob) forces a family: 0-1 general, 10-19 and 21-25 LDS-DMA tile shapes, 20 thin,
// 30 weight streaming, 40 direct, 51-55 small-layer shapes, 60 3 x 3 over 64 channels.
enum ConvPath { PATH_FC, PATH_SMALL, PATH_C64, PATH_DMA, PATH_DIRECT, PATH_THIN, PATH_GENERIC };

static ConvPath choose_path(const ConvGemmArgs& a, int cfg, FcStreamPlan* fp, ThinGeom* tg) {
    if ((cfg < 0 || cfg == 30) && fc_stream_plan(a, fp)) return PATH_FC;
    if (conv_dma_eligible(a) && conv_small_cfg(a, cfg)) return PATH_SMALL;
    if (conv_dma_eligible(a) && conv_c64_chosen(a, cfg)) return PATH_C64;
    if (conv_dma_eligible(a) && (cfg < 0 || (cfg >= 10 && cfg < 20) || (cfg >= 21 && cfg <= 25))) return PATH_DMA;
    if ((cfg < 0 || cfg == 40) && conv_direct_eligible(a)) return PATH_DIRECT;
    if ((cfg < 0 || cfg == 20) && conv_thin_plan(a, tg)) return PATH_THIN;
    return PATH_GENERIC;
}

size_t conv_gemm_partial_bytes(const ConvGemmArgs& a) {
    const int cfg = conv_tile_override();
    FcStreamPlan fp;
    ThinGeom tg;
    switch (choose_path(a, cfg, &fp, &tg)) {
        case PATH_DMA: return plan_conv_dma(a, cfg).partial_bytes;
        // these use none: what the tiled kernel asks for in their place, so that a layer's workspace
        // does not depend on which of them runs it
        case PATH_SMALL:
        case PATH_C64: return cfg < 0 ? plan_conv_dma(a, cfg).partial_bytes : 0;
        case PATH_THIN: return tg.dma ? (size_t)tg.ws_bytes : 0;
        default: return 0;
    }
}

size_t conv_gemm_split_bytes(const ConvGemmArgs& a) {
    const int cfg = conv_tile_override();
    FcStreamPlan fp;
    ThinGeom tg;
    return choose_path(a, cfg, &fp, &tg) == PATH_DMA ? plan_conv_dma(a, cfg).partial_bytes : 0;
}

bool conv_pool_plan(const ConvGemmArgs& a, ThinGeom* g) {
    FcStreamPlan fp;
    return choose_path(a, conv_tile_override(), &fp, g) == PATH_THIN && conv_thin_pool_plan(a, g);
}

static ConvGemmArgs padded_args(const ConvGemmArgs& a, int32_t Cp) {
    ConvGemmArgs b = a;
    b.C = Cp;
    b.x_f32 = 0;
    return b;
}

// C % 8 != 0 beyond the few-channel kernels: two launches (the copies, then the LDS-DMA
// kernel) instead of the general kernel's one, and faster at every size tried (graph-replayed,
// general -> padded): 1 x 1 x 20 -> 32 filters 14.2 -> 5.4 us, 14 x 14 x 100 -> 100 3 x 3 at batch 1
// 205 -> 12.9 us, 50 x 27 x 27 x 36 -> 100 3 x 3 130 -> 21.3 us, 64 rows of 3001 -> 500 611 -> 12.6 us
// (the general kernel gathers 2-byte elements with a division and a bounds test each).
bool conv_pad_plan(const ConvGemmArgs& a, ConvPadPlan* p) {
    const int cfg = conv_tile_override();
    FcStreamPlan fp;
    ThinGeom tg;
    if (a.apair || cfg >= 0 || a.C % 8 == 0 || choose_path(a, cfg, &fp, &tg) != PATH_GENERIC) return false;
    const int64_t Cp = ((int64_t)a.C + 7) / 8 * 8;
    if ((int64_t)a.R * a.S * Cp >= (1 << 30)) return false;
    const ConvGemmArgs b = padded_args(a, (int32_t)Cp);
    if (!conv_dma_eligible(b)) return false;
    p->Cp = (int32_t)Cp;
    const int64_t xb = (int64_t)a.N * a.H * a.W * Cp * 2;
    p->codes_off = (xb + 255) / 256 * 256;
    const int64_t cb = (int64_t)((a.Kf + 63) / 64) * (((int64_t)a.R * a.S * Cp + 63) / 64) * 1024;
    p->partial_off = p->codes_off + cb;
    p->total = p->partial_off + (int64_t)plan_conv_dma(b, cfg).partial_bytes;
    return true;
}

hipError_t launch_conv_padded(const ConvGemmArgs& a, const ConvPadPlan& p, void* ws, hipStream_t stream) {
    uint8_t* const base = reinterpret_cast<uint8_t*>(ws);
    uint32_t* const codes_p = reinterpret_cast<uint32_t*>(base + p.codes_off);
    hipError_t e = launch_pad_fwd(make_pad(a.x, (int64_t)a.N * a.H * a.W, a.C, p.Cp, base), a.x_f32, a.codes, a.Kf,
                                  a.R * a.S, codes_p, stream);
    if (e != hipSuccess) return e;
    ConvGemmArgs b = padded_args(a, p.Cp);
    b.x = base;
    b.codes = codes_p;
    b.partial = reinterpret_cast<float*>(base + p.partial_off);
    return launch_conv_gemm(b, stream);
}

hipError_t launch_conv_gemm(const ConvGemmArgs& args, hipStream_t stream) {
    ConvGemmArgs a = args;
    a.div_q = make_fastdiv((uint32_t)a.Q);
    a.div_pq = make_fastdiv((uint32_t)a.P * (uint32_t)a.Q);
    a.splits = 1;
    a.chunks_per_split = 1 << 30;
    const int cfg = conv_tile_override();
    FcStreamPlan fp;
    ThinGeom tg;
    switch (choose_path(a, cfg, &fp, &tg)) {
        case PATH_FC: return launch_fc_stream(a, fp, stream);
        case PATH_SMALL: return launch_conv_small(a, conv_small_cfg(a, cfg), stream);
        case PATH_C64: return launch_conv_c64(a, stream);
        case PATH_DMA: return launch_conv_dma(a, plan_conv_dma(a, cfg), stream);
        case PATH_DIRECT: return launch_conv_direct(a, stream);
        case PATH_THIN: return launch_conv_thin(a, tg, stream);
        default: break;
    }
    const bool vec = (a.C % 8 == 0) && !a.x_f32;
    if (a.apair) return vec ? launch_mode<A_VEC8, true>(a, cfg, stream) : launch_mode<A_SCALAR, true>(a, cfg, stream);
    return vec ? launch_mode<A_VEC8, false>(a, cfg, stream) : launch_mode<A_SCALAR, false>(a, cfg, stream);
}

}  // namespace tbn
