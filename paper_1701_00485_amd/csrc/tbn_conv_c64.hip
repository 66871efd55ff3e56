// tbn_conv_c64.hip -- the same GEMM as tbn_conv_dma.hip (forward pass, Sec. 2 Eq. 1, and
// backward-data, Sec. 3) for 3 x 3 layers of stride 1 over 64 channels with many output pixels.  Their
// reduction is short (nine 64-element stages), so on the tiled kernel every tile decodes its filters
// again, copies every input pixel nine times, waits at nine barriers, and multiplies little per
// decoded word: 56 x 56 x 64 -> 64 at batch 64 takes 26.8 us against the 7 us of its matrix work.
//
//   * a wave keeps 32 decoded filters in registers (36 operands of 4 registers) for as long as it
//     lives, so nothing is decoded in the loop;
//   * it walks over units of 4 x 8 output pixels.  A unit's input patch (6 x 10 pixels of 128 bytes)
//     is copied once, by eight LDS-DMA instructions, into one of two slots that belong to the wave
//     alone, the next unit's while this one is multiplied; the nine taps read it at shifted rows;
//   * no barriers: a unit is 36 LDS reads of 16 bytes a lane and 36 MFMAs, then the sums turn
//     through 4.5 KB of LDS into 16-byte pieces of output rows;
//   * two waves share a SIMD (two blocks a CU, 160 KB of LDS), so that one multiplies while the other
//     stores its outputs.
// What bounds it: the matrix work and the other instructions of its two waves (each unit 1152 clocks of
// MFMAs and about 120 vector and 110 scalar instructions); without the copies, the stores or the epilogue it
// runs as long.  At 56 x 56 x 64 -> 64, batch 64, 26.8 -> 21.4 us (690 TFLOP/s), of which 7 us are one unit a
// wave: launch, first copies, decoding.  Read depths of 6 or 8, two accumulators in turn and raised
// wave priority were each 1.5 us slower, one block a CU 4 us.
#include <type_traits>

#include "tbn_device.h"
#include "tbn_dma.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

constexpr int C64 = 64;                    // channels
constexpr int TAPS = 9;
constexpr int UP = 4, UQ = 8;              // output pixels of a unit
constexpr int PR = UP + 2, PC = UQ + 2;    // its input patch
constexpr int SLOT = PR * PC * 128;        // bytes
constexpr int PITCH = 36;                  // floats per pixel of the sums (16-byte rows, banks spread)
constexpr int FAC = 2 * SLOT + UP * UQ * PITCH * 4;  // factors and biases of the 32 filters
constexpr int WAVE_LDS = FAC + 256;

struct C64Args {
    ConvGemmArgs g;
    FastDiv div_upi, div_tq;  // units per image, unit columns
    int32_t tiles_p, tiles_q;
    uint32_t units;
    int32_t fgroups;          // groups of 32 filters
    int32_t per;              // waves per group
};

template <bool BWD, bool RES>
__global__ __launch_bounds__(256, 2) void conv_c64_kernel(const C64Args ka) {
    const ConvGemmArgs& a = ka.g;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[4 * WAVE_LDS];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int H = a.H, W = a.W, Kf = a.Kf;

    // the wave's filters and its contiguous range of units
    const uint32_t wid = (uint32_t)xcd_remap(blockIdx.x, gridDim.x) * 4u + (uint32_t)wave;
    const uint32_t fg = wid % (uint32_t)ka.fgroups, wj = wid / (uint32_t)ka.fgroups;
    if (wj >= (uint32_t)ka.per) return;
    const uint32_t ubeg = (uint32_t)((uint64_t)ka.units * wj / (uint32_t)ka.per);
    const uint32_t uend = (uint32_t)((uint64_t)ka.units * (wj + 1) / (uint32_t)ka.per);
    if (ubeg >= uend) return;
    const int n0 = (int)fg * 32;

    const uint32_t M = (uint32_t)a.N * (uint32_t)a.P * (uint32_t)a.Q;
    const v4i rs_x = make_rsrc(a.x, (uint32_t)a.N * (uint32_t)H * (uint32_t)W * 128u);
    const __amdgpu_buffer_rsrc_t rs_y =
        __builtin_amdgcn_make_buffer_rsrc(a.y, 0, (int)(M * (uint32_t)Kf * 2u), 0x00020000);
    __amdgpu_buffer_rsrc_t rs_r = rs_y;
    if constexpr (RES)
        rs_r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.residual), 0, (int)(M * (uint32_t)Kf * 2u), 0x00020000);
    const int wbase = wave * WAVE_LDS;
    float* const sums = reinterpret_cast<float*>(smem + wbase + 2 * SLOT);
    const float* const fac = reinterpret_cast<const float*>(smem + wbase + FAC);
    const uint32_t ring_base = lds_addr(smem) + (uint32_t)wbase;

    // ---- copies: instruction j fills patch pixels 8 j .. 8 j + 7 (row-major, PC a row), lane i the
    //      16-byte segment i % 8 of pixel 8 j + i / 8.  Segments are swizzled by the pixel's column pair
    //      and row parity, so that the 16 lanes that read together use every bank once ----
    uint32_t loff[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int pp = 8 * j + (lane >> 3), pr = pp / PC, pc = pp - pr * PC;
        const int seg = (lane & 7) ^ (((pc >> 1) & 3) | ((pr & 1) << 2));
        loff[j] = (uint32_t)((pr * W + pc) * 128 + 16 * seg);
    }
    struct Unit {
        uint32_t img;
        int p, q;  // first output pixel
    };
    auto locate = [&](uint32_t u) {
        Unit t;
        t.img = fdiv(u, ka.div_upi);
        const uint32_t rem = u - t.img * (uint32_t)(ka.tiles_p * ka.tiles_q);
        const uint32_t tp = fdiv(rem, ka.div_tq);
        t.p = (int)tp * UP;
        t.q = (int)(rem - tp * (uint32_t)ka.tiles_q) * UQ;
        return t;
    };
    // Bits of a count of `n` positions from `first` on that lie in [0, size) (n <= 10; scalar)
    auto inside = [](int first, int n, int size) {
        const int lo = max(0, -first), hi = min(n, size - first);
        return hi > lo ? (1u << hi) - (1u << lo) : 0u;
    };
    // The masks of pixels outside the image (or past the range) are scalar; a lane moves its pixel's bit
    // to bit 31 of its offset, which puts it out of the buffer: two vector instructions a copy and no
    // branch, where tests of row and column took six.
    const uint32_t sh8 = 7u - (uint32_t)(lane >> 3);
    const uint32_t oob = 0x80000000u;
    auto issue = [&](uint32_t u, const Unit& t, int slot) {
        const int h0 = t.p - a.ph, w0 = t.q - a.pw;
        const uint32_t base = (uint32_t)((((int32_t)t.img * H + h0) * W + w0) * 128);
        const uint32_t rows = u < uend ? inside(h0, PR, H) : 0u;
        const uint64_t cols = inside(w0, PC, W);
        uint64_t in = 0;
#pragma unroll
        for (int r = 0; r < PR; ++r) in |= (rows >> r) & 1u ? cols << (PC * r) : 0ull;
        const uint32_t out[2] = {~(uint32_t)in, ~(uint32_t)(in >> 32)};
        const uint32_t dst = ring_base + (uint32_t)(slot * SLOT);
        // always eight copies, so that the waits are constants
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t byte = out[j >> 2] << (24 - 8 * (j & 3));  // pixels 8 j .. 8 j + 7 in bits 24 .. 31
            const uint32_t off = ((byte << sh8) & oob) | (loff[j] + base);
            if (j < 7 || lane < 32) dma_b128(rs_x, dst + 1024u * (uint32_t)j, off);  // 60 pixels
        }
    };
    Unit cur = locate(ubeg), nxt = locate(ubeg + 1 < uend ? ubeg + 1 : ubeg);
    issue(ubeg, cur, 0);
    issue(ubeg + 1, nxt, 1);
    static_assert(PR * PC == 60 && PC == 10, "eight copies, the last of four pixels");

    // ---- the filters, decoded: wf[4 t + u] holds elements 16 u + 8 half .. + 7 of tap t of filter l32 ----
    bf16x8 wf[4 * TAPS];
    {
        const int f = n0 + l32;
        const u32x4* cw = reinterpret_cast<const u32x4*>(a.codes) + ((int64_t)(f >> 6) * TAPS * 64 + (f & 63));
        u32x4 c[TAPS];
#pragma unroll
        for (int t = 0; t < TAPS; ++t) c[t] = cw[t * 64];
        u32x4 base[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            base[u] = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
            // the scale pairs depend on the channel alone, so they are the same for every tap
            if constexpr (BWD) base[u] = *reinterpret_cast<const u32x4*>(a.apair + 8 * u + 4 * half);
        }
#pragma unroll
        for (int t = 0; t < TAPS; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) wf[4 * t + u] = as_bf16x8(decode8(c[t][u] >> (4 * half), base[u]));
    }
    // ---- epilogue: lane i has filters 8 (i % 4) .. + 7 of pixels i / 4 and 16 + i / 4 ----
    {
        const int k = n0 + l32 < Kf ? n0 + l32 : Kf - 1;
        float v;
        if (half) {
            v = a.bias ? a.bias[k] : 0.0f;
        } else {
            v = a.colscale ? a.colscale[k] : 1.0f;
            if (a.scale) v *= a.scale[k];
        }
        reinterpret_cast<float*>(smem + wbase + FAC)[lane] = v;
    }
    const int col = n0 + 8 * (lane & 3);
    uint32_t yl[2];  // byte offset from the unit's first pixel; out of the buffer past Kf (Kf % 8 == 0)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int px = 16 * j + (lane >> 2);
        yl[j] = col < Kf ? (uint32_t)(((px >> 3) * a.Q + (px & 7)) * Kf + col) * 2u : oob;
    }
    const uint32_t sh16 = 15u - (uint32_t)(lane >> 2);

    // operand of tap (r, s), step v: pixel (l32 / 8 + r, l32 % 8 + s), segment 2 v + half
    uint32_t ad[2][3][4];
#pragma unroll
    for (int rp = 0; rp < 2; ++rp)
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int key = ((((l32 & 7) + s) >> 1) & 3) | ((((l32 >> 3) + rp) & 1) << 2);
                ad[rp][s][v] = (uint32_t)(wbase + ((l32 >> 3) * PC + (l32 & 7)) * 128 + 16 * ((2 * v + half) ^ key));
            }

    wait_vmcnt(0);
    auto unit = [&](uint32_t u, auto slot_c) {
        constexpr int slot = decltype(slot_c)::value;
        // after this unit's copies: the next unit's eight and the last unit's two stores
        wait_vmcnt(10);
        asm volatile("" ::: "memory");
        const uint32_t ybase = ((cur.img * (uint32_t)a.P + (uint32_t)cur.p) * (uint32_t)a.Q + (uint32_t)cur.q) * (uint32_t)Kf * 2u;
        const uint32_t cols = inside(cur.q, UQ, a.Q), rows = inside(cur.p, UP, a.P);
        uint32_t in = 0;
#pragma unroll
        for (int r = 0; r < UP; ++r) in |= (rows >> r) & 1u ? cols << (UQ * r) : 0u;
        const uint32_t yo[2] = {(((~in << 16) << sh16) & oob) | (yl[0] + ybase), ((~in << sh16) & oob) | (yl[1] + ybase)};
        u32x4 res[2];
        if constexpr (RES) {
#pragma unroll
            for (int j = 0; j < 2; ++j) res[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_r, (int)yo[j], 0, 0);
        }
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
        // operands read DEPTH steps ahead (left to itself the compiler waits for every read)
        auto rd = [&](int i) {
            const int tap = i >> 2, r = tap / 3, s = tap % 3;
            return *reinterpret_cast<const u32x4*>(smem + ad[r & 1][s][i & 3] + slot * SLOT + (r * PC + s) * 128);
        };
        constexpr int STEPS = 4 * TAPS, DEPTH = 4;
        u32x4 x[DEPTH];
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) x[i] = rd(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            acc = mfma32(wf[i], as_bf16x8(x[i % DEPTH]), acc);
            if (i + DEPTH < STEPS) x[i % DEPTH] = rd(i + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (RES) asm volatile("" : "+v"(res[0]), "+v"(res[1]));  // arrived before the copies that follow
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the patch is read before its slot is refilled
        asm volatile("" ::: "memory");
        cur = nxt;
        nxt = locate(u + 2 < uend ? u + 2 : u);
        issue(u + 2, nxt, slot);

#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4*>(sums + l32 * PITCH + 8 * g + 4 * half) =
                f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
        const f32x4 cs[2] = {*reinterpret_cast<const f32x4*>(fac + 8 * (lane & 3)),
                             *reinterpret_cast<const f32x4*>(fac + 8 * (lane & 3) + 4)};
        const f32x4 bi[2] = {*reinterpret_cast<const f32x4*>(fac + 32 + 8 * (lane & 3)),
                             *reinterpret_cast<const f32x4*>(fac + 32 + 8 * (lane & 3) + 4)};
        float v[2][8];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float* const s8 = sums + (16 * j + (lane >> 2)) * PITCH + 8 * (lane & 3);
            const f32x4 sv[2] = {*reinterpret_cast<const f32x4*>(s8), *reinterpret_cast<const f32x4*>(s8 + 4)};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[j][i] = sv[i >> 2][i & 3] * cs[i >> 2][i & 3] + bi[i >> 2][i & 3];
                if constexpr (RES) v[j][i] += bf16_bits_to_f32(i & 1 ? res[j][i >> 1] >> 16 : res[j][i >> 1] & 0xFFFFu);
            }
        }
        if (a.relu) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i) v[j][i] = fmaxf(v[j][i], 0.0f);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const u32x4 o = {pack_bf16x2(v[j][0], v[j][1]), pack_bf16x2(v[j][2], v[j][3]), pack_bf16x2(v[j][4], v[j][5]),
                             pack_bf16x2(v[j][6], v[j][7])};
            // a buffer store, issued whatever the lanes' offsets are: the waits count it
            __builtin_amdgcn_raw_buffer_store_b128(o, rs_y, (int)yo[j], 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    };
    for (uint32_t u = ubeg; u < uend; u += 2) {
        unit(u, std::integral_constant<int, 0>{});
        if (u + 1 < uend) unit(u + 1, std::integral_constant<int, 1>{});
    }
    wait_vmcnt(0);
}

}  // namespace

// Measured against the tiled kernel (forward with scale, bias and ReLU, graph-replayed, us), by wave
// items (units x groups of 32 filters):
//   12544: 56 x 56 -> 64 at batch 64 26.8 -> 21.4 (with the residual 27.6 -> 21.6), -> 40 29.1 -> 20.6
//   25088: 56 x 56 -> 128 at batch 64 40.2 -> 34.6;  8192: 32 x 32 -> 64 at batch 128 17.8 -> 15.9
//   6272:  56 x 56 -> 64 at batch 32 16.6 -> 14.1;   4125: 41 x 38 -> 96 at batch 25 13.2 -> 10.9
//   3136 and 1568: equal (9.8, 7.6);  1960: 56 x 56 -> 8 at batch 20 10.7 -> 7.3
//   1024:  14 x 14 -> 64 at batch 64 7.4 -> 5.8
//   backward-data from 64 filters at 56 x 56, batch 64: 30.7 -> 25.2 (64 channels), 44.4 -> 37.7 (128)
// 128 filters have the tiled kernel's 64 x 128 tiles while those are few: 12544 items 23.1 -> 21.8, but
// 4480 (28 x 28 at batch 40) 9.2 against 11.8 and 3136 8.9 against 9.8.  Beyond 128 filters the
// tiled kernel's 256-filter tiles decode a word for more pixels (56 x 56 -> 256 at batch 16: 20.7
// against 21.6).  Fewer items belong to the small-layer kernel or were not faster; maps whose units
// lie more than 0.4 past the edges waste more than the difference (at 0.31, 7 x 7 and 14 x 14,
// 8.4 -> 7.7 and equal).
// A wave's range is whole units, so the time goes by rounds of 2048 waves; the tiled kernel's goes by rounds of
// 256 tiles of 128 pixels.  Where its 64- and 128-filter tiles are full the two lie close, and the rounds decide
// (this kernel's share of its time, 1000 random layers; rounds here : there):
//   64 filters:   1:1 to 3:3 0.86-0.98, 2:1, 3:2 and 4:3 1.02-1.14;  4:4 0.82-0.87;  5:4 0.94;  7:6 0.87-0.90;
//                 14:11 0.89;  17:14 0.86
//   128 filters:  5:2 1.11-1.15;  6:3 0.85-0.95, 7:3 0.96-1.00, 8:3 1.09;  8:4 0.92, 10:4 1.03;  12:5 0.99;
//                 13:6 0.89-0.95, 15:6 1.01;  18:8 0.89-0.94;  24:10 0.90;  35:15 0.95
// With fewer filters than its tile has, or 65 to 127, this one is faster at every share (40 to 56 filters
// 0.65-0.97, up to 32 and 96 below 0.94).
bool conv_c64_chosen(const ConvGemmArgs& a, int cfg) {
    if (cfg != 60 && (cfg >= 0 || conv_splits_override() > 0)) return false;
    if (a.C != C64 || a.R != 3 || a.S != 3 || a.sh != 1 || a.sw != 1 || a.y_f32 || a.Kf % 8 != 0) return false;
    const int64_t M = (int64_t)a.N * a.P * a.Q;
    if (M * a.Kf * 2 >= 0x7FFFFFF0ll) return false;
    const int64_t units = (int64_t)a.N * ((a.P + UP - 1) / UP) * ((a.Q + UQ - 1) / UQ);
    if (cfg == 60) return true;
    const int64_t items = units * ((a.Kf + 31) / 32);
    if (a.Kf > 128 || items < (a.Kf == 128 ? 8192 : 1024) || units * (UP * UQ) * 5 > M * 7) return false;
    const int64_t fgroups = (a.Kf + 31) / 32, per = (items < 2048 ? items : 2048) / fgroups;
    const int64_t rounds = (units + per - 1) / per, tiled = (M + 32767) / 32768;
    if (a.Kf == 128) return rounds <= (5 * tiled - 1) / 2;
    return a.Kf != 64 || rounds <= (4 * tiled - 1) / 3;
}

hipError_t launch_conv_c64(const ConvGemmArgs& g, hipStream_t stream) {
    C64Args a;
    a.g = g;
    a.tiles_p = (g.P + UP - 1) / UP;
    a.tiles_q = (g.Q + UQ - 1) / UQ;
    a.div_upi = make_fastdiv((uint32_t)(a.tiles_p * a.tiles_q));
    a.div_tq = make_fastdiv((uint32_t)a.tiles_q);
    a.units = (uint32_t)g.N * (uint32_t)(a.tiles_p * a.tiles_q);
    a.fgroups = (g.Kf + 31) / 32;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    // two blocks a CU; fewer where there are fewer units than waves
    int64_t waves = 8ll * cus;
    if (waves < a.fgroups) waves = a.fgroups;
    const int64_t items = (int64_t)a.units * a.fgroups;
    if (waves > items) waves = items;
    a.per = (int32_t)(waves / a.fgroups);
    const dim3 grid((unsigned)((a.per * (int64_t)a.fgroups + 3) / 4)), block(256);
    if (g.apair)
        hipLaunchKernelGGL((conv_c64_kernel<true, false>), grid, block, 0, stream, a);
    else if (g.residual)
        hipLaunchKernelGGL((conv_c64_kernel<false, true>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((conv_c64_kernel<false, false>), grid, block, 0, stream, a);
    return hipGetLastError();
}

}  // namespace tbn
