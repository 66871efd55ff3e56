// tbn_wgrad_dma.hip -- gradient with respect to the approximate filter (Algorithm 1,
// backward step; Sec. 3 applies it unchanged to the real weights):
//     dW[k][j] = sum_m dy[m][k] * x_col[m][j],   m = (n,p,q) output pixel, j = (r,s,c),
// for bf16 activations with C % 8 == 0 and K % 8 == 0.
//
// Both operands arrive with the reduction index (the pixel) outermost, while the MFMA
// wants 8 consecutive reduction elements per lane.  Instead of transposing in registers,
// the kernels copy the raw tiles into LDS with LDS-DMA buffer loads and form the MFMA
// operands with the gfx950 transposing LDS read (ds_read_b64_tr_b16: a 16-lane group
// turns a 16 x 4 block of 16-bit values into 4 consecutive rows per lane), so the main
// loop spends no vector ALU work on data movement:
//   * a block of 8 waves owns an output tile (256 (k) x 256 (j), each wave 128 x 64, for wide
//     layers) made of 32x32 v_mfma_f32_32x32x16_bf16 tiles with fp32 accumulators;
//   * stages of pixels in a ring of LDS buffers: the DMAs of later stages overlap the
//     MFMAs of the current one, and the operands of each 16-pixel step are read one or two
//     steps earlier;
//   * the pixel range is split over the grid (split-K): each split writes fp32 partials
//     that a second kernel adds in a fixed order (deterministic result).
// Two kernels: 256 x 256 tiles for wide layers, narrow tiles where K or J would leave most of
// such a tile empty.
#include <cstdlib>
#include <type_traits>

#include "tbn_device.h"
#include "tbn_dma.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

struct WgradDmaArgs {
    WgradArgs a;
    FastDiv div_q, div_pq;
    int32_t pf_dist;  // wide kernel: stages between a copy and the L2 prefetch issued with it
};

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

__device__ __forceinline__ v4i16 read_tr(uint32_t addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(uintptr_t)addr);
}

// Per-lane select by a wave-uniform 64-bit lane mask: bit i of `mask` set -> lane i gets
// `if_set`.  One v_cndmask with the mask in a scalar register pair.
__device__ __forceinline__ uint32_t lane_select(uint64_t mask, uint32_t if_clear, uint32_t if_set) {
    uint32_t r;
    asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(if_clear), "v"(if_set), "s"(mask));
    return r;
}

// Instruction order of one 16-pixel step: its 8 MFMAs alternate with the 12 transposing
// reads of a later step's operands (two after each of the first four MFMAs, one after each
// of the others) and with the scalar work of the copy table, so that neither is issued in
// one burst (the reads spread this way measured ~6% faster than the compiler's own order
// on the 256 x 2304 training-layer gradient).
__device__ __forceinline__ void interleave_reads() {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // two LDS reads
        __builtin_amdgcn_sched_group_barrier(0x004, 8, 0);  // scalar work of the copy table
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x004, 8, 0);
    }
}

// Narrow variant: block tiles of TK x TJ = 32 TM WM x 32 TN WN (filters x columns) for layers
// whose K or J leaves most of a 256 x 256 tile empty.  A block is two groups of four waves; each
// group reduces its own half of the split's pixels with its own LDS ring, and group 1 hands its
// sums to group 0 through LDS (half as many partial gradients in memory as with two blocks).
//
// A stage holds PIX pixels as rows of the dy tile, then rows of the x tile, copied 1 KiB at a
// time: with RS = 8-channel segments per row an LDS-DMA instruction takes 64 / RS whole rows, so
// requests cover runs of TK or TJ channels.  Which memory piece a lane fetches is free, where it
// lands is not, so the bank spread comes from the fetch: slot s of pixel p holds segment s ^ f(p),
//   f(p) = 4 (p % 4) for RS >= 16, 4 (p / 2 % 2) for RS = 8, 0 for RS = 4,
// and the 8 pixels x 64 bytes of a transposing read cover every bank exactly twice.
// Where each pixel's taps start in x comes from a table in LDS (byte offset, top-left
// coordinates): one wave of the group fills it for a later stage, so that a copy costs a lane one
// LDS read and about nine vector operations rather than two divisions.
//
// One barrier per stage, ahead of its last 16-pixel step: stage it + 1 has landed and every wave
// holds the operands of stage it's last step, so the copies of stage it + STAGES go into its slot
// and the next stage's first operands are read under that step's MFMAs.
struct TapEntry {
    uint32_t off;  // byte offset of the pixel's (h0, w0, channel 0) in x, modulo 2^32
    int32_t hw;    // h0 << 16 | w0 & 0xFFFF; h0 = -32768: not a pixel of this split (at no tap: R <= 32768)
};

template <int RS>
__device__ __forceinline__ int row_swizzle(int p) {  // f(p) / 4
    return RS >= 16 ? (p & 3) : RS == 8 ? ((p >> 1) & 1) : 0;
}

template <int TM, int TN, int WM, int WN, int PIX>
struct NarrowLayout {
    static constexpr int TK = 32 * TM * WM, TJ = 32 * TN * WN;
    static constexpr int STAGES = 3, G = 2, TABS = 4;
    static constexpr int X = PIX * TK * 2;          // x rows behind the dy rows
    static constexpr int STAGE = X + PIX * TJ * 2;
    static constexpr int RING = STAGES * STAGE;
    static constexpr int TAB = G * RING;            // TABS tables of PIX entries per group
    static constexpr int BYTES = TAB + G * TABS * PIX * 8;
    static constexpr int SUMS = 256 * TM * TN * 16 * 4;
    static_assert(BYTES <= 160 * 1024 && SUMS <= TAB, "LDS");
};

template <int TM, int TN, int WM, int WN, int PIX>
__global__ __launch_bounds__(512, 1) void wgrad_narrow_kernel(const WgradDmaArgs ka) {
    using L = NarrowLayout<TM, TN, WM, WN, PIX>;
    constexpr int TK = L::TK, TJ = L::TJ, STAGES = L::STAGES, G = L::G, TABS = L::TABS;
    constexpr int RSY = TK / 8, RSX = TJ / 8;        // segments per row
    constexpr int PY = 64 / RSY, PX = 64 / RSX;      // rows per copy instruction
    constexpr int NY = PIX / PY, NX = PIX / PX;      // copy instructions per stage
    constexpr int YD = NY >= 4 ? NY / 4 : 1, XD = NX >= 4 ? NX / 4 : 1;  // ... per wave
    constexpr int NU = PIX / 16;
    static_assert(WM * WN == 4 && NU >= 2 && PIX <= 64, "group");
    const WgradArgs& a = ka.a;

    __shared__ __attribute__((aligned(1024))) uint8_t smem[L::BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int grp = __builtin_amdgcn_readfirstlane(tid >> 8);
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    const int wm = wave / WN, wn = wave % WN;

    const int K = a.K, C = a.C;
    const int J = a.R * a.S * C;
    const uint32_t PQ = (uint32_t)a.P * a.Q;
    const int64_t M = (int64_t)a.N * PQ;
    const int tilesJ = (J + TJ - 1) / TJ;
    const int tiles = tilesJ * ((K + TK - 1) / TK);
    const int t_ = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int split = t_ / tiles;
    const int k0 = ((t_ % tiles) / tilesJ) * TK;
    const int j0 = ((t_ % tiles) % tilesJ) * TJ;
    // this split's pixels (ranges in 64-pixel chunks), and its group's stages; both groups run the
    // same number (rows past the end are zeros)
    const int64_t s_begin = (int64_t)split * a.chunks_per_split * 64;
    const int64_t s_end = min(s_begin + (int64_t)a.chunks_per_split * 64, M);
    const int nst = s_end > s_begin ? (int)((s_end - s_begin + G * PIX - 1) / (G * PIX)) : 0;
    const int64_t m_begin = s_begin + (int64_t)grp * nst * PIX;

    // rows of dy past the split's end are past the end of this buffer
    const v4i rs_dy = make_rsrc(a.dy, (uint32_t)(max(s_end, (int64_t)0) * K * 2));
    const v4i rs_x = make_rsrc(a.x, (uint32_t)((int64_t)a.N * a.H * a.W * C * 2));
    uint8_t* const ring = smem + grp * L::RING;
    const uint32_t ring_base = lds_addr(ring);
    TapEntry* const tabs = reinterpret_cast<TapEntry*>(smem + L::TAB) + grp * TABS * PIX;

    // ---- copies.  Instruction d of a stage (wave w: d = w, w + 4, ..) fills rows PY d (PX d) on;
    //      waves with no instruction of their own repeat another's, identical bytes, so that every
    //      wave has the same number in flight ----
    const int yrow = PY * (wave % (NY < 4 ? NY : 4)) + lane / RSY;
    const int xrow = PX * (wave % (NX < 4 ? NX : 4)) + lane / RSX;
    const int yseg = (lane % RSY) ^ (4 * row_swizzle<RSY>(yrow));
    const int xseg = (lane % RSX) ^ (4 * row_swizzle<RSX>(xrow));
    const bool y_ok = k0 + 8 * yseg < K;
    // a row's offset may pass 2^31 only past the buffer's end (< 2 GiB); columns past K start there
    const uint32_t y_lane = y_ok ? (uint32_t)((m_begin + yrow) * K + k0 + 8 * yseg) * 2u : 0x80000000u;
    const uint32_t y_step = (uint32_t)(PIX * K * 2);
    const int jx = j0 + 8 * xseg;
    const bool x_ok = jx < J;
    const int tap = x_ok ? jx / C : 0;
    const int xr = tap / a.S, xs = tap - (tap / a.S) * a.S;
    const uint32_t x_lane = (uint32_t)((xr * a.W + xs) * C + (x_ok ? jx - tap * C : 0)) * 2u;

    auto table = [&](int st) {  // where the taps of each pixel of stage st start
        if (lane < PIX) {
            const int64_t m = m_begin + (int64_t)st * PIX + lane;
            TapEntry e = {0u, -32768 * 65536};
            if (m < s_end) {
                const uint32_t img = fdiv((uint32_t)m, ka.div_pq);
                const uint32_t pq = (uint32_t)m - img * PQ;
                const uint32_t p = fdiv(pq, ka.div_q);
                const int h0 = (int)p * a.sh - a.ph, w0 = (int)(pq - p * (uint32_t)a.Q) * a.sw - a.pw;
                e.off = ((img * (uint32_t)a.H + (uint32_t)h0) * (uint32_t)a.W + (uint32_t)w0) * (uint32_t)C * 2u;
                e.hw = (int32_t)((uint32_t)h0 << 16 | ((uint32_t)w0 & 0xFFFFu));
            }
            tabs[(st % TABS) * PIX + lane] = e;
        }
    };
    auto issue = [&](int st, int slot) {
        const uint32_t base = ring_base + (uint32_t)(slot * L::STAGE);
#pragma unroll
        for (int d = 0; d < YD; ++d) {
            // the stage's rows in one add (wraps only where y_lane is past the end, and stays there:
            // an offset past the buffer grows by less than 2 GiB over the whole split)
            const uint32_t off = y_ok ? y_lane + (uint32_t)st * y_step + (uint32_t)(4 * PY * d * K * 2) : 0x80000000u;
            dma_b128(rs_dy, base + (uint32_t)((wave % (NY < 4 ? NY : 4) + 4 * d) * 1024), off);
        }
#pragma unroll
        for (int d = 0; d < XD; ++d) {
            const TapEntry e = tabs[(st % TABS) * PIX + xrow + 4 * PX * d];
            const int h = (e.hw >> 16) + xr, w = (int)(int16_t)e.hw + xs;
            const bool ok = x_ok && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
            dma_b128(rs_x, base + (uint32_t)(L::X + (wave % (NX < 4 ? NX : 4) + 4 * d) * 1024),
                     ok ? e.off + x_lane : 0x80000000u);
        }
    };
    constexpr int kDmas = YD + XD;

    // ---- operand addresses: lane (g = lane / 16, i = lane % 16) reads 8 bytes, channels
    //      16 (g % 2) + 4 (i % 4) .. + 3 of a 32-channel tile, at pixel 8 (g / 2) + i / 4 of a step
    //      (and + 4 in the second read) ----
    const int g = lane >> 4, i16 = lane & 15;
    const int prow = 8 * (g >> 1) + (i16 >> 2);
    const uint32_t in_tile = (uint32_t)(16 * (2 * (g & 1) + ((i16 & 3) >> 1)) + 8 * (i16 & 1));
    uint32_t ra[STAGES][TM], rb[STAGES][TN];
#pragma unroll
    for (int sl = 0; sl < STAGES; ++sl) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
            ra[sl][i] = (ring_base + (uint32_t)(sl * L::STAGE + prow * TK * 2 +
                                                64 * ((wm * TM + i) ^ row_swizzle<RSY>(prow))) + in_tile) & 0x3FFFFu;
#pragma unroll
        for (int t = 0; t < TN; ++t)
            rb[sl][t] = (ring_base + (uint32_t)(sl * L::STAGE + L::X + prow * TJ * 2 +
                                                64 * ((wn * TN + t) ^ row_swizzle<RSX>(prow))) + in_tile) & 0x3FFFFu;
    }
    auto operand = [&](uint32_t addr, uint32_t four_rows) {
        const v4i16 lo = read_tr(addr);
        const v4i16 hi = read_tr(addr + four_rows);
        typedef short v8i16 __attribute__((ext_vector_type(8)));
        const v8i16 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    };
    auto load = [&](int sl, int u, bf16x8* af, bf16x8* bf) {
#pragma unroll
        for (int t = 0; t < TN; ++t) bf[t] = operand(rb[sl][t] + (uint32_t)(16 * u * TJ * 2), 4 * TJ * 2);
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = operand(ra[sl][i] + (uint32_t)(16 * u * TK * 2), 4 * TK * 2);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.0f;

    table(wave);  // the first TABS = 4 stages, one per wave
    __syncthreads();
#pragma unroll
    for (int c = 0; c < STAGES; ++c)
        if (c < nst) issue(c, c);
    auto wait_stage = [&](int x) {  // stage x landed; up to STAGES - 1 later ones may be in flight
        const int later = min(nst - 1 - x, STAGES - 1);
        if (later >= 2)
            wait_vmcnt(2 * kDmas);
        else if (later == 1)
            wait_vmcnt(kDmas);
        else
            wait_vmcnt(0);
    };
    bf16x8 af[2][TM], bf[2][TN];
    if (nst > 0) {
        wait_stage(0);
        __syncthreads();
        load(0, 0, af[0], bf[0]);
    }
    auto stage = [&](int it, auto slot) {
        constexpr int SL = decltype(slot)::value;
        constexpr int SN = SL + 1 == STAGES ? 0 : SL + 1;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u + 1 < NU) {
                load(SL, u + 1, af[(u + 1) & 1], bf[(u + 1) & 1]);
            } else {
                // stages 0 .. it + STAGES - 1 are issued
                if (it + STAGES - 1 < nst)
                    wait_vmcnt((STAGES - 2) * kDmas);
                else
                    wait_vmcnt(0);
                __syncthreads();
                if (it + STAGES < nst) issue(it + STAGES, SL);
                if (wave == (it & 3) && it + STAGES + 1 < nst) table(it + STAGES + 1);
                load(SN, 0, af[(u + 1) & 1], bf[(u + 1) & 1]);  // unused after the last stage
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[i][t] = mfma32(af[u & 1][i], bf[u & 1][t], acc[i][t]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    static_assert(NU % 2 == 0 && STAGES == 3, "operand sets alternate, ring unrolled over three slots");
    for (int it = 0; it < nst; it += STAGES) {
        stage(it, std::integral_constant<int, 0>{});
        if (it + 1 < nst) stage(it + 1, std::integral_constant<int, 1>{});
        if (it + 2 < nst) stage(it + 2, std::integral_constant<int, 2>{});
    }

    // ---- group 1 hands its sums over (16-byte pieces, lane-contiguous) ----
    __syncthreads();
    f32x4* const xch = reinterpret_cast<f32x4*>(smem) + wave * 64 + lane;
    if (grp == 1) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    xch[((i * TN + t) * 4 + v) * 256] =
                        f32x4{acc[i][t][4 * v], acc[i][t][4 * v + 1], acc[i][t][4 * v + 2], acc[i][t][4 * v + 3]};
    }
    __syncthreads();
    if (grp == 1) return;  // no barrier follows
    float* out = a.out + (int64_t)split * K * J;
    const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int col = j0 + wn * 32 * TN + 32 * t + l32;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = k0 + wm * 32 * TM + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row < K && col < J) {
                    float* o = out + (int64_t)row * J + col;
                    const float s = acc[i][t][v] + xch[((i * TN + t) * 4 + (v >> 2)) * 256][v & 3];
                    *o = a.accumulate ? *o + s : s;
                }
            }
        }
    }
}

// Wide variant: a stage holds PIXR pixels of the dy tile (256 channels, 512 bytes)
// then the same pixels of the x tile (256 columns).  Pixel rows are stored in pairs:
// pixels i and i + PIXR/2 of the stage share a 1088-byte slot (512 + 512 + 64 bytes of
// padding), so one DMA instruction with all 64 lanes active copies two pixels (each lane
// 16 bytes; the vector memory pipe issues a 32-lane copy at the cost of a full one) and
// every request covers whole 128-byte lines.  A transposing read touches four
// consecutive stage pixels and the four 8 further on (then the next four of each); in
// consecutive slots those rows start 64 bytes apart modulo 256, so every LDS bank is used
// at most twice.  The order in which the pixels enter the reduction follows this layout
// (a permutation within the stage).
constexpr int PP = 1088;  // bytes per pair of pixel rows

// PIXR pixels per stage (a multiple of 16), STAGES-deep ring; 2 x 4 waves of 128 x 64,
// two waves per SIMD.  (One wave per SIMD with 128 x 128 wave tiles reads a third less
// from LDS per MFMA but measured slower: the stage boundaries are no longer covered.)
// LIN: linear copy addressing (see below), chosen by the host.
template <int PIXR, int STAGES, bool PF, bool LIN>
__global__ __launch_bounds__(512, 1) void wgrad_rows_kernel(const WgradDmaArgs ka) {
    const WgradArgs& a = ka.a;
    constexpr int WAVES = 8;
    constexpr int WNW = 4;              // waves along j
    constexpr int TM = 4, TN = 2;       // wave tile 128 x 64 of the 256 x 256 block tile
    constexpr int NPAIR = PIXR / 2;     // pixel pairs per stage
    constexpr int PAIRS = NPAIR / WAVES;  // pairs each wave copies per stage
    constexpr int PR_OP = NPAIR * PP;   // one operand tile of a stage
    constexpr int PR_STAGE = 2 * PR_OP;
    constexpr int DUMP = STAGES * PR_STAGE;  // 256 bytes that the L2 prefetches land in
    static_assert(PIXR % 16 == 0 && NPAIR % WAVES == 0, "stage size");
    static_assert(DUMP + 256 <= 160 * 1024, "LDS");

    __shared__ __attribute__((aligned(1024))) uint8_t smem[DUMP + 256];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WNW;
    const int wn = wave % WNW;

    const int K = a.K, C = a.C;
    const int J = a.R * a.S * C;
    const uint32_t PQ = (uint32_t)a.P * a.Q;
    const int64_t M = (int64_t)a.N * PQ;
    const int tilesJ = (J + 255) / 256;
    const int tiles = tilesJ * ((K + 255) / 256);
    const int t_ = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int split = t_ / tiles;
    const int k0 = ((t_ % tiles) / tilesJ) * 256;
    const int j0 = ((t_ % tiles) % tilesJ) * 256;
    // this split's pixels (the ranges are given in 64-pixel chunks) and its stages
    const int64_t m_begin = (int64_t)split * a.chunks_per_split * 64;
    const int64_t m_end = min(m_begin + (int64_t)a.chunks_per_split * 64, M);
    const int nst = m_end > m_begin ? (int)((m_end - m_begin + PIXR - 1) / PIXR) : 0;

    const v4i rs_dy = make_rsrc(a.dy, (uint32_t)(M * K * 2));
    const v4i rs_x = make_rsrc(a.x, (uint32_t)((int64_t)a.N * a.H * a.W * C * 2));
    const uint32_t smem_base = lds_addr(smem);

    // this lane's 8-channel segment of the dy row and of the x column tile, and which
    // pixel of a pair it copies
    const int seg = lane & 31;
    const int half = lane >> 5;
    const bool dy_ok = k0 + 8 * seg < K;
    const uint32_t dy_col = (uint32_t)(k0 + 8 * seg) * 2u;
    const uint32_t dy_bad = dy_ok ? 0u : 0x80000000u;
    const int jx = j0 + 8 * seg;
    const bool x_ok = jx < J;
    const int rsx = x_ok ? jx / C : 0;
    const int xc = x_ok ? jx - rsx * C : 0;
    const int xr = rsx / a.S, xs = rsx - (rsx / a.S) * a.S;
    const uint32_t HWC = (uint32_t)((int64_t)a.H * a.W * C);

    // (image, h, w) of output pixel m, for the x tap (r, s)
    auto locate = [&](uint32_t mm, int r, int s_, uint32_t* img, int* h, int* w) {
        *img = fdiv(mm, ka.div_pq);
        const uint32_t pq = mm - *img * PQ;
        const uint32_t p = fdiv(pq, ka.div_q);
        const uint32_t q_ = pq - p * (uint32_t)a.Q;
        *h = (int)p * a.sh - a.ph + r;
        *w = (int)q_ * a.sw - a.pw + s_;
    };

    // Byte offsets of this lane's copies of a stage (bit 31 set: outside the image or past
    // the split's last pixel, the hardware returns zeros): pair jj of the wave holds stage
    // pixels PAIRS wave + jj and that + NPAIR.  Computed for the next stage while the
    // MFMAs of the current one run.
    uint32_t o_dy[PAIRS], o_x[PAIRS];
    // the PAIRS pixels of a lane are consecutive: the first is located by division, the
    // others step q (and carry into p and the image)
    const int q_step = a.sw, p_step = a.sh;
    auto table_general = [&](int st_i) {
        const int64_t m0 = m_begin + (int64_t)st_i * PIXR + PAIRS * wave + NPAIR * half;
        uint32_t mm = m0 < m_end ? (uint32_t)m0 : 0u;
        uint32_t img = fdiv(mm, ka.div_pq);
        const uint32_t pq = mm - img * PQ;
        uint32_t p = fdiv(pq, ka.div_q);
        uint32_t q_ = pq - p * (uint32_t)a.Q;
        int h = (int)p * a.sh - a.ph + xr, w = (int)q_ * a.sw - a.pw + xs;
#pragma unroll
        for (int jj = 0; jj < PAIRS; ++jj) {
            const bool mok = m0 + jj < m_end;
            const uint32_t mj = mm + jj;
            o_dy[jj] = mok ? (mj * (uint32_t)K * 2u + dy_col) | dy_bad : 0x80000000u;
            const bool ok = mok && x_ok && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
            o_x[jj] = ok ? (img * HWC + (uint32_t)((h * a.W + w) * C + xc)) * 2u : 0x80000000u;
            if (jj + 1 < PAIRS) {  // next output pixel
                ++q_;
                w += q_step;
                if (q_ == (uint32_t)a.Q) {
                    q_ = 0;
                    w -= a.Q * q_step;
                    ++p;
                    h += p_step;
                    if (p == (uint32_t)a.P) {
                        p = 0;
                        h -= a.P * p_step;
                        ++img;
                    }
                }
            }
        }
    };
    // Linear copies: a stride-1 convolution whose output has the input's size (P = H,
    // Q = W) maps output pixel m and tap (r, s) to input pixel m + (r - ph) W + (s - pw),
    // and with C % 256 == 0 the 256 columns of a block share one tap.  Then both halves'
    // offsets are one wave-uniform pixel offset (the first pixel of the pair; the second
    // lies NPAIR pixels on) plus a per-lane constant, and only the validity of the two
    // pixels (inside the image for the tap, before the split's end) is tested, on the
    // scalar unit; per copy one add and one select remain on the vector unit.
    const int tap = j0 / (LIN ? C : 1);
    const int tr = tap / a.S, ts = tap - (tap / a.S) * a.S;  // the block's tap (linear copies)
    const uint32_t ldy = dy_col + (uint32_t)(half * NPAIR * K * 2);
    const uint32_t lx = (uint32_t)(seg * 16 + half * NPAIR * C * 2);
    const int32_t x_shift = ((tr - a.ph) * a.W + (ts - a.pw)) * C + (LIN ? j0 - tap * C : 0);
    const uint64_t dyok_lanes = __builtin_amdgcn_ballot_w64(dy_ok);
    const uint32_t oob = 0x80000000u;
    // The linear table is built in two parts: a vector pass in which lane i tests stage
    // pixel i (inside the split, and inside the image for the block's tap) and the wave
    // collects the answers as one 64-bit mask, then per pair a few scalar bit tests that
    // turn the mask bits of its two pixels into the lane masks of the selects.  The main
    // loop places the parts between the MFMAs of different steps.
    uint64_t xin = 0;  // bit i: stage pixel i is in the split and its tap inside the image
    auto table_linear_mask = [&](int st_i) {
        const int32_t s0 = (int32_t)m_begin + st_i * PIXR;  // first pixel of the stage (< 2^31)
        const int32_t ms = s0 + lane;
        const bool in = lane < PIXR && ms < (int32_t)m_end;
        const uint32_t mm = in ? (uint32_t)ms : 0u;
        const uint32_t pq = mm - fdiv(mm, ka.div_pq) * PQ;
        const uint32_t p = fdiv(pq, ka.div_q);
        const uint32_t q_ = pq - p * (uint32_t)a.Q;
        const bool inside = (unsigned)((int)p - a.ph + tr) < (unsigned)a.H &&
                            (unsigned)((int)q_ - a.pw + ts) < (unsigned)a.W;
        xin = __builtin_amdgcn_ballot_w64(in && inside);
    };
    auto table_linear_select = [&](int st_i) {
        const int32_t s0 = (int32_t)m_begin + st_i * PIXR;
        const int32_t rem = (int32_t)m_end - s0;  // pixels of the split from the stage's first on
        const int32_t mA0 = s0 + PAIRS * wave;
#pragma unroll
        for (int jj = 0; jj < PAIRS; ++jj) {
            // stage pixels of the pair: A (lanes 0-31) and B = A + NPAIR (lanes 32-63)
            const int iA = PAIRS * wave + jj, iB = iA + NPAIR;
            const uint64_t ld_ok = (iA < rem ? 0x00000000FFFFFFFFull : 0ull) | (iB < rem ? 0xFFFFFFFF00000000ull : 0ull);
            const uint64_t lx_ok = (((xin >> iA) & 1ull) ? 0x00000000FFFFFFFFull : 0ull) |
                                   (((xin >> iB) & 1ull) ? 0xFFFFFFFF00000000ull : 0ull);
            const uint32_t mj = (uint32_t)(mA0 + jj);  // wraps harmlessly where masked off
            o_dy[jj] = lane_select(ld_ok & dyok_lanes, oob, mj * (uint32_t)K * 2u + ldy);
            o_x[jj] = lane_select(lx_ok, oob, (mj * (uint32_t)C + (uint32_t)x_shift) * 2u + lx);
        }
    };
    auto table = [&](int st_i) {
        if constexpr (LIN) {
            table_linear_mask(st_i);
            table_linear_select(st_i);
        } else {
            table_general(st_i);
        }
    };
    // The table of stage Y is needed when Y is issued, two steps before the end of stage
    // Y - STAGES, and may be built once stage Y-1 has been issued.  In stage `it` the
    // linear table of stage it+STAGES+1 starts in the last step (the mask pass) and that of
    // stage it+STAGES is finished in the first step (the selects); with two steps per stage
    // all of it in the last step.  The general table is built whole in the last step.
    constexpr int NSTEP = PIXR / 16;
    auto table_part = [&](int it, int u) {
        if constexpr (LIN) {
            if (NSTEP == 2) {
                if (u == 1) table(it + STAGES + 1);
            } else {
                if (u == NSTEP - 1) table_linear_mask(it + STAGES + 1);
                if (u == 0) table_linear_select(it + STAGES);
            }
        } else {
            if (u == NSTEP - 1) table_general(it + STAGES + 1);
        }
    };
    int islot = 0;  // ring slot of the next stage to issue
    auto issue = [&](int) {
        const uint32_t st = smem_base + (uint32_t)(islot * PR_STAGE);
        islot = islot + 1 == STAGES ? 0 : islot + 1;
#pragma unroll
        for (int jj = 0; jj < PAIRS; ++jj) {
            const int j = PAIRS * wave + jj;  // pair slot (wave-uniform)
            dma_b128(rs_dy, st + (uint32_t)(j * PP), o_dy[jj]);
            dma_b128(rs_x, st + (uint32_t)(PR_OP + j * PP), o_x[jj]);
        }
    };
    constexpr int kDmas = 2 * PAIRS;

    // L2 prefetch of a later stage: one 4-byte copy per thread into a dump area touches one
    // 128-byte line (waves 0-3: the dy rows, stage pixel (tid % 256) / 4, line tid % 4 of
    // its 512 bytes; waves 4-7: the same for the x rows), so that the copies of that stage
    // find their lines in L2.
    const int pf_line = tid & 3;
    const int pf_pix = (tid & 255) >> 2;
    const bool pf_is_x = wave >= 4;  // wave-uniform
    const int pf_k = k0 + 64 * pf_line;
    const int pf_j = j0 + 64 * pf_line;
    const bool pf_jok = pf_j < J;
    const int pf_rs = pf_jok ? pf_j / C : 0;
    const int pf_c = pf_jok ? pf_j - pf_rs * C : 0;
    const int pf_r = pf_rs / a.S, pf_s = pf_rs - (pf_rs / a.S) * a.S;
    auto prefetch = [&](int st_i) {
        const int64_t m = m_begin + (int64_t)st_i * PIXR + pf_pix;
        const bool mok = pf_pix < PIXR && m < m_end;
        const uint32_t mm = mok ? (uint32_t)m : 0u;
        if (pf_is_x) {
            uint32_t img;
            int h, w;
            locate(mm, pf_r, pf_s, &img, &h, &w);
            const bool ok = mok && pf_jok && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
            dma_b32(rs_x, smem_base + DUMP,
                    ok ? (img * HWC + (uint32_t)((h * a.W + w) * C + pf_c)) * 2u : 0x80000000u);
        } else {
            dma_b32(rs_dy, smem_base + DUMP,
                    mok && pf_k < K ? (mm * (uint32_t)K + (uint32_t)pf_k) * 2u : 0x80000000u);
        }
    };
    const int pf_dist = ka.pf_dist;

    // transposing reads: lane (g = lane / 16, i = lane % 16) reads the 8 bytes of channels
    // 16 (g % 2) + 4 (i % 4) .. + 3 of stage pixel 16 u + 8 (g / 2) + i / 4 (+ 4 for the
    // second read) in step u; stage pixel r sits at (r % NPAIR) * PP + (r / NPAIR) * 512.
    // One address register per (ring slot, step, operand), masked to the LDS size so that
    // the compiler can prove it non-negative and fold the constant offsets of the other
    // rows of the wave tile into the read instructions.
    constexpr int NU = PIXR / 16;
    const int g = lane >> 4, i16 = lane & 15;
    const int rho = 8 * (g >> 1) + (i16 >> 2);
    const uint32_t col_off = (uint32_t)((16 * (g & 1) + 4 * (i16 & 3)) * 2);
    const uint32_t a_base = (uint32_t)(wm * 128 * 2);
    const uint32_t b_base = (uint32_t)PR_OP + (uint32_t)(wn * 32 * TN * 2);
    uint32_t ra[STAGES][NU], rb[STAGES][NU];
#pragma unroll
    for (int sl = 0; sl < STAGES; ++sl)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int r = 16 * u + rho;
            const uint32_t ro = (uint32_t)((r % NPAIR) * PP + (r / NPAIR) * 512) + col_off;
            ra[sl][u] = (smem_base + (uint32_t)(sl * PR_STAGE) + a_base + ro) & 0x3FFFFu;
            rb[sl][u] = (smem_base + (uint32_t)(sl * PR_STAGE) + b_base + ro) & 0x3FFFFu;
        }
    auto operand = [&](uint32_t addr) {
        const v4i16 lo = read_tr(addr);
        const v4i16 hi = read_tr(addr + 4 * PP);
        typedef short v8i16 __attribute__((ext_vector_type(8)));
        const v8i16 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.0f;

    // Pipeline: every ring slot is filled in the prologue; stage `it` is multiplied step by
    // step with the operands of each step read two steps earlier.  Two steps before the end
    // of stage `it` a barrier certifies that every wave is done reading stage `it` (the
    // operands of its last two steps are already in registers) and that stage it+1 has
    // landed; the copies of stage it + STAGES then go into stage it's slot, and the last
    // two steps' MFMAs overlap the copies and the reads of stage it+1's first two steps.
    // So no wave waits on LDS reads at a stage boundary, and every read has a whole step
    // of MFMAs to complete.  With PF every issue() is followed by one prefetch; a stage's
    // copies are complete once at most the copies (and prefetches) issued after them are
    // outstanding.
#pragma unroll
    for (int c = 0; c < STAGES; ++c) {
        table(c);
        if (c < nst) {
            issue(c);
            if constexpr (PF) prefetch(c + pf_dist);
        }
    }
    table(STAGES);
    // wait until stage x's copies landed, with the copies of the `later` stages issued after
    // it (stages x+1 .. x+later) still allowed in flight; where fewer than that were issued
    // (the last stages), wait for everything
    auto wait_stage = [&](int x, auto later_c) {
        constexpr int later = decltype(later_c)::value;
        if (x + later < nst)
            wait_vmcnt(PF ? later * (kDmas + 1) + 1 : later * kDmas);
        else
            wait_vmcnt(0);
    };
    // in the order the MFMAs use them (row 0 with every column first), so that the first
    // MFMAs of a step wait only for the reads issued earliest
    auto load = [&](int sl, int u, bf16x8* af, bf16x8* bf) {
        af[0] = operand(ra[sl][u]);
#pragma unroll
        for (int t = 0; t < TN; ++t) bf[t] = operand(rb[sl][u] + (uint32_t)(64 * t));
#pragma unroll
        for (int i = 1; i < TM; ++i) af[i] = operand(ra[sl][u] + (uint32_t)(64 * i));
    };
    bf16x8 af[TM], bf[TN];    // operands of the next step to multiply
    bf16x8 af1[TM], bf1[TN];  // ... and of the step after it
    if (nst > 0) {
        wait_stage(0, std::integral_constant<int, STAGES - 1>{});  // stages 0 .. STAGES-1 issued
        __syncthreads();
        load(0, 0, af, bf);
        load(0, 1, af1, bf1);
    }
    // one stage, in ring slot SL (a compile-time constant: the loop below is unrolled over
    // the ring)
    auto stage = [&](int it, auto slot) {
        constexpr int SL = decltype(slot)::value;
        constexpr int SN = SL + 1 == STAGES ? 0 : SL + 1;
#pragma unroll
        for (int u = 0; u < NSTEP; ++u) {
            bf16x8 naf[TM], nbf[TN];  // operands of step u + 2
            if (u + 2 < NSTEP) {
                load(SL, u + 2, naf, nbf);
            } else {
                if (u + 2 == NSTEP) {
                    // stage it+1 landed (this wave's copies, then every wave's) and every
                    // wave is done reading stage it
                    wait_stage(it + 1, std::integral_constant<int, STAGES - 2>{});  // 0 .. it+STAGES-1 issued
                    __syncthreads();
                }
                load(SN, u + 2 - NSTEP, naf, nbf);  // unused after the last stage
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[i][t] = mfma32(af[i], bf[t], acc[i][t]);
            // the copies of stage it + STAGES into stage it's slot, behind the MFMAs of the
            // step that follows the barrier
            if (u + 2 == NSTEP && it + STAGES < nst) {
                issue(it + STAGES);
                if constexpr (PF) prefetch(it + STAGES + pf_dist);
            }
            // copy offsets between the MFMAs (harmless past the last stage: nothing issues
            // them)
            table_part(it, u);
            interleave_reads();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                af[i] = af1[i];
                af1[i] = naf[i];
            }
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                bf[t] = bf1[t];
                bf1[t] = nbf[t];
            }
        }
    };
    for (int it = 0; it < nst; it += STAGES) {
        stage(it, std::integral_constant<int, 0>{});
        if constexpr (STAGES > 1)
            if (it + 1 < nst) stage(it + 1, std::integral_constant<int, 1>{});
        if constexpr (STAGES > 2)
            if (it + 2 < nst) stage(it + 2, std::integral_constant<int, 2>{});
        if constexpr (STAGES > 3)
            if (it + 3 < nst) stage(it + 3, std::integral_constant<int, 3>{});
    }
    static_assert(STAGES <= 4, "ring unrolled up to four slots");

    float* out = a.out + (int64_t)split * K * J;
    const int l32 = lane & 31;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int col = j0 + wn * 32 * TN + 32 * t + l32;
        if (col >= J) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = k0 + wm * 128 + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row < K) {
                    float* o = out + (int64_t)row * J + col;
                    *o = a.accumulate ? *o + acc[i][t][v] : acc[i][t][v];
                }
            }
    }
}

}  // namespace

bool wgrad_dma_eligible(const WgradArgs& a) {
    const int64_t M = (int64_t)a.N * a.P * a.Q;
    const int64_t xbytes = (int64_t)a.N * a.H * a.W * a.C * 2;
    return a.C % 8 == 0 && a.K % 8 == 0 && M * a.K * 2 < 0x7FFFFFF0ll && xbytes < 0x7FFFFFF0ll;
}

WgradDmaPlan wgrad_dma_plan(const WgradArgs& a) {
    WgradDmaPlan p;
    const int K = a.K, J = a.R * a.S * a.C;
    const int64_t chunks = ((int64_t)a.N * a.P * a.Q + 63) / 64;
    const int forced = knob(KNOB_WGRAD_CFG);
    // the table's 16-bit coordinates; a row of no pixel stays above the image at every tap
    const bool narrow_ok = a.H + a.ph <= 32767 && a.W + a.pw <= 32767 && a.ph <= 32767 && a.pw <= 32767 && a.R <= 32768;
    // A tile and what follows from it (output tiles, least chunks of a split); returns the blocks and, by way of
    // `us`, an estimate of its time for tiles of 256 columns: launch, rounds of 256 blocks of (epilogue + chunks),
    // and the reduction of the partials.
    auto take = [&](int tk, int tj, double* us) {
        p.tk = tk;
        p.tj = tj;
        p.cfg = tk == 256 && tj == 256 ? 1 : 0;
        p.tiles = ((K + tk - 1) / tk) * ((J + tj - 1) / tj);
        // The narrow kernel's blocks take a split's chunks two at a time: small gradients (whose partials
        // cost little) go down to 2, measured 8.1 against 18.3 us with 16 for 13 x 13 x 296 -> 8 at batch 9
        // and 10.8 against 18.8 us for 13 x 13 x 8 -> 120 at batch 90; larger ones stop at 8 (28 x 28 x 128 ->
        // 128, 3 x 3, batch 64: 36.3 us with 8, 38.3 with 1)
        p.min_chunks = p.cfg == 1 ? 16 : (int64_t)K * J < 65536 ? 2 : 8;
        const int64_t by_len = chunks / p.min_chunks > 1 ? chunks / p.min_chunks : 1;
        const int64_t by_cus = 256 / p.tiles > 1 ? 256 / p.tiles : 1;
        const int64_t splits = by_len < by_cus ? by_len : by_cus;
        const double epilogue = tk == 32 ? 2.3 : tk == 64 ? 4.2 : tk == 128 ? 8.5 : 7.7;
        const double chunk = tk == 32 ? 0.58 : tk == 64 ? 0.67 : tk == 128 ? 0.92 : 1.27;
        const double partials = splits > 1 ? 2.5 + (double)(splits + 1) * K * J * 4 / 4.2e6 : 0.0;
        const double block = epilogue + chunk * (double)((chunks + splits - 1) / splits);
        *us = 3.0 + (double)((p.tiles * splits + 255) / 256) * block + partials;
        return p.tiles * splits;
    };
    // Narrow tiles up to 128 filters or 64 columns, against 256 x 256 ones (graph-replayed, with the
    // reduction of the partials): 32 x 32 x 128 -> 128 3 x 3 at batch 128 60 against 76 us, 56 x 56 x 64
    // -> 64 at batch 64 43 / 65, 36 x 39 x 384 -> 24 at batch 135 114 / 224, 1 x 1 8 -> 354 over 127 k
    // pixels 57 / 70; the segment-major kernel they replace (64-pixel stages, one 16-byte piece of 64
    // different rows per copy) took 80, 74, 276 and 83 us.
    double us;
    int64_t blocks;
    if (!narrow_ok || forced == 1 || (forced < 0 && K > 128 && J > 64))
        blocks = take(256, 256, &us);
    else if (J > 64)
        blocks = take(K <= 32 ? 32 : K <= 64 ? 64 : 128, 256, &us);
    else
        blocks = take(K <= 64 ? 64 : 256, 64, &us);
    // Short reductions leave a large tile's blocks few, and most of their time is the epilogue.  Below 192 blocks:
    // 64 filters for 256 x 64; of 256-column tiles the one with the least estimate if that gains 7%.  The
    // constants are fitted to 15 layers (64 to 1024 filters, 512 to 13600 columns) over 49 to 12800 pixels with all
    // four tiles; there the least estimate is on average 0.2% slower than the best tile and the choice never more than
    // 3.4% slower than the largest (400 -> 136 3 x 3 over 1568 pixels: 15.2 / 17.6 / 23.9 / 41.6 us with 32 / 64 /
    // 128 / 256 filters; 256 -> 512 5 x 5 over 3200: 69.8 / 43.5 / 47.7 / 44.3).
    // From 192 blocks on the large tile stays.  40 -> 104 3 x 3 over 25650 pixels, 256 blocks, would take 23.6 / 18.8 /
    // 17.2 us with 128 / 64 / 32 by itself; but in a training iteration, with the workspace left to torch's
    // allocator, the smaller workspace shares cached blocks with the other calls' buffers: 68.8 us the iteration
    // with 128, 64.2 to 72.8 with 64, 73.5 with 32.
    if (forced < 0 && narrow_ok && blocks < 192) {
        if (p.tj == 64) {
            take(64, 64, &us);
        } else {
            const int largest = p.tk;
            int tile = largest;
            double best = 0.93 * us, t;
            for (int tk = largest / 2; tk >= 32; tk /= 2) {
                take(tk, 256, &t);
                if (t < best) {
                    best = t;
                    tile = tk;
                }
            }
            take(tile, 256, &us);
        }
    }
    p.resident_blocks = 256;  // one block per CU
    // wide kernel: 48-pixel stages in a three-deep ring (measured best of 32 / 48 / 64)
    p.pix = 48;
    const int px = knob(KNOB_WGRAD_PIX);
    if (px == 32 || px == 64) p.pix = px;
    return p;
}

template <bool LIN>
static void launch_rows(int pix, bool pf, dim3 grid, const WgradDmaArgs& ka, hipStream_t stream) {
    switch (pix) {
        case 32: hipLaunchKernelGGL((wgrad_rows_kernel<32, 4, false, LIN>), grid, dim3(512), 0, stream, ka); break;
        case 64: hipLaunchKernelGGL((wgrad_rows_kernel<64, 2, false, LIN>), grid, dim3(512), 0, stream, ka); break;
        default:
            if (pf)
                hipLaunchKernelGGL((wgrad_rows_kernel<48, 3, true, LIN>), grid, dim3(512), 0, stream, ka);
            else
                hipLaunchKernelGGL((wgrad_rows_kernel<48, 3, false, LIN>), grid, dim3(512), 0, stream, ka);
            break;
    }
}

hipError_t launch_wgrad_dma(const WgradArgs& a, hipStream_t stream) {
    WgradDmaArgs ka;
    ka.a = a;
    ka.div_q = make_fastdiv((uint32_t)a.Q);
    ka.div_pq = make_fastdiv((uint32_t)a.P * (uint32_t)a.Q);
    // L2 prefetch of a later stage: off by default (measured ~9% slower on the training
    // layer once the reads and MFMAs are interleaved); the prefetch knob (stages ahead)
    // turns it on
    const int pf = knob(KNOB_WGRAD_PF);
    ka.pf_dist = pf > 0 ? pf : 0;
    const WgradDmaPlan p = wgrad_dma_plan(a);
    const dim3 grid((unsigned)(p.tiles * a.splits));
    if (p.cfg == 1) {
        // linear copy addressing: stride 1, output the input's size, whole 256-column
        // blocks of one tap
        const bool lin = a.sh == 1 && a.sw == 1 && a.P == a.H && a.Q == a.W && a.C % 256 == 0;
        if (lin)
            launch_rows<true>(p.pix, ka.pf_dist > 0, grid, ka, stream);
        else
            launch_rows<false>(p.pix, ka.pf_dist > 0, grid, ka, stream);
    } else if (p.tj == 64 && p.tk == 64) {
        hipLaunchKernelGGL((wgrad_narrow_kernel<1, 1, 2, 2, 64>), grid, dim3(512), 0, stream, ka);
    } else if (p.tj == 64) {
        hipLaunchKernelGGL((wgrad_narrow_kernel<2, 2, 4, 1, 32>), grid, dim3(512), 0, stream, ka);
    } else if (p.tk == 32) {
        hipLaunchKernelGGL((wgrad_narrow_kernel<1, 2, 1, 4, 32>), grid, dim3(512), 0, stream, ka);
    } else if (p.tk == 64) {
        hipLaunchKernelGGL((wgrad_narrow_kernel<2, 2, 1, 4, 32>), grid, dim3(512), 0, stream, ka);
    } else {
        hipLaunchKernelGGL((wgrad_narrow_kernel<4, 2, 1, 4, 32>), grid, dim3(512), 0, stream, ka);
    }
    return hipGetLastError();
}

}  // namespace tbn
