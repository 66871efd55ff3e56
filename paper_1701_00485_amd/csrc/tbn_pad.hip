// tbn_pad.hip -- what is prepared ahead of a GEMM: the codes of the transposed, flipped filters for
// backward-data; and for channel counts that are no multiple of 8 the copies that bring such a layer
// to the LDS-DMA kernels (16-byte pieces of 8 bf16 channels).  A tensor is copied into Cp channels, a multiple
// of 8, with zeros beyond the real ones; a filter's two-bit codes are re-packed from rows of C to rows of Cp channels (the codes
// of the added channels multiply zeros, so they may be anything: their bits are clear).
#include "tbn_device.h"
#include "tbn_kernels.h"

namespace tbn {

namespace {

// One 8-channel group of one pixel: channels c0 .. c0 + 7, zeros from C on.
//
// bf16 rows of an odd or uneven width start at any 2-byte offset, so the group is read as the
// (at most five) 4-byte words that hold it and shifted into place: a quarter of the load
// instructions of a load per channel.  A last word that would reach past the end of the tensor
// is read as 2 bytes.
__device__ __forceinline__ u32x4 load_group(const uint16_t* __restrict__ x, int64_t total, int64_t e0, int valid) {
    const uint32_t* const xw = reinterpret_cast<const uint32_t*>(x);
    const int64_t w0 = e0 >> 1;
    const int odd = (int)(e0 & 1);
    const int words = (valid + odd + 1) >> 1;
    uint32_t w[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        w[j] = 0;
        if (j < words) w[j] = 2 * (w0 + j) + 1 < total ? xw[w0 + j] : (uint32_t)x[2 * (w0 + j)];
    }
    u32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = odd ? (w[j] >> 16) | (w[j + 1] << 16) : w[j];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (2 * j + 1 >= valid) r[j] &= 0xFFFFu;
        if (2 * j >= valid) r[j] = 0;
    }
    return r;
}

__device__ __forceinline__ u32x4 load_group(const float* __restrict__ x, int64_t, int64_t e0, int valid) {
    float v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = c < valid ? x[e0 + c] : 0.0f;
    return u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}

template <typename T>
__device__ __forceinline__ void pad_group(const PadArgs& a, int64_t i) {
    const int groups = a.Cp / 8;
    if (i >= a.pixels * groups) return;
    const int64_t pix = a.small ? (int64_t)fdiv((uint32_t)i, a.div_groups) : i / groups;
    const int c0 = (int)(i - pix * groups) * 8;
    *reinterpret_cast<u32x4*>(a.xp + pix * a.Cp + c0) =
        load_group(reinterpret_cast<const T*>(a.x), a.pixels * a.C, pix * a.C + c0, min(a.C - c0, 8));
}

// One packed word of the forward filters re-packed from C to Cp channels.
__device__ __forceinline__ void repack_fwd_word(const RepackFwdArgs& r, int64_t gid) {
    // word (filter block, element block, filter, quarter) of the re-packed codes: elements
    // 64 eb + 16 q .. + 15 of filter k.  Cp is a multiple of 8, so each half of the word lies in
    // one tap and takes a run of at most 8 consecutive elements of the C-channel filter, which
    // lie in at most two of its words.
    if (gid >= r.words) return;
    const uint32_t g32 = (uint32_t)gid;  // < 2^29 words, checked by the host
    const uint32_t row = g32 & 255, blk = g32 >> 8;
    const uint32_t kb = fdiv(blk, r.div_nbp);
    const uint32_t e0 = (blk - kb * r.nbp) * 64 + (row & 3) * 16;
    const uint32_t* const src = r.codes + (int64_t)kb * r.nb * 256 + (row >> 2) * 4;  // filter's words
    uint32_t run[2], lo[2], hi[2], at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t e = e0 + 8 * h;
        const uint32_t rs = fdiv(e, r.div_cp);
        const uint32_t c0 = e - rs * (uint32_t)r.Cp;
        run[h] = rs < (uint32_t)r.taps && c0 < (uint32_t)r.C ? min((uint32_t)r.C - c0, 8u) : 0u;
        const uint32_t i = run[h] ? rs * (uint32_t)r.C + c0 : 0u;
        const uint32_t last = run[h] ? i + run[h] - 1 : 0u;
        at[h] = i & 15;
        lo[h] = src[(i >> 6) * 256 + ((i & 63) >> 4)];
        hi[h] = src[(last >> 6) * 256 + ((last & 63) >> 4)];
    }
    uint32_t word = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c) {
            const uint32_t p = at[h] + c;  // element within the first word, past 15 in the second
            const uint32_t w = p < 16 ? lo[h] : hi[h], b = 16 * (p & 1) + ((p & 15) >> 1);
            const uint32_t e = 8 * h + c, to = 16 * (e & 1) + (e >> 1);
            // magnitude bit b and sign bit b + 8 move together
            const uint32_t code = (w >> b) & 0x101u;
            word |= c < run[h] ? code << to : 0u;
        }
    }
    r.out[gid] = word;
}

// One packed word of the codes of the transposed, spatially flipped filters [C][R][S][K]
// (backward-data operand): 16 consecutive elements take one code each from up to 16 filters, whose
// words are all requested before the first is used (a launch that is all latency: 4.0 us in a training
// iteration, 4.4 with a loop that loads and uses one word at a time).
// K may exceed the layer's Kreal filters (a gradient padded to a multiple of 8 channels): filters
// k >= Kreal read the zero padding bits of the last 64-filter block and get scale 0.
__device__ __forceinline__ void repack_bwd_word(const RepackBwdArgs& r, int64_t gid) {
    // every count below is < 2^31 (R*S*C and R*S*K < 2^30, checked by the host)
    const uint32_t K = (uint32_t)r.K, S = (uint32_t)r.S, R = (uint32_t)r.R, C = (uint32_t)r.C;
    if (gid < r.words) {
        const uint32_t g32 = (uint32_t)gid, row = g32 & 255, blk = g32 >> 8;
        const uint32_t cblk = fdiv(blk, r.div_nbt);
        const uint32_t c = cblk * 64 + (row >> 2);
        const uint32_t et0 = (blk - cblk * r.nbt) * 64 + (row & 3) * 16;
        uint32_t word = 0;
        if (c < C && et0 < r.nt) {
            uint32_t rs = fdiv(et0, r.div_k), k = et0 - rs * K;
            uint32_t i = (R * S - 1 - rs) * C + c;  // element of forward filter k (flipped tap)
            uint32_t src[16], bit[16];
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
                const uint32_t at = ((k >> 6) * r.nb + (i >> 6)) * 256 + (k & 63) * 4 + ((i & 63) >> 4);
                src[e] = et0 + e < r.nt ? r.codes[at] : 0u;
                bit[e] = 16 * (i & 1) + ((i & 15) >> 1);
                if (++k == K) {
                    k = 0;
                    i -= C;
                }
            }
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e)  // magnitude bit b and sign bit b + 8 move together
                word |= ((src[e] >> bit[e]) & 0x101u) << (16 * (e & 1) + (e >> 1));
        }
        r.codes_t[gid] = word;
    }
    if (gid < r.pairs) {
        uint32_t v = 0;
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
            const uint32_t et = 2 * (uint32_t)gid + h;
            if (et < r.nt) {
                const uint32_t kk = et - fdiv(et, r.div_k) * K;
                uint32_t b = kk < (uint32_t)r.Kreal ? f32_to_bf16_bits(r.alpha[kk]) : 0u;
                if ((b & 0x7F80u) == 0) b = 0;  // a denormal scale is flushed: exponent + 1 would not double it
                v |= b << (16 * h);
            }
        }
        r.apair[gid] = v;
    }
}

// Up to two tensors and one set of codes in one launch (none reads what another writes, and each
// is too short to be worth a launch of its own): a thread per 8-channel group or packed word.
template <typename T>
__global__ __launch_bounds__(256) void prepare_kernel(const PadArgs a, const PadArgs b, const RepackFwdArgs f,
                                                      const RepackBwdArgs t) {
    int64_t block = blockIdx.x;
    if (block < a.blocks) return pad_group<T>(a, block * 256 + threadIdx.x);
    block -= a.blocks;
    if (block < b.blocks) return pad_group<uint16_t>(b, block * 256 + threadIdx.x);
    block -= b.blocks;
    if (f.words)
        repack_fwd_word(f, block * 256 + threadIdx.x);
    else
        repack_bwd_word(t, block * 256 + threadIdx.x);
}

}  // namespace

PadArgs make_pad(const void* x, int64_t pixels, int32_t C, int32_t Cp, void* xp) {
    PadArgs a;
    a.x = x;
    a.xp = reinterpret_cast<uint16_t*>(xp);
    a.pixels = pixels;
    a.C = C;
    a.Cp = Cp;
    const int64_t n = pixels * (Cp / 8);
    a.blocks = (n + 255) / 256;
    a.small = n < 0x7FFFFFFF - 256;
    a.div_groups = make_fastdiv((uint32_t)(Cp / 8));
    return a;
}

static hipError_t launch_prepare(int x_f32, const PadArgs& a, const PadArgs& b, const RepackFwdArgs& f,
                                 const RepackBwdArgs& t, hipStream_t stream) {
    const int64_t items = f.words ? f.words : (t.words > t.pairs ? t.words : t.pairs);
    const int64_t blocks = a.blocks + b.blocks + (items + 255) / 256;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (x_f32)
        hipLaunchKernelGGL((prepare_kernel<float>), dim3((unsigned)blocks), dim3(256), 0, stream, a, b, f, t);
    else
        hipLaunchKernelGGL((prepare_kernel<uint16_t>), dim3((unsigned)blocks), dim3(256), 0, stream, a, b, f, t);
    return hipGetLastError();
}

hipError_t launch_pad_channels(const PadArgs& a, const PadArgs& b, hipStream_t stream) {
    return launch_prepare(0, a, b, RepackFwdArgs{}, RepackBwdArgs{}, stream);
}

hipError_t launch_pad_fwd(const PadArgs& a, int x_f32, const uint32_t* codes, int32_t K, int32_t taps,
                          uint32_t* codes_p, hipStream_t stream) {
    RepackFwdArgs r;
    r.codes = codes;
    r.out = codes_p;
    r.C = a.C;
    r.Cp = a.Cp;
    r.taps = taps;
    r.nb = (int32_t)(((int64_t)taps * a.C + 63) / 64);
    r.nbp = (uint32_t)(((int64_t)taps * a.Cp + 63) / 64);
    r.words = (int64_t)((K + 63) / 64) * r.nbp * 256;
    r.div_cp = make_fastdiv((uint32_t)a.Cp);
    r.div_nbp = make_fastdiv(r.nbp);
    if (r.words > ((int64_t)1 << 29)) return hipErrorInvalidValue;  // the LDS-DMA kernel's limit, 2 GiB
    return launch_prepare(x_f32, a, PadArgs{}, r, RepackBwdArgs{}, stream);
}

hipError_t launch_repack_bwd(const uint32_t* codes, const float* alpha, int32_t K, int32_t Kreal, int32_t R,
                             int32_t S, int32_t C, uint32_t* codes_t, uint32_t* apair, const PadArgs& dy,
                             hipStream_t stream) {
    RepackBwdArgs r;
    r.codes = codes;
    r.alpha = alpha;
    r.codes_t = codes_t;
    r.apair = apair;
    r.K = K;
    r.Kreal = Kreal;
    r.R = R;
    r.S = S;
    r.C = C;
    r.nb = (uint32_t)(((int64_t)R * S * C + 63) / 64);
    r.nt = (uint32_t)((int64_t)R * S * K);
    r.nbt = (r.nt + 63) / 64;
    r.words = (int64_t)((C + 63) / 64) * r.nbt * 256;
    r.pairs = (int64_t)r.nbt * 32;
    r.div_k = make_fastdiv((uint32_t)K);
    r.div_nbt = make_fastdiv(r.nbt);
    return launch_prepare(0, dy, PadArgs{}, RepackFwdArgs{}, r, stream);
}

}  // namespace tbn
