// Matrix-core kernel for 1x1 and 3x3 convolutions: one wave per block of at most 64 output pixels and slice of the input
// channels, no workgroup-wide pipeline.
//
// As in tbn_conv_mfma.hip only the R = p / gcd(F, p) distinct +-1 filters are computed and channel o = u + t * R is
// written as alpha(o) * Z[u] (Eq. 4-5 on the flattened (O, C, kh, kw) weight; the paper's replicated-channel example in
// Section "CNN Architectures").
//
// What bounds these layers is neither the matrix pipe nor memory but the work around them: in the block kernel a workgroup zeroed its patch, transposed the filter bits in LDS (2.8 us), staged the input with 4-byte
// LDS stores (two elements each, colliding on the banks) behind a barrier per 32 channels, and every wave expanded the
// filter operands anew for its own 16 pixels.  Here
//   * a wave owns 64 (or 32) pixels x up to four tiles of MT filters over its own channels: an expanded filter operand
//     serves all pixel tiles and planes, and no barrier is needed in the channel loop, because the wave stages its
//     channels in LDS that only it touches; waves with different channels of the same pixels add their sums through LDS
//     once, at the end;
//   * a lane stages eight channels of one pixel: eight loads whose addresses are a scalar channel base plus one 32-bit
//     lane offset, converted in registers (float32: the exact three-term bf16 split), one 16-byte LDS store per plane.
//     The patch lies in LDS as [plane][group of 8 channels][pixel][16 bytes]: consecutive pixels are consecutive 16-byte
//     pieces for the stores and for the operand reads, so neither collides, and a tap is an immediate offset (dx) on one
//     of three row registers (dy);
//   * the filter bits never pass through LDS: the 8 channels x 9 taps that a lane supplies are 72 consecutive bits of the
//     tile (c * 9 + tap runs fastest), fetched with one unaligned window per chunk; bits `tap` of two neighbouring
//     channels are nine apart, so one v_pk_lshlrev_b16 puts them on the two sign positions and one v_and_or merges the
//     pattern of 1.0: two instructions per register of the operand;
//   * barriers of the final reduction order LDS only and the scalars of the replicas sit in lanes: a full barrier or a
//     load between the stores waits for every store before it (1 - 2 us each time).
//
// Measured (us per call, this kernel against tbn_conv_mfma.hip; 3x3, N x C x map -> O):
//   float32   32 x 64 x 56^2 -> 64, k = 4: 23.0 / 36.9    128 x 256 x 14^2 -> 256, k = 8: 24.6 / 28.1
//             8 x 64 x 112^2 -> 64, k = 4: 23.3 / 37.0    16 x 16 x 100^2 -> 32, k = 4: 15.0 / 44.6
//             128 x 256 x 14^2 -> 256, k = 3 (256 filters, one alpha): 101 / 127
//   bfloat16  32 x 64 x 56^2 -> 64, k = 4: 13.5 / 31.3    128 x 256 x 14^2 -> 256, k = 8: 15.8 / 22.7
//   1x1       32 x 64 x 56^2 -> 256, k = 4 / 2, float32 / bfloat16: 27.5 / 30.2, 29.6 / 39.1
// Layers it is slower on go to that kernel (prefer_wave).
// Stamps (bfloat16 56^2, all waves resident at once): set-up 1.0 us, first loads to LDS 3.7, product 1.3, sums 0.5, stores
// 2.0: the kernel is bound by its chain of memory latencies (25.7 MB are 5 us at copy rate), float32 at 256 channels by
// the matrix pipe as well (three planes: 5.8 us).
#include "tbn_common.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

namespace tbn {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));

constexpr int kMaxWaves = 8;

// n / d for 0 <= n < 2^31 by a multiplication (Granlund and Montgomery, "Division by invariant integers using multiplication",
// 1994; the set-up of a wave divides a dozen times; as instructions of a general
// division that was 1 us before the first load)
struct FastDiv {
    uint32_t mul, shift, d;
    FastDiv() = default;
    explicit FastDiv(int64_t v) : shift(0), d(static_cast<uint32_t>(v)) {
        while ((uint64_t(1) << shift) < d) ++shift;
        mul = static_cast<uint32_t>(((uint64_t(1) << 32) * ((uint64_t(1) << shift) - d)) / d + 1);
    }
    __device__ __forceinline__ int div(int n) const {
        return static_cast<int>((__umulhi(static_cast<uint32_t>(n), mul) + static_cast<uint32_t>(n)) >> shift);
    }
};

struct WaveConvParams {
    int64_t HW;             // elements of an input plane
    int64_t plane_out;      // Ho * Wo
    int64_t O, F, R, p;
    int32_t C, H, W, Ho, Wo;
    int32_t sh, sw, ph, pw;
    int32_t n_words, aligned, n_alpha, relu;
    int32_t rows, cols, n_colblk, n_blk;   // pixel block, column blocks per row of blocks, blocks per image
    int32_t PR, PC, pitch;  // patch rows and columns in LDS, LDS pixels from one row to the next
    int32_t step;           // tile bits from one chunk of a wave to its next, modulo p
    FastDiv d_img, d_blk, d_col, d_cols, d_items, d_group;   // workgroups per image, blocks per grid row, column blocks, columns, loads per patch row and channel
    int32_t even;           // bfloat16, 3x3: loads begin at even elements of a plane
    int32_t ks_log2, ps;    // channel slices (power of two) and pixel blocks per workgroup
    int32_t n_chunks;
};

// px: neighbouring pixels in the 4 bytes that a lane of a 1x1 layer loads of a channel
template <typename XT> struct WTraits;
template <> struct WTraits<float> { static constexpr int planes = 3, px = 1; };
template <> struct WTraits<uint16_t> { static constexpr int planes = 1, px = 2; };

// LDS pixels of a patch (the last one takes the stores of idle lanes) and the loads per lane and channel that cover them: pixels or pairs
// of one channel group after the other, or (RUNS) runs of four pixels of all groups at once, at most run_limit per group.
constexpr int kCapF32 = 100;   // two workgroups of eight waves per CU
constexpr int slots_of(int CAP) { return CAP == kCapF32 ? 104 : CAP; }
constexpr int loads_of(bool f32, int CAP, bool RUNS) { return RUNS ? 1 : f32 ? (CAP - 1 + 63) / 64 : (CAP - 1 + 127) / 128; }
constexpr int kRunLimit = 32;
// registers: what the LDS lets share a SIMD anyway
constexpr int wave_bound(bool f32, int MT, int T, int PW, int NFT, int CAP) {
    if (NFT * PW > 64) return 2;
    if (T == 1) return MT == 16 ? 3 : 4;
    return f32 ? (CAP <= 100 ? 4 : CAP == 128 ? 3 : 2) : CAP == 128 ? 4 : 3;
}

__device__ __forceinline__ uint32_t load_raw(const char *p) {   // 4 bytes, 2-byte aligned for bfloat16 pairs
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}

__device__ __forceinline__ uint32_t pack_hi16(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }

__device__ __forceinline__ void pack_out(const float (&w)[4], float (&r)[4]) { __builtin_memcpy(r, w, 16); }
__device__ __forceinline__ void pack_out(const float (&w)[8], uint16_t (&r)[8]) {   // round to nearest even, NaN stays NaN
    uint32_t p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(p[e]) : "v"(w[2 * e]), "v"(w[2 * e + 1]));
    __builtin_memcpy(r, p, 16);
}

template <int MT> struct Acc;
template <> struct Acc<32> {
    typedef f32x16_t type;
    static constexpr int n = 16;
    static __device__ __forceinline__ type mma(bf16x8_t a, bf16x8_t b, type c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int i, int q) { return 8 * (i / 4) + 4 * q + i % 4; }
};
template <> struct Acc<16> {
    typedef f32x4_t type;
    static constexpr int n = 4;
    static __device__ __forceinline__ type mma(bf16x8_t a, bf16x8_t b, type c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int i, int q) { return 4 * q + i; }
};

// XT: input and output type; MT: filters (and pixels) of an MFMA tile; T: taps; PW: pixels per wave; NFT: filter tiles
// per wave; kCap: LDS pixels of a patch; ALL: float32, add what the split of small activations leaves out
template <typename XT, int MT, int T, int PW, int NFT, int kCap, bool RUNS, bool ALL = false>
__global__ __launch_bounds__(64 * kMaxWaves, (wave_bound(sizeof(XT) == 4, MT, T, PW, NFT, kCap) - (ALL ? 1 : 0))) void conv_wave_kernel(const XT *__restrict__ x, XT *__restrict__ y,
                                                                                         const uint32_t *__restrict__ tile,
                                                                                         const float *__restrict__ alpha, WaveConvParams P) {
    constexpr int NP = WTraits<XT>::planes;
    constexpr int G = 64 / MT, CK = 8 * G;          // channel groups of 8 per MFMA step, channels per chunk
    constexpr int J = PW / MT;                      // pixel tiles per wave
    constexpr int LP = RUNS ? 4 : WTraits<XT>::px;  // pixels per load
    constexpr int IT = loads_of(sizeof(XT) == 4, kCap, RUNS);
    constexpr int kSlots = slots_of(kCap), kGroup = kSlots * 16, kPlane = G * kGroup, kRegion = NP * kPlane;
    constexpr int NA = Acc<MT>::n;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave & ((1 << P.ks_log2) - 1), ps = wave >> P.ks_log2, KS = 1 << P.ks_log2;
    const int ln = lane & (MT - 1), q = lane / MT;

    // all workgroups of an image on one XCD (ids are dealt round-robin): the patches overlap and the filter blocks share them
    uint32_t blk_x, blk_z;
    int64_t img;
    {
        const uint32_t lid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
        const uint32_t per_img = gridDim.x * gridDim.z, n_img = gridDim.y;
        const uint32_t xcd = lid & 7, slot = lid >> 3, full = (n_img / 8) * per_img;
        uint32_t inner;
        if (slot < full) {
            const uint32_t d = static_cast<uint32_t>(P.d_img.div(static_cast<int>(slot)));
            inner = slot - d * per_img;
            img = d * 8 + xcd;
        } else {
            const uint32_t rest = lid - full * 8, d = static_cast<uint32_t>(P.d_img.div(static_cast<int>(rest)));
            inner = rest - d * per_img;
            img = (n_img / 8) * 8 + d;
        }
        blk_z = static_cast<uint32_t>(P.d_blk.div(static_cast<int>(inner)));
        blk_x = inner - blk_z * gridDim.x;
    }
    const int blk = static_cast<int>(blk_x) * P.ps + ps;
    const bool live = blk < P.n_blk;                 // a wave past the last block only takes part in the barriers
    const int rb = live ? P.d_col.div(blk) : 0, cb = live ? blk - rb * P.n_colblk : 0;
    const int row0 = rb * P.rows, col0 = cb * P.cols;
    const int rows = P.Ho - row0 < P.rows ? P.Ho - row0 : P.rows;
    const int cols = P.Wo - col0 < P.cols ? P.Wo - col0 : P.cols;
    // slots of the block's pixels, P.cols to a row (a narrower last column block leaves some of them unused)
    const int PX = live ? rows * P.cols : 0;
    const int64_t u0 = int64_t(blk_z) * (MT * NFT);

    // ---- staging: which input elements a lane reads and where they go -----------------------------------
    // RUNS: a lane takes a run of four neighbouring pixels of a patch row in one channel group, one load per channel: a load takes
    // the CU's load path about ten cycles however little a lane takes of it, and 512 of them per chunk and CU (16 waves, 16 channels of
    // two pixels a lane, float32) were 1.9 us in front of the first product, 0.7 now, and as much beside the second chunk's (128 x 256 x
    // 14^2 -> 256, k = 8: 22.6 us before, 21.3 now; 16 x 512 x 7^2 -> 512, k = 8 19.2 / 17.3).  Else a load covers LP neighbouring pixels of an image row (one where a 1x1 layer
    // strides).  A load is moved so that it stays inside the plane (1x1: inside the row), and bfloat16 loads of 3x3 layers begin at
    // even elements where all planes do (pairs at odd ones took 10 cycles instead of 7: 32 x 64 x 56^2 -> 64, k = 4 13.2 us / 12.0; runs
    // for its tiles of 16 filters, two per lane, cost the registers of the operand reads, 12.4 - 13.8).  738 drawn layers with runs: 1.04 times as
    // fast as with pixels and pairs on the mean; three are more than 3 % slower, float32 with full patches on 3000 and more waves (26 x 512 x 37 x
    // 36 -> 64, k = 4 0.91; neighbours of these are faster, by no rule that was found).  Even pairs: 1.02 - 1.1 on the mean of a form,
    // single layers 0.94 (7 x 160 x 66 x 64 -> 128, k = 2 19.9 us / 21.2).  Positions outside the image stay zero.
    uint32_t goff[IT];     // byte offset inside a channel plane (RUNS: with that of the lane's channel group)
    uint32_t loff[IT][(LP + 1) / 2];   // byte offsets inside a channel group of the patch (RUNS: with that of the group), two to a word
    auto lds_off = [&](int it, int h) __attribute__((always_inline)) { return LP == 1 ? loff[it][0] : h & 1 ? loff[it][h / 2] >> 16 : loff[it][h / 2] & 0xffffu; };
    const int per_group = P.PR * static_cast<int>(P.d_items.d);   // RUNS: loads per channel of a group
    {
        const int iy0 = row0 * P.sh - P.ph, ix0 = col0 * P.sw - P.pw;
        const int sy = T == 1 ? P.sh : 1, sx = T == 1 ? P.sw : 1;         // image steps between patch positions
        const int per = T == 9 ? LP : LP == 2 && sx == 1 ? 2 : 1;         // patch pixels per load
        const int n_items = live ? (RUNS ? G : 1) * per_group : 0;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int v = it * 64 + lane, g = RUNS ? P.d_group.div(v) : 0, w = v - g * per_group;
            const int py = P.d_items.div(w), px = (w - py * static_cast<int>(P.d_items.d)) * per;
            const int iy = iy0 + py * sy, ix = ix0 + px * sx;
            if constexpr (T == 9 && LP > 1) {
                const bool ok = v < n_items && iy >= 0 && iy < P.H;
                const int flat = iy * P.W, last = static_cast<int>(P.HW) - LP;
                int at = flat + ix - ((flat + ix0) & P.even);
                at = at < 0 ? 0 : at > last ? last : at;
                goff[it] = ok ? static_cast<uint32_t>(at) * static_cast<uint32_t>(sizeof(XT)) + static_cast<uint32_t>(8 * g) * static_cast<uint32_t>(P.HW * sizeof(XT)) : 0u;
                const int c0 = at - flat, p0 = c0 - ix0;                 // image and patch column of the load's first element
                const uint32_t base = static_cast<uint32_t>((g * kSlots + py * P.pitch + p0) * 16);
#pragma unroll
                for (int h = 0; h < LP; ++h) {   // (a moved load's elements may be another one's too)
                    const bool use = ok && static_cast<unsigned>(c0 + h) < static_cast<unsigned>(P.W) && static_cast<unsigned>(p0 + h) < static_cast<unsigned>(P.PC);
                    const uint32_t off = use ? base + 16u * h : (kSlots - 1) * 16u;
                    loff[it][h / 2] = h & 1 ? loff[it][h / 2] | (off << 16) : off;
                }
            } else {
                const bool ok = v < n_items && iy >= 0 && iy < P.H && ix > -per && ix < P.W;   // some of its pixels lie in the image
                int sx0 = ix;                                             // image column where the load starts
                if (LP == 2) sx0 = ix < 0 ? 0 : ix > P.W - 2 ? P.W - 2 : ix;
                goff[it] = ok ? static_cast<uint32_t>((iy * P.W + sx0) * static_cast<int>(sizeof(XT))) : 0u;
#pragma unroll
                for (int h = 0; h < LP; ++h) {
                    const int d = sx0 + h - ix;                          // which of the load's patch pixels this element is
                    const bool use = ok && d >= 0 && d < per && px + d < P.PC;
                    const uint32_t off = static_cast<uint32_t>((use ? py * P.PC + px + d : kSlots - 1) * 16);
                    loff[it][h / 2] = h & 1 ? loff[it][h / 2] | (off << 16) : off;
                }
            }
        }
    }
    unsigned char *region = lds_raw + wave * kRegion;
    const int64_t hw = P.HW;
    const char *x_img = reinterpret_cast<const char *>(x + img * P.C * hw);
    const int64_t hwb = hw * static_cast<int64_t>(sizeof(XT));
    // RUNS: the first channel in its chunk of this lane's load, worked out where the last channels need it.  With one filter tile and float32 patches
    // of up to 100 pixels the kernel has 128 registers for four waves per SIMD: held over the loop, this and the unpacked LDS offsets (below) were
    // two too many, and spilled; without either it takes 127 and the same time (128 x 256 x 14^2 -> 256, k = 8 21.9 us).
    constexpr bool kTight = RUNS && sizeof(XT) == 4 && kCap == kCapF32 && NFT * PW <= 64;
    static_assert(!RUNS || IT == 1, "");
    auto first_channel = [&]() __attribute__((always_inline)) {
        int l = lane;
        asm volatile("" : "+v"(l));
        return 8 * P.d_group.div(l);
    };

    // Loads of a 1x1 layer run two chunks ahead (a chunk is a handful of MFMAs), those of a 3x3 layer one.
    constexpr int kSets = T == 1 ? 2 : 1;
    constexpr int GL = RUNS ? 1 : G, RW = RUNS ? static_cast<int>(sizeof(XT)) : 1;   // groups a lane loads of, words per load
    uint32_t staged[kSets][GL][IT][8][RW];
    auto load_chunk = [&](int chunk, auto set_c) {
        auto &st = staged[decltype(set_c)::value];
        const int c0 = chunk * CK;
        const char *b = x_img + c0 * hwb;
        if constexpr (RUNS) {
            const int c_left = P.C - c0;
            if (c_left >= CK) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
#pragma unroll
                    for (int it = 0; it < IT; ++it) __builtin_memcpy(st[0][it][j], b + goff[it], 4 * RW);
                    b += hwb;
                }
            } else {
                // Past the last channel: that one again, dropped below.  Lanes without a load stay at the first element of channels of the chunk.
                // 32-bit offsets, one addition per channel: a 64-bit address and product per lane and channel, which the compiler also moved in front
                // of the first load, took back what runs give one-chunk waves (float32, 8 x 16 x 68^2 -> 512, k = 4 52.4 us by pixels, 55.1 with
                // them, 51.6 now; bfloat16, 2 x 24 x 7^2 -> 96, k = 2 5.5 / 5.9 / 5.5).
                const uint32_t plane = static_cast<uint32_t>(hwb);
                const int first = first_channel();
                uint32_t at = goff[0];
                if (first >= c_left && at != 0u) at -= static_cast<uint32_t>(first - (c_left - 1)) * plane;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    __builtin_memcpy(st[0][0][j], b + at, 4 * RW);
                    at += first + j + 1 < c_left ? plane : 0u;
                }
            }
        } else {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
#pragma unroll
                    for (int it = 0; it < IT; ++it) st[g][it][j][0] = load_raw(b + goff[it]);
                    b += c0 + g * 8 + j + 1 < P.C ? hwb : 0;   // past the last channel: that one again, dropped below
                }
        }
    };
    uint32_t low_bits = 0u;   // ALL: of the third terms; the low 16 have no place in a bfloat16 (activations below 2^-110)
    auto store_chunk = [&](int chunk, auto set_c) __attribute__((always_inline)) {
        auto &st = staged[decltype(set_c)::value];
        const int c_left = P.C - chunk * CK;
        if constexpr (kTight) asm volatile("" : "+v"(loff[0][0]), "+v"(loff[0][1]));   // unpacked here, for each chunk
        if (c_left < CK) {   // channels past the last one are zeros
            const int first = RUNS ? first_channel() : 0;
#pragma unroll
            for (int g = 0; g < GL; ++g)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int it = 0; it < IT; ++it)
#pragma unroll
                        for (int e = 0; e < RW; ++e)
                            st[g][it][j][e] = (RUNS ? first : 8 * g) + j < c_left ? st[g][it][j][e] : 0u;
        }
#pragma unroll
        for (int g = 0; g < GL; ++g)
#pragma unroll
            for (int it = 0; it < IT; ++it) {
#pragma unroll
                for (int h = 0; h < LP; ++h) {
                    unsigned char *dst = region + lds_off(it, h) + (RUNS ? 0 : g * kGroup);
                    if constexpr (NP == 1) {   // channel pairs of one pixel
                        u32x4_t v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_perm(st[g][it][2 * e + 1][h / 2], st[g][it][2 * e][h / 2], h & 1 ? 0x07060302u : 0x05040100u);
                        *reinterpret_cast<u32x4_t *>(dst) = v;
                    } else {   // exact three-term split: the top 8 significand bits, the next 8, the rest
                        u32x4_t v0, v1, v2;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t sa = st[g][it][2 * e][h], sb = st[g][it][2 * e + 1][h];
                            const float a = __uint_as_float(sa), b = __uint_as_float(sb);
                            const float a1 = a - __uint_as_float(sa & 0xffff0000u), b1 = b - __uint_as_float(sb & 0xffff0000u);
                            const float a2 = a1 - __uint_as_float(__float_as_uint(a1) & 0xffff0000u);
                            const float b2 = b1 - __uint_as_float(__float_as_uint(b1) & 0xffff0000u);
                            if (ALL) low_bits |= __float_as_uint(a2) | __float_as_uint(b2);
                            v0[e] = pack_hi16(sa, sb);
                            v1[e] = pack_hi16(__float_as_uint(a1), __float_as_uint(b1));
                            v2[e] = pack_hi16(__float_as_uint(a2), __float_as_uint(b2));
                        }
                        *reinterpret_cast<u32x4_t *>(dst) = v0;
                        *reinterpret_cast<u32x4_t *>(dst + kPlane) = v1;
                        *reinterpret_cast<u32x4_t *>(dst + 2 * kPlane) = v2;
                    }
                }
            }
    };

    // ---- filter bits: cyclic tile position of the lane's window, one per filter tile ---------------------
    constexpr int kBits = 8 * T;                     // bits a lane supplies per chunk
    const int32_t p32 = static_cast<int32_t>(P.p);
    int32_t pos[NFT];
    typedef uint32_t words_t __attribute__((ext_vector_type(T == 1 ? 2 : 4)));
    typedef words_t words_a4_t __attribute__((aligned(4)));
    words_t raw[NFT];
#pragma unroll
    for (int ft = 0; ft < NFT; ++ft) {
        int64_t u = u0 + ft * MT + ln;
        if (u >= P.R) u = 0;                         // its sums are dropped
        const int64_t f = u * P.F + (ks * CK + 8 * q) * T;
        pos[ft] = static_cast<int32_t>(P.aligned ? f : f % P.p);   // whole filters: u < R = p / F (channels past C belong to zero activations)
    }
    // One load per window: the lanes' windows lie in lines of their own, and a load takes the CU's load path as many cycles as it
    // touches lines, whatever its width.  Against four loads of a word (3x3, bfloat16): 27 x 512 x 35^2 -> 256, k = 2 122 us before,
    // 103 now; 5 x 512 x 8 x 7 -> 256, k = 4, stride 2 11.7 / 9.8; 128 x 256 x 14^2 -> 256, k = 8, float32 26.8 / 26.9 (graph replays; through the
    // wrapper, at a higher clock, 24.7 / 24.5); 99 drawn bfloat16 layers 1.025 times as fast on the mean, 101 float32 ones 1.004.
    // Nothing is read past the tile: a lane whose window ends there takes the last words and moves them down before it uses them.
    // (1x1: two words, where the moving costs what a load does.)
    const int32_t last_words = P.n_words - 4;
    auto load_bits = [&]() {
#pragma unroll
        for (int ft = 0; ft < NFT; ++ft) {
            const int32_t w = pos[ft] >> 5;
            if constexpr (T == 1) raw[ft] = words_t{tile[w < P.n_words ? w : P.n_words - 1], tile[w + 1 < P.n_words ? w + 1 : P.n_words - 1]};
            else raw[ft] = *reinterpret_cast<const words_a4_t *>(tile + (w < last_words ? w : last_words));
        }
    };

    typename Acc<MT>::type acc[NFT][J];
#pragma unroll
    for (int a = 0; a < NFT; ++a)
#pragma unroll
        for (int b = 0; b < J; ++b)
#pragma unroll
            for (int i = 0; i < NA; ++i) acc[a][b][i] = 0.f;

    // the lane's operand addresses: pixel ln of pixel tile j, channel group q, patch row dy
    constexpr int DY = T == 1 ? 1 : 3;
    const unsigned char *rd[J][DY];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        int px = j * MT + ln;
        px = px < PX ? px : 0;                       // lanes past the block read a valid pixel; their sums are dropped
        const int yo = P.d_cols.div(px), xo = px - yo * P.cols;
#pragma unroll
        for (int dy = 0; dy < DY; ++dy)
            rd[j][dy] = region + q * kGroup + (T == 1 ? yo * P.PC + xo : (yo * P.sh + dy) * P.pitch + xo * P.sw) * 16;
    }
    const int n_tiles = (PX + MT - 1) / MT;          // pixel tiles with pixels (uniform)
    uint32_t sign_mask = 0x80008000u, one_bits = 0x3f803f80u;
    asm volatile("" : "+v"(sign_mask), "+v"(one_bits));

    union Frag { bf16x8_t v; uint32_t u[4]; u32x4_t r; };
    auto multiply = [&](auto j_c, bool more) {   // more: fetch the windows of the wave's next chunk
        constexpr int JL = decltype(j_c)::value;
        uint32_t half[NFT][T == 1 ? 1 : 4];          // words starting at bits 0, 16, 32, 48 of the inverted window
#pragma unroll
        for (int ft = 0; ft < NFT; ++ft) {
            const uint32_t sft = static_cast<uint32_t>(pos[ft] & 31);
            if constexpr (T != 1) {
                const int32_t past = (pos[ft] >> 5) - last_words;
                if (__any(past > 0)) {
                    if (past > 0 && (past & 1)) raw[ft] = words_t{raw[ft][1], raw[ft][2], raw[ft][3], raw[ft][3]};
                    if (past > 0 && (past & 2)) raw[ft] = words_t{raw[ft][2], raw[ft][3], raw[ft][3], raw[ft][3]};
                }
            }
            uint32_t w[T == 1 ? 1 : 3];
#pragma unroll
            for (int i = 0; i < (T == 1 ? 1 : 3); ++i) w[i] = __builtin_amdgcn_alignbit(raw[ft][i + 1], raw[ft][i], sft);
            if (!P.aligned) {                        // a tile end inside the window: it goes on at the tile's first bit
                const int32_t left = p32 - pos[ft];
                if (left < kBits) {
                    const uint32_t h0 = tile[0], h1 = tile[1], h2 = tile[2];
#pragma unroll
                    for (int i = 0; i < (T == 1 ? 1 : 3); ++i) {
                        const int32_t rem = left - 32 * i;
                        if (rem <= 0) {
                            const int32_t s = -rem;
                            const uint32_t lo = s < 32 ? h0 : h1, hi = s < 32 ? h1 : h2;
                            w[i] = __builtin_amdgcn_alignbit(hi, lo, static_cast<uint32_t>(s & 31));
                        } else if (rem < 32) {
                            w[i] = (w[i] & ((1u << rem) - 1u)) | (h0 << rem);
                        }
                    }
                }
            }
            if constexpr (T == 1) {
                half[ft][0] = __builtin_amdgcn_perm(~w[0], ~w[0], 0u);   // the byte, four times
            } else {
                half[ft][0] = ~w[0];
                half[ft][1] = ~__builtin_amdgcn_alignbit(w[1], w[0], 16);
                half[ft][2] = ~w[1];
                half[ft][3] = ~__builtin_amdgcn_alignbit(w[2], w[1], 16);
            }
        }
        if (more) {
#pragma unroll
            for (int ft = 0; ft < NFT; ++ft) {
                pos[ft] += P.step;
                if (pos[ft] >= p32) pos[ft] -= p32;
            }
            load_bits();
        }
        // register e of the filter operand ft of a tap: channels 2e and 2e + 1 of the lane's eight, bits a and b of the window
        auto expand = [&](int tap, int ft, int e) -> uint32_t {
            const int a = T == 1 ? 2 * e : tap + 18 * e, b = T == 1 ? 2 * e + 1 : a + 9;
            const int hs = T == 1 ? 0 : a / 16;
            const int ra = a - 16 * hs, rb2 = b - 16 * hs;
            const u16x2_t src = __builtin_bit_cast(u16x2_t, half[ft][hs]);
            const u16x2_t sel = {src[0], src[rb2 / 16]};
            const u16x2_t sh = {static_cast<uint16_t>(15 - ra), static_cast<uint16_t>(15 - rb2 % 16)};
            return (__builtin_bit_cast(uint32_t, static_cast<u16x2_t>(sel << sh)) & sign_mask) | one_bits;
        };
        // The product is a chain of steps (tap, pixel tile, plane): one operand read, NFT MFMAs.  Reads run kAhead steps ahead
        // (left to itself the compiler reads one step ahead and every MFMA waits for the LDS), the operands of the next tap
        // are expanded in equal parts next to the MFMAs of a tap.
        constexpr int S = JL * NP, kSteps = T * S;
        constexpr int kDepth = NFT == 1 ? (NP == 3 && kCap <= 100 ? 1 : MT == 16 ? 3 : 4) : NFT == 2 ? 4 : NP == 3 ? 1 : 2, kAhead = kSteps - 1 < kDepth ? kSteps - 1 : kDepth;
        auto read = [&](int st) -> u32x4_t {
            const int tap = st / S, j = (st % S) / NP, pl = st % NP;
            return *reinterpret_cast<const u32x4_t *>(rd[j][tap / 3] + (tap % 3) * 16 + pl * kPlane);
        };
        Frag xf[kAhead + 1], wf[2][NFT];
#pragma unroll
        for (int st = 0; st < kAhead; ++st) xf[st].r = read(st);
#pragma unroll
        for (int r = 0; r < 4 * NFT; ++r) wf[0][r / 4].u[r % 4] = expand(0, r / 4, r % 4);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const int tap = st / S, i = st % S, j = i / NP;
            if (st + kAhead < kSteps) xf[(st + kAhead) % (kAhead + 1)].r = read(st + kAhead);
            if (tap + 1 < T) {
#pragma unroll
                for (int r = i * 4 * NFT / S; r < (i + 1) * 4 * NFT / S; ++r) wf[(tap + 1) & 1][r / 4].u[r % 4] = expand(tap + 1, r / 4, r % 4);
            }
#pragma unroll
            for (int ft = 0; ft < NFT; ++ft) acc[ft][j] = Acc<MT>::mma(wf[tap & 1][ft].v, xf[st % (kAhead + 1)].v, acc[ft][j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (PX > 0) {
        std::integral_constant<int, 0> set0;
        std::integral_constant<int, kSets - 1> set1;
        if (ks < P.n_chunks) {
            load_chunk(ks, set0);
            load_bits();
            if (kSets == 2 && ks + KS < P.n_chunks) load_chunk(ks + KS, set1);
        }
        // halo positions stay zero for the whole kernel; valid positions are written again for every chunk
        for (int i = lane * 16; i < kRegion; i += 1024) *reinterpret_cast<u32x4_t *>(region + i) = u32x4_t{0u, 0u, 0u, 0u};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        auto pass = [&](int chunk, auto j_c, auto set_c) {
            store_chunk(chunk, set_c);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (chunk + kSets * KS < P.n_chunks) load_chunk(chunk + kSets * KS, set_c);
            multiply(j_c, chunk + KS < P.n_chunks);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        auto chunk_loop = [&](auto j_c) {
            for (int chunk = ks; chunk < P.n_chunks; chunk += kSets * KS) {
                pass(chunk, j_c, set0);
                if (kSets == 2 && chunk + KS < P.n_chunks) pass(chunk + KS, j_c, set1);
            }
        };
        if constexpr (J == 1) {
            chunk_loop(std::integral_constant<int, 1>{});
        } else {
            if (n_tiles > J / 2) chunk_loop(std::integral_constant<int, J>{});
            else chunk_loop(std::integral_constant<int, J / 2>{});
        }
    }

    // ---- sums of the channel slices, scaling, stores ----------------------------------------------------
    // red[pixel block][slice][filter of the tile][pixel]: a thread adds 16 bytes worth of neighbouring pixels of one filter
    // and writes every replica of them
    constexpr int PG = 16 / static_cast<int>(sizeof(XT));
    float *red = reinterpret_cast<float *>(lds_raw) + ps * (KS * MT * PW);
    const bool per_replica = P.n_alpha == 1 || P.aligned;   // alpha depends on the replica only
    const int reps = static_cast<int>((P.O + P.R - 1) / P.R);
    // one alpha per replica, held in the lanes: a load between the stores would wait for all of them
    float al_lane = per_replica ? alpha[P.n_alpha == 1 ? 0 : (lane < reps ? lane : 0)] : 0.f;
    const bool whole_rows = P.cols == P.Wo;                 // the block's pixels are consecutive in the output plane
    const int tps = (ks << 6) + lane;                       // thread among those of the pixel block
    // barriers that order LDS only: a full one would also wait for the stores of the filter tile before
    auto lds_barrier = [] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    bool small = false;   // an activation of the workgroup has bits below 2^-133
    if constexpr (ALL) {
        uint32_t *flag = reinterpret_cast<uint32_t *>(lds_raw);
        lds_barrier();
        if (lane == 0) flag[wave] = 0u;
        if ((low_bits << 16) != 0u) flag[wave] = 1u;   // (LDS operations of a wave stay in order)
        lds_barrier();
        for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) small = small || flag[w] != 0u;
    }
    for (int ft = 0; ft < NFT; ++ft) {   // (a real loop around everything but the registers: the code is fetched once)
        lds_barrier();
        float *mine = red + ks * (MT * PW);
#pragma unroll
        for (int f = 0; f < NFT; ++f)
            if (f == ft) {
#pragma unroll
                for (int j = 0; j < J; ++j)
#pragma unroll
                    for (int i = 0; i < NA; ++i) mine[Acc<MT>::row(i, q) * PW + j * MT + ln] = acc[f][j][i];
            }
        lds_barrier();
        for (int g = tps; g < MT * PW / PG; g += 64 * KS) {
            const int f = g / (PW / PG), px = (g % (PW / PG)) * PG;
            const int64_t u = u0 + ft * MT + f;
            if (u >= P.R || px >= PX) continue;
            float v[PG];
#pragma unroll
            for (int e = 0; e < PG; ++e) v[e] = red[f * PW + px + e];
            for (int s = 1; s < KS; ++s)
#pragma unroll
                for (int e = 0; e < PG; ++e) v[e] += red[s * (MT * PW) + f * PW + px + e];
            // A NaN may come from an infinity minus its own leading term: such sums are formed again by elements, so that the
            // staging need not look for infinities.  ALL: the bits left out of small activations, likewise.
            if constexpr (NP == 3) {
                bool again = ALL && small;
#pragma unroll
                for (int e = 0; e < PG; ++e) again = again || v[e] != v[e];
                if (__builtin_expect(__any(again), 0)) {
                    int fo = f, po = px;
                    asm volatile("" : "+v"(fo), "+v"(po));   // nothing of this is formed ahead of the loops
#pragma unroll 1
                    for (int e = 0; e < PG; ++e) {
                        float z = v[0];
#pragma unroll
                        for (int i = 1; i < PG; ++i) z = i == e ? v[i] : z;
                        const bool full = z != z;
                        const int oy = P.d_cols.div(po + e), ox = po + e - oy * P.cols;
                        if (po + e >= PX || ox >= cols || !(full || (ALL && small))) continue;
                        const int iy0 = (row0 + oy) * P.sh - P.ph, ix0 = (col0 + ox) * P.sw - P.pw;
                        int64_t bit = (u0 + ft * MT + fo) * P.F % P.p;
                        float sum = 0.f;
                        for (int c = 0; c < P.C; ++c)
                            for (int tap = 0; tap < T; ++tap) {
                                const int iy = iy0 + tap / 3, ix = ix0 + tap % 3;
                                if (iy >= 0 && iy < P.H && ix >= 0 && ix < P.W) {
                                    float a = *reinterpret_cast<const float *>(x_img + c * hwb + (int64_t(iy) * P.W + ix) * 4);
                                    if (!full) {
                                        const float a1 = a - __uint_as_float(__float_as_uint(a) & 0xffff0000u);
                                        const float a2 = a1 - __uint_as_float(__float_as_uint(a1) & 0xffff0000u);
                                        a = fabsf(a) < 1.f ? a2 - __uint_as_float(__float_as_uint(a2) & 0xffff0000u) : 0.f;
                                    }
                                    sum += ((tile[bit >> 5] >> (bit & 31)) & 1u) ? a : -a;
                                }
                                if (++bit == P.p) bit = 0;
                            }
#pragma unroll
                        for (int i = 0; i < PG; ++i)
                            if (i == e) v[i] = full ? sum : v[i] + sum;
                    }
                }
            }
            const int yo = whole_rows ? 0 : P.d_cols.div(px), xo = px - yo * P.cols;
            const bool run = whole_rows ? px + PG <= PX : xo + PG <= cols;   // all of them exist and are consecutive in memory
            XT *dst0 = y + (img * P.O + u) * P.plane_out + int64_t(row0 + yo) * P.Wo + col0 + xo;
            auto write = [&](int t, float al) {
                float w[PG];
                XT r[PG];
#pragma unroll
                for (int e = 0; e < PG; ++e) {
                    w[e] = v[e] * al;
                    if (P.relu) w[e] = fmaxf(w[e], 0.f);
                }
                pack_out(w, r);
                XT *dst = dst0 + t * P.R * P.plane_out;
                if (run) {
                    __builtin_memcpy(dst, r, sizeof(r));
                } else {
#pragma unroll
                    for (int e = 0; e < PG; ++e) {
                        const int y1 = P.d_cols.div(px + e), x1 = px + e - y1 * P.cols;
                        if (px + e < PX && x1 < cols) dst[whole_rows ? int64_t(e) : int64_t(y1 - yo) * P.Wo + (x1 - xo)] = r[e];
                    }
                }
            };
            if (per_replica) {
                for (int t = 0; t < reps && u + t * P.R < P.O; ++t)
                    write(t, P.n_alpha == 1 ? al_lane : t < 64 ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(al_lane), t)) : alpha[t]);
            } else {
                for (int t = 0; t < reps; ++t) {
                    const int64_t o = u + t * P.R;
                    if (o < P.O) write(t, alpha[(o * P.F) / P.p]);
                }
            }
        }
    }
}

constexpr double kLineCost = 6;   // cycles per output line of a wave

struct WavePlan {
    bool ok;
    int mt, pw, nft, cap, rows, cols, n_colblk, n_rowblk, PR, PC, pitch, ks_log2, ps, n_chunks, waves;
    size_t lds;
    int64_t total_waves;
    bool runs;        // staged four pixels at a time
    bool even;        // bfloat16 loads begin at even elements
    bool all_bits;
    bool preferred;   // over tbn_conv_mfma.hip
};

WavePlan plan_wave_for(const ConvArgs &a, int nft) {
    WavePlan pl{};
    const bool one = a.kh == 1 && a.kw == 1, three = a.kh == 3 && a.kw == 3;
    if (!one && !three) return pl;
    const int T = one ? 1 : 9;
    const int64_t F = a.C * T;
    if (a.p < F || a.p < 128 || a.p >= (int64_t(1) << 31) - 4096) return pl;   // one tile end per window; positions in 32 bits
    if (a.W < 2 && !(a.dt == TBN_F32)) return pl;                              // pixels are loaded in pairs
    if (a.Wo <= 0 || a.Ho <= 0 || a.N > 65535 || a.C > (1 << 20)) return pl;
    if (a.H * a.W >= (int64_t(1) << 28) || a.H + 2 * int64_t(a.ph) >= (1 << 24) || a.W + 2 * int64_t(a.pw) >= (1 << 24)) return pl;
    if (a.sh > 64 || a.sw > 64) return pl;
    const int64_t R = unique_rows(a.O, F, a.p);
    const bool f32 = a.dt == TBN_F32;
    const int np = f32 ? 3 : 1;
    pl.nft = nft;
    // Pixel block: rows x cols output pixels of at most pw (64, or 32 where a 64-pixel patch would not fit) whose patch fits
    // the LDS pixels that `it` loads per lane cover.  The cost of a map is its number of blocks times what a wave spends
    // on 32 channels of a block, in cycles: staging per load, operand expansion per filter tile, MFMAs per pixel tile.  (Fitted to loads of
    // single pixels and pairs, as are the limits of `fits`: whether a map allows runs is not known here, and where it does the staging
    // costs less.)
    double best = 0;
    for (int mt : {16, 32}) {
        if (mt == 16 && (f32 || R > 16)) continue;
        const double steps = mt == 16 ? 1.0 : 2.0;   // chunks per 32 channels
        const double c_stage = f32 ? 530 * steps : 480, c_exp = 32.0 * T * pl.nft * steps, c_mma = double(mt) * T * np * pl.nft * steps;
        for (int pw : {64, 32}) {
            for (int big : {0, 1}) {
                const int it = one ? 1 : (f32 ? 2 : 1) + big;
                // instantiated: 1x1 with 64 pixels; 3x3 with 64 pixels on either patch, 32 on the larger one (16
                // filters per MFMA: not the larger one, whose loads do not fit the registers)
                if (one ? (pw == 32 || big) : (pw == 32 && !big)) continue;
                if (big && mt == 16) continue;
                const int cap = (f32 ? (one ? 65 : big ? 192 : 128) : (one ? 129 : big ? 256 : 128)) - 1;
                for (int64_t cols = std::min<int64_t>(a.Wo, pw); cols >= 1; --cols) {
                    const int64_t n_col = (a.Wo + cols - 1) / cols;
                    if (n_col > 1 && cols % (f32 ? 4 : 8) != 0 && cols > 8) continue;   // column blocks: whole 16-byte stores
                    int64_t rows = std::min<int64_t>(a.Ho, pw / cols);
                    const int64_t PC = one ? cols : (cols - 1) * a.sw + 3;
                    const int64_t loads = f32 || (one && a.sw > 1) ? PC : (PC + 1) / 2;   // per patch row
                    auto fits = [&](int64_t r) {
                        const int64_t pr = one ? r : (r - 1) * a.sh + 3;
                        return pr * PC <= cap && pr * loads <= 64 * it;
                    };
                    while (rows >= 1 && !fits(rows)) --rows;
                    if (rows < 1) continue;
                    const int64_t n_row = (a.Ho + rows - 1) / rows;
                    // pixel tiles that the blocks multiply (half of a wave's or all): full blocks, and the shorter last ones
                    auto tiles = [&](int64_t r, int64_t c) {
                        const int64_t j = pw / mt, n = (r * c + mt - 1) / mt;
                        return double(j > 1 && n <= j / 2 ? j / 2 : j);
                    };
                    const int64_t lr = a.Ho - (n_row - 1) * rows, lc = a.Wo - (n_col - 1) * cols;
                    const double nt = tiles(rows, cols) * double((n_row - 1) * (n_col - 1)) + tiles(lr, cols) * double(n_col - 1) +
                                      tiles(rows, lc) * double(n_row - 1) + tiles(lr, lc);
                    const double work = double(n_row * n_col) * (c_stage * it + c_exp) + nt * c_mma;
                    // lines of 128 bytes that the replicas of a block's filters touch
                    const double run = double(cols * (f32 ? 4 : 2)) * (cols == a.Wo ? double(rows) : 1.0);
                    const double lines = (run / 128 + 1) * (cols == a.Wo ? 1.0 : double(rows)) * double(std::min<int64_t>(R, mt * nft) * a.O / R);
                    const double cost = work * double(a.C) / 32 + kLineCost * double(n_row * n_col) * lines;
                    if (!pl.ok || cost < best) {
                        best = cost;
                        pl.ok = true;
                        pl.mt = mt; pl.pw = pw; pl.cap = cap + 1;
                        pl.rows = static_cast<int>(rows); pl.cols = static_cast<int>(cols);
                        pl.n_colblk = static_cast<int>(n_col); pl.n_rowblk = static_cast<int>(n_row);
                        pl.PC = static_cast<int>(PC);
                        pl.PR = static_cast<int>(one ? rows : (rows - 1) * a.sh + 3);
                    }
                }
            }
        }
    }
    if (!pl.ok) return pl;
    pl.ok = false;
    const int CK = 8 * (64 / pl.mt);
    pl.n_chunks = static_cast<int>((a.C + CK - 1) / CK);
    const int64_t fblocks = (R + pl.mt * pl.nft - 1) / (pl.mt * pl.nft);
    const int64_t blocks = int64_t(pl.n_rowblk) * pl.n_colblk;
    if (fblocks > 65535 || blocks > (1 << 24) || blocks * a.N * fblocks > 0x3fffffffLL) return pl;
    // Channel slices, each at least one chunk: until the chip (1024 SIMDs) has about four waves per SIMD, which cover each
    // other's waits.  A float32 patch of more than 100 pixels takes 12 - 18 KiB of LDS per wave: workgroups of eight waves
    // would leave room for one per CU, so eight slices are for grids that would leave SIMDs empty.
    // Runs of four pixels: 3x3, patches of up to 128 pixels whose runs fit, planes that hold one, offsets over 32 channels in 32 bits
    const int row_px = pl.PC + (f32 || a.H * a.W % 2 != 0 ? 0 : 1);
    pl.runs = three && pl.cap == 128 && pl.mt == 32 && pl.PR * ((row_px + 3) / 4) <= kRunLimit && a.H * a.W >= 4 && a.H * a.W < (int64_t(1) << 25);
    pl.even = three && !f32 && a.H * a.W % 2 == 0 && (pl.runs || pl.PR * ((row_px + 1) / 2) <= (pl.cap == 128 ? 64 : 128));
    if (f32 && !one && pl.cap == 128 && pl.PR * pl.PC <= kCapF32 - 1) pl.cap = kCapF32;
    // an odd number of LDS pixels per row where one is free: the runs that 16 lanes store then lie on different banks
    pl.pitch = pl.runs && pl.PC % 4 == 0 && pl.PR * (pl.PC + 1) <= slots_of(pl.cap) - 1 ? pl.PC + 1 : pl.PC;
    int ks_log2 = 0;
    const int64_t units = blocks * a.N * fblocks, want8 = f32 && !one && pl.cap != kCapF32 ? 1024 : 4096;
    while (ks_log2 < 3 && (2 << ks_log2) <= pl.n_chunks && units << ks_log2 < (ks_log2 == 2 ? want8 : 4096)) {
        // 1x1: a chunk is little work next to adding the slices' sums
        if (one && units << ks_log2 >= 1024 && (8 << ks_log2) > pl.n_chunks) break;
        ++ks_log2;
    }
    pl.total_waves = units << ks_log2;
    pl.ks_log2 = ks_log2;
    pl.ps = ks_log2 >= 2 ? 1 : 4 >> ks_log2;
    if (pl.ps > blocks) pl.ps = static_cast<int>(blocks);
    pl.waves = pl.ps << ks_log2;
    const size_t region = size_t(np) * (64 / pl.mt) * slots_of(pl.cap) * 16;
    const size_t red = size_t(pl.waves) * pl.mt * pl.pw * 4;
    pl.lds = std::max(region * pl.waves, red);
    pl.ok = pl.lds <= 160 * 1024;
    return pl;
}

// A 1x1 layer that neither strides nor pads takes the planes as single rows: full pixel blocks whatever the width, and
// blocks that start at multiples of 64 pixels (bfloat16, k = 2, by image rows / as one row / in tbn_conv_mfma.hip: 65 x 256 x
// 55 x 55 -> 64 59.2 / 42.1 / 42.3 us, 14 x 512 x 53 x 53 -> 128 36.0 / 26.9 / 23.7).
ConvArgs as_rows(ConvArgs a) {
    if (a.kh == 1 && a.kw == 1 && a.sh == 1 && a.sw == 1 && a.ph == 0 && a.pw == 0 && a.H * a.W < (1 << 24)) {
        a.W = a.Wo = a.H * a.W;
        a.H = a.Ho = 1;
    }
    return a;
}

// Where tbn_conv_mfma.hip is the faster kernel: small grids whose epilogue is long, since the 64 threads of a channel slice
// write all replicas of their filters where its workgroups have 256 or 512 (float32, 2 x 16 x 93 x 93 -> 512, 1x1, stride 2,
// k = 8: 24.1 us here, 9.6 there).  Below 1024 waves (one per SIMD) both are estimated, in microseconds: here a constant, the
// chunks per slice (16 channels, 32 where a tile has 16 filters), the 16-byte stores per thread and the waves / 1024; there a
// constant, the chunks of 32 channels, the replicas and the pixel blocks / 256.  Least squares over 9169 random layers
// of common sizes, 10 - 15 % off on the average, so the other kernel has to be estimated 9 % faster.  Of 16550 layers (also
// larger ones) 1543 were more than 4 % slower here than there with this kernel always; by this rule 663 are, and 67 are
// slower there than here (margin 3 %: 550 and 207).  (The 3x3 rows of the table are from before one load fetched a window, which took this
// kernel to 0.98 of that time on the mean in bfloat16 and the same in float32, and from before runs and even pairs, 0.96 - 0.97 of it in both.)
bool prefer_wave(const ConvArgs &a, const WavePlan &pl) {
    struct Model { double wave[4], block[4]; };
    static const Model models[2][2] = {   // [bfloat16][3x3]
        {{{3.27, 1.53, 0.23, 1.30}, {3.45, 0.61, 0.36, 2.35}}, {{2.89, 4.08, 0.23, 1.84}, {4.97, 1.35, 0.37, 3.26}}},
        {{{3.82, 1.18, 0.25, 0.87}, {3.46, 0.47, 0.43, 2.08}}, {{2.93, 2.39, 0.27, 1.72}, {5.14, 0.90, 0.41, 2.86}}}};
    if (pl.total_waves >= 1024) return true;
    const Model &m = models[a.dt == TBN_F32 ? 0 : 1][a.kh == 3 ? 1 : 0];
    const double waves = static_cast<double>(pl.total_waves), slices = 1 << pl.ks_log2;
    const int64_t R = unique_rows(a.O, a.C * a.kh * a.kw, a.p);
    const double reps = static_cast<double>(a.O) / static_cast<double>(R);
    const double stores = static_cast<double>(std::min<int64_t>(R, pl.mt * pl.nft)) * reps * pl.pw / (a.dt == TBN_F32 ? 4 : 8) / (64 * slices);
    const double here = m.wave[0] + m.wave[1] * pl.n_chunks / slices + m.wave[2] * stores + m.wave[3] * waves / 1024;
    const double there = m.block[0] + m.block[1] * static_cast<double>((a.C + 31) / 32) + m.block[2] * reps + m.block[3] * waves / slices / 256;
    return 0.91 * here <= there;
}

// Filters per wave: as many tiles of 32 as there are (at most four: the staged input then feeds four times the MFMAs), but
// fewer where the grid would leave SIMDs empty.
WavePlan search_wave(const ConvArgs &layer) {
    const ConvArgs a = as_rows(layer);
    if (a.kh < 1 || a.kh != a.kw || a.p < 1) return WavePlan{};
    const int64_t R = unique_rows(a.O, a.C * a.kh * a.kw, a.p);
    WavePlan pl{};
    // Float32 layers that are too large for tbn_conv_mfma.hip (more channels than its LDS holds filters for, maps wider than
    // its blocks) were float32 FMAs before and keep every bit of their activations; the others never had those below 2^-133.
    const bool other = conv_mfma_supported(layer), all_bits = a.dt == TBN_F32 && !other;
    for (int nft = R <= 32 ? 1 : R <= 64 || (a.dt == TBN_F32 && a.kh == 3) ? 2 : 4; nft >= 1; nft /= 2) {
        pl = plan_wave_for(a, nft);
        pl.all_bits = all_bits;
        pl.preferred = pl.ok && (!other || prefer_wave(a, pl));
        if (pl.ok && (a.kh == 1 ? pl.total_waves >> pl.ks_log2 >= 2048 : pl.total_waves >= 1024)) break;   // (1x1: rather more filter blocks than channel slices)
    }
    return pl;
}

thread_local int64_t n_searches = 0;

// The search takes 1 - 3 us of host time, as long as a small layer: each thread remembers its last shapes (sizes only), four
// to a set, 256 in all: the twenty-odd different layers of a ResNet run in a loop without a search (with 16 shapes, one to
// a set, 19 of the 52 calls of a pass searched again).
WavePlan plan_wave(const ConvArgs &a) {
    struct Entry {
        int64_t key[14];
        WavePlan plan;
        bool used;
    };
    constexpr int kSets = 64, kWays = 4;
    static thread_local Entry cache[kSets][kWays] = {};
    static thread_local uint8_t next[kSets] = {};   // the way that is replaced
    const int64_t key[14] = {a.dt, a.N, a.C, a.H, a.W, a.O, a.kh, a.kw, a.sh, a.sw, a.ph, a.pw, a.p, a.k};
    uint64_t h = 0;
    for (int64_t v : key) h = (h ^ static_cast<uint64_t>(v)) * 0x9e3779b97f4a7c15ull;
    const uint64_t set = h >> 58;
    for (const Entry &e : cache[set])
        if (e.used && std::memcmp(e.key, key, sizeof(key)) == 0) return e.plan;
    Entry &e = cache[set][next[set]];
    next[set] = static_cast<uint8_t>((next[set] + 1) % kWays);
    ++n_searches;
    e.plan = search_wave(a);
    std::memcpy(e.key, key, sizeof(key));
    e.used = true;
    return e.plan;
}

template <typename XT, int MT, int T, int PW, int NFT, int CAP, bool RUNS = false, bool ALL = false>
tbn_status launch_wave_t(const ConvArgs &a, const WaveConvParams &P, const WavePlan &pl, dim3 grid) {
    if constexpr (sizeof(XT) == 4 && !ALL)
        if (pl.all_bits) return launch_wave_t<XT, MT, T, PW, NFT, CAP, RUNS, true>(a, P, pl, grid);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_wave_kernel<XT, MT, T, PW, NFT, CAP, RUNS, ALL>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) {
        set_error("tbn_conv2d_forward: cannot reserve %zu bytes of LDS", pl.lds);
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL((conv_wave_kernel<XT, MT, T, PW, NFT, CAP, RUNS, ALL>), grid, dim3(64 * pl.waves), pl.lds, a.stream,
                       static_cast<const XT *>(a.x), static_cast<XT *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_conv2d_forward (one wave per pixel block)");
}

template <typename XT, int MT, int NFT>
tbn_status launch_wave_shape(const ConvArgs &a, const WaveConvParams &P, const WavePlan &pl, dim3 grid) {
    constexpr bool f32 = sizeof(XT) == 4;
    if (a.kh == 1 || (f32 && NFT == 4)) return launch_wave_t<XT, MT, 1, 64, NFT, f32 ? 65 : 129>(a, P, pl, grid);
    if constexpr (!(f32 && NFT == 4)) {   // (three planes of 128 filters do not fit the registers)
    constexpr int kLarge = f32 ? 192 : 256;
    if constexpr (MT == 32) {
        if (pl.pw == 32) return launch_wave_t<XT, MT, 9, 32, NFT, kLarge>(a, P, pl, grid);
        if (pl.cap == kLarge) return launch_wave_t<XT, MT, 9, 64, NFT, kLarge>(a, P, pl, grid);
    }
    if constexpr (MT == 16) {   // (no runs)
        return launch_wave_t<XT, MT, 9, 64, NFT, 128>(a, P, pl, grid);
    } else {
        if constexpr (f32)
            if (pl.cap == kCapF32)
                return pl.runs ? launch_wave_t<XT, MT, 9, 64, NFT, kCapF32, true>(a, P, pl, grid) : launch_wave_t<XT, MT, 9, 64, NFT, kCapF32>(a, P, pl, grid);
        return pl.runs ? launch_wave_t<XT, MT, 9, 64, NFT, 128, true>(a, P, pl, grid) : launch_wave_t<XT, MT, 9, 64, NFT, 128>(a, P, pl, grid);
    }
    }
}

}  // namespace

bool conv_wave_preferred(const ConvArgs &a) { return plan_wave(a).preferred; }

int64_t conv_wave_searches() { return n_searches; }

void conv_wave_describe(const ConvArgs &a, char *text, size_t size) {
    const WavePlan pl = plan_wave(a);
    const bool pairs = a.dt != TBN_F32 && (a.kh == 3 || a.sw == 1);
    std::snprintf(text, size, "wave filters=%dx%d pixels=%d patch=%d slices=%d waves=%lld block=%dx%d pitch=%d staged=%s%s%s", pl.nft, pl.mt,
                  pl.pw, pl.cap, 1 << pl.ks_log2, static_cast<long long>(pl.total_waves), pl.rows, pl.cols, pl.pitch, pl.even ? "even-" : "",
                  pl.runs ? "runs" : pairs ? "pairs" : "pixels", pl.all_bits ? " all-bits" : "");
}

tbn_status launch_conv_wave(const ConvArgs &layer) {
    const WavePlan pl = plan_wave(layer);
    const ConvArgs a = as_rows(layer);
    if (!pl.ok) {
        set_error("tbn_conv2d_forward: shape not supported by the kernel with one wave per pixel block");
        return TBN_ERR_UNSUPPORTED;
    }
    WaveConvParams P;
    P.HW = a.H * a.W;
    P.plane_out = a.Ho * a.Wo;
    P.O = a.O; P.F = a.C * a.kh * a.kw; P.p = a.p;
    P.R = unique_rows(a.O, P.F, a.p);
    P.C = static_cast<int32_t>(a.C); P.H = static_cast<int32_t>(a.H); P.W = static_cast<int32_t>(a.W);
    P.Ho = static_cast<int32_t>(a.Ho); P.Wo = static_cast<int32_t>(a.Wo);
    P.sh = a.sh; P.sw = a.sw; P.ph = a.ph; P.pw = a.pw;
    P.n_words = static_cast<int32_t>((a.p + 31) / 32);
    P.aligned = a.p % P.F == 0 ? 1 : 0;
    P.n_alpha = a.n_alpha;
    P.relu = (a.flags & TBN_FLAG_RELU) ? 1 : 0;
    P.rows = pl.rows; P.cols = pl.cols; P.n_colblk = pl.n_colblk; P.n_blk = pl.n_rowblk * pl.n_colblk;
    P.PR = pl.PR; P.PC = pl.PC; P.pitch = pl.pitch;
    const int CK = 8 * (64 / pl.mt);
    P.step = static_cast<int32_t>(((int64_t(CK) << pl.ks_log2) * a.kh * a.kw) % a.p);
    P.ks_log2 = pl.ks_log2; P.ps = pl.ps; P.n_chunks = pl.n_chunks;
    const int64_t fblocks = (P.R + pl.mt * pl.nft - 1) / (pl.mt * pl.nft);
    const int64_t gx = (P.n_blk + pl.ps - 1) / pl.ps;
    P.d_img = FastDiv(gx * fblocks);
    P.d_blk = FastDiv(gx);
    P.d_col = FastDiv(pl.n_colblk);
    P.d_cols = FastDiv(pl.cols);
    P.even = pl.even && (reinterpret_cast<uintptr_t>(a.x) & 3u) == 0 ? 1 : 0;
    const int row_px = pl.PC + (pl.even ? 1 : 0);
    P.d_items = FastDiv(pl.runs ? (row_px + 3) / 4 : a.dt == TBN_F32 || (a.kh == 1 && a.sw > 1) ? pl.PC : (row_px + 1) / 2);
    P.d_group = FastDiv(int64_t(P.PR) * P.d_items.d);
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(a.N), static_cast<unsigned>(fblocks));
    tbn_status st;
    if (a.dt == TBN_F32)
        st = pl.nft == 1 ? launch_wave_shape<float, 32, 1>(a, P, pl, grid)
             : pl.nft == 2 ? launch_wave_shape<float, 32, 2>(a, P, pl, grid) : launch_wave_shape<float, 32, 4>(a, P, pl, grid);
    else if (pl.mt == 16)
        st = launch_wave_shape<uint16_t, 16, 1>(a, P, pl, grid);
    else
        st = pl.nft == 1 ? launch_wave_shape<uint16_t, 32, 1>(a, P, pl, grid)
             : pl.nft == 2 ? launch_wave_shape<uint16_t, 32, 2>(a, P, pl, grid) : launch_wave_shape<uint16_t, 32, 4>(a, P, pl, grid);
    if (st != TBN_OK || a.n_alpha == 1 || P.aligned) return st;
    return launch_conv_tile_ends(layer);   // channels whose filter contains a tile start: two alphas
}

}  // namespace tbn
