// Fully-connected tiled-bit layer with a tile of whole weight rows, any row length and alignment: what the other
// matrix-core kernels do not take (in no multiple of 8, activations that are not 16-byte aligned: the 196-token mixing
// layers of an MLP-Mixer, 300- or 2050-wide rows), and the small and middle-sized layers it is faster on.
//
// What is computed (Section "Method", Eq. 4-5 and the scaling after Eq. 8): with p a multiple of `in` the weight is
// the U = p / in rows of the tile stacked k times, copy t scaled by alpha[t]; Z = X * T^T is formed once and
// Y[:, t*U + u] = alpha[t] * Z[:, u].
//
// What bounds it: such layers are small (8192 x 196 -> 384 moves 19 MB), so the time goes into latency: how many waves
// have loads in flight and how few dependent steps lie between the launch and the stores.  The waves of a workgroup share
// 32 batch rows and up to 128 distinct columns and take the 256-byte chunks of K in turn; each stages its chunk
// through 8 KiB of LDS of its own (no barrier in the K loop) into the operand layout of v_mfma_f32_32x32x16_bf16.
//   * Rows start at any element: activations are read 16 bytes per lane at element alignment.  The last chunk of a row
//     reads its last pieces at the row's end instead of past it and shifts them into place, zeros behind: no load
//     leaves its row and no load is conditional.
//   * The +-1 operand: 32 or 64 tile bits per lane, column and chunk at any bit position (two or three words and a
//     funnel shift; the shift never changes), a byte of them through a 256-entry table in LDS.
//   * float32 activations are split into three bfloat16 terms, every product is exact and the sums are float32; what the terms
//     leave out of activations below 2^-110 is added in a second walk, which costs 1 % where there is nothing to add.
//   * The waves leave their sums in LDS as rows of 32 columns; all threads of the workgroup add them in wave order (the
//     result does not depend on timing) and store four (float32) or eight (bfloat16) columns of a row at once.
//
// Microseconds per call (graph replays), before (a batch row and 16 columns per thread on the vector ALUs) / now:
// float32 8192 x 196 -> 384, k = 4: 32.9 / 7.8; 12608 x 197 -> 96, k = 4: 27.6 / 5.7; 8192 x 1199 -> 1024, k = 2:
// 330 / 41; bfloat16 8192 x 2050 -> 1026, k = 2: 490 / 44; 16 x 4095 -> 4096, k = 8: 275 / 13; 8192 x 4096 -> 4096,
// k = 8 with activations at an odd element: 1077 / 72.  Its relative error in float32 against 64-bit sums: 2.5e-7 / 5.6e-8
// at the first of these, 5.6e-8 at in = 1199; the leading terms have one float32 sum per wave, so that it grows with the steps.
#include "tbn_common.h"

#include <type_traits>

namespace tbn {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// 16 bytes at the alignment of an element
template <typename XT> struct Piece;
template <> struct Piece<float> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Piece<uint16_t> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(2))); };

union Frag {
    bf16x8_t v;
    u32x4_t q;
};

constexpr int kChunkBytes = 256;   // bytes of a row per chunk: 64 floats (four MFMA steps) or 128 bfloat16 (eight)
constexpr int kMaxNT = 4;          // column tiles of 32 per workgroup

struct DirectLinearParams {
    int64_t M, out, in;
    int64_t chunks;       // ceil(in / elements per chunk)
    int64_t last_word;    // of the tile
    int32_t U;
    int32_t reps, n_alpha, relu;
    uint32_t groups;      // groups of NT * 32 distinct columns
    uint32_t row_tiles;   // tiles of 32 batch rows
    uint32_t grid_x;      // workgroups per grid row
    int64_t p;            // ENDS: tile bits
    int32_t k;            // ENDS: tile repeats
};

// Row of the weight that contains the start of tile number c, and the start's position in it (0: the tile starts with the
// row).  c * p < 2^53, so that the float64 quotient is off by at most one.
__device__ __forceinline__ int32_t tile_start_row(const DirectLinearParams &P, int32_t c, int32_t &j_e) {
    const int64_t f = int64_t(c) * P.p;
    int64_t q = static_cast<int64_t>(static_cast<double>(f) / static_cast<double>(P.in)), r = f - q * P.in;
    if (r < 0) { r += P.in; --q; }
    if (r >= P.in) { r -= P.in; ++q; }
    j_e = static_cast<int32_t>(r);
    return static_cast<int32_t>(q);
}

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // round to nearest even in hardware
}

// Truncation split of eight floats into three bf16x8 operands (8 + 8 + 8 significand bits: exact).  A NaN stays one in the
// second term, and an infinity, minus itself, puts one there: sums that come out as a NaN are formed again by elements in the
// epilogue.  A bfloat16 has no bits below 2^-133: what an activation has there (the low 16 bits of the third term,
// activations below 2^-110 only) is left out and `lost` set.
__device__ __forceinline__ void split8(const float (&x)[8], Frag (&t)[3], bool &lost) {
    uint32_t h[3][8], low = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t t0 = __float_as_uint(x[i]) & 0xffff0000u;
        const float r1 = x[i] - __uint_as_float(t0);
        const uint32_t t1 = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(t1);
        h[0][i] = t0; h[1][i] = t1; h[2][i] = __float_as_uint(r2);
        low |= h[2][i];
    }
    lost = lost || __any((low << 16) != 0u);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)   // high halves of two words in one: (lo >> 16) | (hi & 0xffff0000)
            t[j].q[v] = __builtin_amdgcn_perm(h[j][2 * v + 1], h[j][2 * v], 0x07060302u);
}

// What split8 leaves out of eight floats, scaled by 2^64: at most 16 bits each, two operands.
__device__ __forceinline__ void rest8(const float (&x)[8], Frag (&t)[2]) {
    uint32_t h[2][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float r1 = x[i] - __uint_as_float(__float_as_uint(x[i]) & 0xffff0000u);
        const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
        float r3 = (r2 - __uint_as_float(__float_as_uint(r2) & 0xffff0000u)) * 0x1p64f;
        r3 = fabsf(x[i]) < 1.f ? r3 : 0.f;   // infinities and NaN are in the terms already
        h[0][i] = __float_as_uint(r3) & 0xffff0000u;
        h[1][i] = __float_as_uint(r3 - __uint_as_float(h[0][i]));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) t[j].q[v] = __builtin_amdgcn_perm(h[j][2 * v + 1], h[j][2 * v], 0x07060302u);
}

// drops the first `bits` bits (a multiple of 16) of a piece and moves the rest down, zeros on top
__device__ __forceinline__ u32x4_t shift_down(u32x4_t v, uint32_t bits) {
    const uint32_t words = bits >> 5, odd = bits & 16u;
    uint32_t w[5] = {v[0], v[1], v[2], v[3], 0u};
    if (words & 1) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = 0u; }
    if (words & 2) { w[0] = w[2]; w[1] = w[3]; w[2] = w[3] = 0u; }
    if (words >= 4) w[0] = w[1] = w[2] = w[3] = 0u;
    u32x4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __funnelshift_r(w[i], w[i + 1], odd);
    return r;
}

template <int NT, int KW>
struct Lds {
    static constexpr int kRegion = NT * 4096 > 8192 ? NT * 4096 : 8192;   // a wave's chunk of X, later its sums
    static constexpr int kBytes = 4096 + KW * kRegion;
};

// ENDS (NT = 1): the columns whose weight row contains a tile start, sixteen per workgroup, each as two rows of the operand:
// row c has the weights before the start (the tile's last bits) and zeros, row 16 + c zeros and the weights from it on (the
// tile's first bits); y = alpha[c - 1] * first + alpha[c] * second.  The pass is a read of X: 8192 x 3000 in bfloat16 19.4 us
// in the small-batch kernel's form (16 rows per workgroup, 64 bytes of a row per load instruction), 14.6 here; 12000 x 264
// 9.2 against 4.7.
// WIDE: rows or tiles whose offsets need 64 bits (2^25 elements in a row, 2^36 tile bits).
template <typename XT, int NT, int KW, bool ENDS = false, bool WIDE = false>
__global__ __launch_bounds__(64 * KW) __attribute__((amdgpu_waves_per_eu(2))) void linear_direct_kernel(const XT *__restrict__ x, XT *__restrict__ y,
                                                               const uint32_t *__restrict__ tile,
                                                               const float *__restrict__ alpha, DirectLinearParams P) {
    typedef Lds<NT, KW> L;
    typedef typename Piece<XT>::type piece_t;
    typedef typename std::conditional<WIDE, int64_t, int32_t>::type idx_t;
    typedef typename std::make_unsigned<idx_t>::type uidx_t;
    const idx_t in = static_cast<idx_t>(P.in), chunks = static_cast<idx_t>(P.chunks);
    const uidx_t last_word = static_cast<uidx_t>(P.last_word);
    constexpr bool kF32 = std::is_same<XT, float>::value;
    constexpr int kCE = kChunkBytes / static_cast<int>(sizeof(XT));   // elements of K per chunk
    constexpr int kEP = 16 / static_cast<int>(sizeof(XT));            // elements per piece
    constexpr int kSteps = kCE / 16;                                  // MFMA steps per chunk
    constexpr int kWords = kCE / 64;                                  // 32-bit windows per lane half, column and chunk
    extern __shared__ __attribute__((aligned(16))) unsigned char s_raw[];
    u32x4_t *s_table = reinterpret_cast<u32x4_t *>(s_raw);
    u32x4_t *s_keep = reinterpret_cast<u32x4_t *>(s_raw + 4096 + KW * L::kRegion);   // ENDS: element masks of a byte
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, lg = lane >> 5;
    unsigned char *region = s_raw + 4096 + wave * L::kRegion;   // this wave's

    // the column groups of a row tile take consecutive slots of one XCD (ids are dealt round-robin to the eight of them):
    // the rows of X they share come from HBM once
    uint32_t rt, cg;
    {
        const uint32_t bid = blockIdx.y * P.grid_x + blockIdx.x, xcd = bid & 7, slot = bid >> 3, full = (P.row_tiles / 8) * P.groups;
        if (bid >= P.row_tiles * P.groups) return;   // the last grid row
        if (slot < full) {
            const uint32_t q = slot / P.groups;
            cg = slot - q * P.groups;
            rt = q * 8 + xcd;
        } else {   // the remaining row tiles: plain order
            const uint32_t rest = bid - full * 8, q = rest / P.groups;
            cg = rest - q * P.groups;
            rt = (P.row_tiles / 8) * 8 + q;
        }
    }
    const int64_t m0 = int64_t(rt) * 32;
    const int32_t u0 = static_cast<int32_t>(cg) * (NT * 32);

    // loads: piece (i, h) of a chunk is row 8i + lane/8, bytes 128h + 16*(lane%8) .. + 15: eight lanes read 128 bytes in
    // a row.  Rows past M repeat the last one; they are never written.
    const unsigned char *x_blk = reinterpret_cast<const unsigned char *>(x + m0 * P.in);
    const int rows_last = static_cast<int>(P.M - 1 - m0 < 31 ? P.M - 1 - m0 : 31);
    uidx_t ld_off[4];        // bytes from x_blk
    // byte positions in the wave's region: 256 bytes per row, piece p of row r at place p ^ (r % 16); piece (i, h) is at
    // 2048 i + st_pos[(i + h) % 2]
    uint32_t st_pos[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + (lane >> 3);
        ld_off[i] = static_cast<uidx_t>(r < rows_last ? r : rows_last) * static_cast<uidx_t>(in) * static_cast<uidx_t>(sizeof(XT));
    }
    st_pos[0] = static_cast<uint32_t>((lane >> 3) * 256 + (((lane & 7) ^ (lane >> 3)) << 4));
    st_pos[1] = st_pos[0] ^ 128u;
    const int e_lane = (lane & 7) * kEP;   // first element of piece h in a chunk: e_lane + h * kCE / 2

    u32x4_t xr[8];   // the chunk in flight: [i][h]
    auto load_chunk = [&](idx_t c) {
        if ((c + 1) * kCE <= in) {
            const unsigned char *src = x_blk + int64_t(c) * kChunkBytes;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    xr[2 * i + h] = *reinterpret_cast<const piece_t *>(src + (ld_off[i] + 16 * (lane & 7)) + h * (kChunkBytes / 2));
        } else if (in >= kEP) {   // the last chunk: pieces that would leave the row are read at its end
            const idx_t lim = in - kEP;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const idx_t e = c * kCE + e_lane + h * (kCE / 2);
                const uidx_t off = static_cast<uidx_t>(e < lim ? e : lim) * static_cast<uidx_t>(sizeof(XT));
#pragma unroll
                for (int i = 0; i < 4; ++i) xr[2 * i + h] = *reinterpret_cast<const piece_t *>(x_blk + (ld_off[i] + off));
            }
        } else {   // rows shorter than a piece
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uidx_t off = ld_off[i];
                asm volatile("" : "+v"(off));   // the address is formed here, not kept in registers through the loops
                const XT *row = reinterpret_cast<const XT *>(x_blk + off);
                u32x4_t v = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < kEP - 1; ++j) {
                    if (j >= in) break;
                    if constexpr (kF32) v[j] = __float_as_uint(row[j]);
                    else v[j / 2] |= uint32_t(row[j]) << (16 * (j & 1));
                }
                xr[2 * i] = (lane & 7) == 0 ? v : u32x4_t{0u, 0u, 0u, 0u};
                xr[2 * i + 1] = u32x4_t{0u, 0u, 0u, 0u};
            }
        }
    };

    // tile words of this lane's column in every column tile: bit u * in + k, lane half lg covers kWords windows per chunk
    uidx_t word0[NT];
    uint32_t sh[NT];
    int32_t split = 0;   // ENDS: first element of the row that belongs to the tile that starts in it
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if constexpr (ENDS) {   // bit of element 0 (before the tile's start, where it is masked, for the second row)
            const int32_t tc = static_cast<int32_t>(cg) * 16 + (ln & 15) + 1;
            tile_start_row(P, tc < P.k ? tc : 1, split);
            const int64_t bit = (ln < 16 ? P.p - split : int64_t(-split)) + lg * (kCE / 2);
            word0[t] = static_cast<uidx_t>(bit >> 5);   // may be "negative": see load_words
            sh[t] = static_cast<uint32_t>(bit & 31);
        } else {
            const int32_t u = u0 + 32 * t + ln < P.U ? u0 + 32 * t + ln : P.U - 1;   // columns past U repeat the last one; never written
            const uint64_t bit = uint64_t(u) * static_cast<uint64_t>(in) + static_cast<uint32_t>(lg * (kCE / 2));
            word0[t] = static_cast<uidx_t>(bit >> 5);
            sh[t] = static_cast<uint32_t>(bit & 31);
        }
    }
    uint32_t wr[NT][kWords + 1];
    // words past the tile's end belong to positions past the row's end (ENDS: past the first part), words before its start
    // (as unsigned numbers past it as well) to positions before the second part: any value will do
    auto load_words = [&](idx_t c) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int w = 0; w <= kWords; ++w) {
                const uidx_t i = word0[t] + static_cast<uidx_t>(c * (kCE / 32) + w);
                wr[t][w] = tile[i < last_word ? i : last_word];
            }
    };

    if (wave < chunks) {
        load_chunk(wave);
        load_words(wave);
    }
    // sign table: entry e, element i is +1 if bit i of e is set, else -1
    for (int e = tid; e < 256; e += 64 * KW) {
        u32x4_t t;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            t[v] = (((e >> (2 * v)) & 1) ? 0x3f80u : 0xbf80u) | ((((e >> (2 * v + 1)) & 1) ? 0x3f80u : 0xbf80u) << 16);
        s_table[e] = t;
        if constexpr (ENDS) {
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = (((e >> (2 * v)) & 1) ? 0xffffu : 0u) | (((e >> (2 * v + 1)) & 1) ? 0xffff0000u : 0u);
            s_keep[e] = t;
        }
    }
    __syncthreads();

    // float32: the two small terms of the split have sums of their own, so that they are not rounded to the large sum's
    // last place at every step (relative error at in = 1199: 5.6e-8, against 2.3e-7 with one sum)
    f32x16_t acc[NT], low[kF32 ? NT : 1];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            acc[t][e] = 0.f;
            if constexpr (kF32) low[t][e] = 0.f;
        }

    // the chunk in flight into the region; returns its MFMA steps
    auto stage = [&](idx_t c) __attribute__((always_inline)) {
        int steps = kSteps;
        if ((c + 1) * kCE > in) {   // the last chunk of a row that does not fill it
            const int tail = static_cast<int>(in - c * kCE);
            if (tail < kCE / 2) steps = (tail + 7) / 8;   // step s takes elements 8s .. + 7 of both halves of the chunk
            if (in >= kEP) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int past = e_lane + h * (kCE / 2) - (tail - kEP);   // elements that the load was moved back by
                    const uint32_t bits = past > 0 ? static_cast<uint32_t>(past) * (8u * sizeof(XT)) : 0u;
#pragma unroll
                    for (int i = 0; i < 4; ++i) xr[2 * i + h] = shift_down(xr[2 * i + h], bits);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<u32x4_t *>(region + st_pos[(i + h) & 1] + 2048 * i) = xr[2 * i + h];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();   // lanes read what other lanes of the wave wrote (LDS operations of a wave stay in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        return steps;
    };
    auto release = [] {   // the next chunk overwrites the region
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the +-1 operand from a byte of tile bits whose first element is e of the chunk
    auto operand = [&](uint32_t byte, idx_t c, int e) __attribute__((always_inline)) {
        Frag sg;
        sg.q = s_table[byte & 0xffu];
        if constexpr (ENDS) {
            int32_t n = split - static_cast<int32_t>(c * kCE + lg * (kCE / 2) + e);   // of the eight elements, those before the start
            n = n < 0 ? 0 : n > 8 ? 8 : n;
            const uint32_t before = (1u << n) - 1u;
            sg.q &= s_keep[ln < 16 ? before : 0xffu ^ before];
        }
        return sg;
    };
    bool lost = false;
    for (idx_t c = wave; c < chunks; c += KW) {
        uint32_t wc[NT][kWords];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int w = 0; w < kWords; ++w) wc[t][w] = __funnelshift_r(wr[t][w], wr[t][w + 1], sh[t]);
        const int steps = stage(c);
        if (c + KW < chunks) {
            load_chunk(c + KW);
            load_words(c + KW);
        }
        // operands of row ln.  float32: step s of lane half lg takes floats 32*lg + 8*s .. + 7, pieces 8*lg + 2*s and + 1;
        // bfloat16: elements 64*lg + 8*s .. + 7, piece 8*lg + s
        auto sign = [&](int t, int s) { return operand(wc[t][s / 4] >> (8 * (s % 4)), c, 8 * s).v; };
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            if (s >= steps) break;
            if constexpr (kF32) {
                const f32x4_t a = *reinterpret_cast<const f32x4_t *>(region + ln * 256 + (((8 * lg + 2 * s) ^ (ln & 15)) << 4));
                const f32x4_t b = *reinterpret_cast<const f32x4_t *>(region + ln * 256 + (((8 * lg + 2 * s + 1) ^ (ln & 15)) << 4));
                const float xs[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
                Frag terms[3];
                split8(xs, terms, lost);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const bf16x8_t sg = sign(t, s);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg, terms[0].v, acc[t], 0, 0, 0);
                    low[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg, terms[2].v, low[t], 0, 0, 0);
                    low[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg, terms[1].v, low[t], 0, 0, 0);
                }
            } else {
                Frag xt;
                xt.q = *reinterpret_cast<const u32x4_t *>(region + ln * 256 + (((8 * lg + s) ^ (ln & 15)) << 4));
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sign(t, s), xt.v, acc[t], 0, 0, 0);
            }
        }
        release();
    }

    if constexpr (kF32) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] += low[t];
        // activations with bits below 2^-133: the wave goes through its chunks again, one column tile at a time, and adds
        // those bits, scaled by 2^64, times signs scaled by 2^-64
        if (__builtin_expect(lost, 0)) {
#pragma unroll 1
            for (int tt = 0; tt < NT; ++tt) {
                uidx_t first = word0[0];
                uint32_t shift = sh[0];
#pragma unroll
                for (int t = 1; t < NT; ++t)
                    if (tt == t) { first = word0[t]; shift = sh[t]; }
                f32x16_t sum;
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[e] = 0.f;
#pragma unroll 1
                for (idx_t c = wave; c < chunks; c += KW) {
                    load_chunk(c);
                    uint32_t w[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uidx_t i = first + static_cast<uidx_t>(c * (kCE / 32) + j);
                        w[j] = tile[i < last_word ? i : last_word];
                    }
                    const uint32_t window = __funnelshift_r(w[0], w[1], shift);
                    const int steps = stage(c);
#pragma unroll 1
                    for (int s = 0; s < steps; ++s) {
                        const f32x4_t a = *reinterpret_cast<const f32x4_t *>(region + ln * 256 + (((8 * lg + 2 * s) ^ (ln & 15)) << 4));
                        const f32x4_t b = *reinterpret_cast<const f32x4_t *>(region + ln * 256 + (((8 * lg + 2 * s + 1) ^ (ln & 15)) << 4));
                        const float xs[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
                        Frag rest[2];
                        rest8(xs, rest);
                        Frag sg = operand(window >> (8 * s), c, 8 * s);
                        sg.q &= 0xdfffdfffu;   // 1 -> 2^-64
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg.v, rest[1].v, sum, 0, 0, 0);
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg.v, rest[0].v, sum, 0, 0, 0);
                    }
                    release();
                }
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (tt == t) acc[t] += sum;
            }
        }
    }
    // The wave's sums, 32 rows of 32 columns per tile: register 4q + e is column 8q + 4lg + e of row ln; the four columns of
    // group g of row r sit at group g ^ (r & 7).
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4_t *>(region + t * 4096 + ln * 128 + (((2 * q + lg) ^ (ln & 7)) << 4)) =
                f32x4_t{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
    __syncthreads();

    if constexpr (ENDS) {   // 32 rows x 16 columns, neighbouring threads neighbouring columns
        for (int unit = tid; unit < 512; unit += 64 * KW) {
            const int r = unit >> 4, c = unit & 15;
            const int32_t tc = static_cast<int32_t>(cg) * 16 + c + 1;
            if (m0 + r >= P.M || tc >= P.k) continue;
            int32_t j_e;
            const int32_t o = tile_start_row(P, tc, j_e);
            if (j_e == 0) continue;   // the tile starts with the row: nothing to repair
            float z[2] = {0.f, 0.f};
#pragma unroll
            for (int w = 0; w < KW; ++w)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int col = 16 * h + c;
                    z[h] += *reinterpret_cast<const float *>(s_raw + 4096 + w * L::kRegion + r * 128 + (((col >> 2) ^ (r & 7)) << 4) + 4 * (col & 3));
                }
            if (__builtin_expect(z[0] != z[0] || z[1] != z[1], 0)) {   // 0 x infinity in a masked operand, or a NaN: by elements
                const XT *row = x + (m0 + r) * P.in;
                z[0] = z[1] = 0.f;
                for (int32_t j = 0; j < in; ++j) {
                    const int64_t bit = (j < j_e ? P.p : 0) + j - j_e;
                    const float e = ElemIO<XT>::load(row + j), w = ((tile[bit >> 5] >> (bit & 31)) & 1u) ? e : -e;
                    if (j < j_e) z[0] += w; else z[1] += w;
                }
            }
            float v = alpha[tc - 1] * z[0] + alpha[tc] * z[1];
            if (P.relu) v = fmaxf(v, 0.f);
            ElemIO<XT>::store(y + (m0 + r) * P.out + o, v);
        }
        return;
    }
    // y[m, u + t*U] = alpha[t] * Z[m, u]: a thread adds and writes kEP adjacent columns of a row, neighbouring threads
    // neighbouring columns.  bfloat16 leaves threads without such columns (384 of 512 with one column tile): they share the
    // replicas and each adds the sums anew (one column tile and eight waves, 2 / 4 / 8 / 16 replicas: 1.00 / 1.03 / 1.10 / 1.21
    // times faster, columns in no multiple of 8 1.03 / 1.12 / 1.28 / 1.47 times; 17 x 80 -> 2157, k = 16: 9.4 / 5.6 us).  In
    // float32, where half the threads have columns, one replica lost 2 % by it and 16 gained 5 %: left alone.
    constexpr int kGroupsPerRow = NT * 32 / kEP, kUnits = 32 * kGroupsPerRow;
    constexpr int kShare = !kF32 && 64 * KW > kUnits ? 64 * KW / kUnits : 1;
    static_assert(kUnits % 64 == 0, "a wave has one part");
    const int share = kShare > 1 && P.reps >= 2 ? kShare : 1;
    for (int i = tid; i < kUnits * share; i += 64 * KW) {
        // (the same for a whole wave: alpha comes by scalar loads, a vector load would wait for the stores before it)
        const int part = kShare > 1 ? __builtin_amdgcn_readfirstlane(i / kUnits) : 0, unit = i - part * kUnits;
        const int r = unit / kGroupsPerRow, g = unit - r * kGroupsPerRow;
        const int64_t m = m0 + r;
        const int32_t u = u0 + g * kEP;
        if (m >= P.M || u >= P.U) continue;
        const int t = g * kEP / 32, g4 = (g * kEP % 32) / 4;
        f32x4_t z[kEP / 4];
#pragma unroll
        for (int w = 0; w < KW; ++w)
#pragma unroll
            for (int j = 0; j < kEP / 4; ++j) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t *>(s_raw + 4096 + w * L::kRegion + t * 4096 + r * 128 + (((g4 + j) ^ (r & 7)) << 4));
                z[j] = w == 0 ? v : z[j] + v;
            }
        if constexpr (kF32) {   // a NaN in a sum may come from an infinity, minus itself in the split: by elements
            bool again = false;
#pragma unroll
            for (int e = 0; e < kEP; ++e) again = again || (u + e < P.U && z[e / 4][e % 4] != z[e / 4][e % 4]);
            if (__builtin_expect(__any(again), 0)) {
                int32_t col = u;
                asm volatile("" : "+v"(col));   // nothing of this is formed ahead
#pragma unroll 1
                for (int e = 0; e < kEP; ++e) {
                    float s = z[0][0];
#pragma unroll
                    for (int i = 1; i < kEP; ++i) s = i == e ? z[i / 4][i % 4] : s;
                    if (col + e >= P.U || s == s) continue;
                    const XT *row = x + m * P.in;
                    const int64_t first = int64_t(col + e) * in;
                    s = 0.f;
                    for (idx_t j = 0; j < in; ++j) {
                        const int64_t bit = first + j;
                        s += ((tile[bit >> 5] >> (bit & 31)) & 1u) ? static_cast<float>(row[j]) : -static_cast<float>(row[j]);
                    }
#pragma unroll
                    for (int i = 0; i < kEP; ++i)
                        if (i == e) z[i / 4][i % 4] = s;
                }
            }
        }
        XT *dst = y + m * P.out + u + part * P.U;
        const bool whole = u + kEP <= P.U;
        for (int32_t rep = part; rep < P.reps; rep += share, dst += share * P.U) {
            const float al = alpha[P.n_alpha == 1 ? 0 : rep];
            float v[kEP];
#pragma unroll
            for (int e = 0; e < kEP; ++e) {
                v[e] = al * z[e / 4][e % 4];
                if (P.relu) v[e] = fmaxf(v[e], 0.f);
            }
            if (whole) {
                u32x4_t pk;
                if constexpr (kF32) pk = u32x4_t{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
                else pk = u32x4_t{pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4 % kEP], v[5 % kEP]), pack2(v[6 % kEP], v[7 % kEP])};
                *reinterpret_cast<piece_t *>(dst) = pk;
            } else {
#pragma unroll
                for (int e = 0; e < kEP; ++e)
                    if (u + e < P.U) ElemIO<XT>::store(dst + e, v[e]);
            }
        }
    }
}

// A launch has fewer than 2^32 threads along x (beyond that the count wraps and the workgroups behind it never run): the
// workgroups are dealt to rows of 2^22.
constexpr uint32_t kGridX = 1u << 22;
static_assert(uint64_t(kGridX) * 512 < (uint64_t(1) << 32), "threads per grid row");
dim3 grid_of(DirectLinearParams &P) {
    const uint32_t n = P.row_tiles * P.groups;   // < 2^31
    P.grid_x = n < kGridX ? n : kGridX;
    return dim3(P.grid_x, (n + P.grid_x - 1) / P.grid_x);
}

template <typename XT, int NT, int KW, bool WIDE = false>
tbn_status launch_one(const LinearArgs &a, DirectLinearParams P) {
    typedef Lds<NT, KW> L;
    // dynamic LDS above the default limit has to be allowed once per kernel (thread-safe static initialisation)
    static const hipError_t attr = L::kBytes > 65536
        ? hipFuncSetAttribute(reinterpret_cast<const void *>(&linear_direct_kernel<XT, NT, KW, false, WIDE>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, L::kBytes)
        : hipSuccess;
    if (attr != hipSuccess) {
        set_error("tbn_linear_forward: cannot reserve %d bytes of LDS", L::kBytes);
        return TBN_ERR_DEVICE;
    }
    const dim3 grid = grid_of(P);
    hipLaunchKernelGGL((linear_direct_kernel<XT, NT, KW, false, WIDE>), grid, dim3(64 * KW), L::kBytes, a.stream,
                       static_cast<const XT *>(a.x), static_cast<XT *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward (direct kernel)");
}

// What `plan` gives: float32 four or eight waves, of eight at most 384 workgroups (two column tiles come only with more than 512 row tiles); bfloat16
// eight waves with one column tile, four with up to two, since more tiles come with more than 1024 workgroups.
constexpr bool planned(bool f32, int NT, int KW) {
    return f32 ? KW == 4 || (KW == 8 && NT != 2) : KW <= 2 || (KW == 4 && NT <= 2) || (KW == 8 && NT == 1);
}

template <typename XT, int NT, int KW = 8>
tbn_status launch_kw(const LinearArgs &a, const DirectLinearParams &P, int kw) {
    if constexpr (planned(std::is_same<XT, float>::value, NT, KW))
        if (kw == KW) return launch_one<XT, NT, KW>(a, P);
    if constexpr (KW > 1) return launch_kw<XT, NT, KW / 2>(a, P, kw);
    set_error("tbn_linear_forward: the direct kernel has no instance of %d column tiles and %d waves", NT, kw);
    return TBN_ERR_UNSUPPORTED;
}

template <typename XT>
tbn_status launch_nt(const LinearArgs &a, const DirectLinearParams &P, int nt, int kw) {
    switch (nt) {
        case 4: return launch_kw<XT, 4>(a, P, kw);
        case 3: return launch_kw<XT, 3>(a, P, kw);
        case 2: return launch_kw<XT, 2>(a, P, kw);
    }
    return launch_kw<XT, 1>(a, P, kw);
}

struct DirectPlan {
    int nt, kw;
    bool wide;
    int64_t groups, row_tiles, chunks;
};

// W = 32 x 32 tiles of Z.  Up to 1024 of them a workgroup takes one and as many waves as bring the chip to 3072 in bfloat16 (12 per
// CU; 8192 x 196 -> 96: 8.0 us with four waves, 9.0 with two, 10.9 with eight), to 2048 in float32, see below.  Beyond that float32 takes four column
// tiles and at least four waves: more columns share the split of an activation (2500 x 520 -> 1400: 23.5 us against 27.7
// with two tiles; 6000 x 2504 -> 640: 65.8 against 80.1).  bfloat16 takes two (12000 x 520 -> 152: 10.8 us against 13.4
// with four), and above 4096 as many as leave the fewest empty ones (8192 x 2050 -> 513: 41.9 us with three, 45.3 with
// four).
// float32 takes eight waves only while every workgroup has a CU to itself: their registers (134 a lane with one tile) or their LDS
// (132 KB with four) leave room for one of them per CU, so that of 257 - 384 the second round finds most CUs without one; of four waves three
// (two with four tiles) run at once.  One tile: 120 drawn layers 1.19 times as fast on the mean, 1.04 at the least (3556 x 382 -> 90 7.5 us with
// eight, 6.4 with four).  Four tiles: with up to 12 chunks of K, where load and sums are most of the time, one tile per workgroup instead
// (2319 x 368 -> 465 12.7 us with eight waves of four tiles, 10.4 now; 2340 x 579 -> 477 17.0 / 14.3); longer rows 1.06 on the mean over
// 70 against four waves of two tiles, which beat eight waves of four by 1.02 - 1.18.
// The error against 64-bit sums decides where that ends.  Four waves add fewer partial sums at the end, but twice as many steps go into each sum:
// measured over six sizes of 257 - 384 workgroups, four waves' error over eight waves' is 0.81 at 2051 elements, 0.85 at 4099, 0.92 at 8196, 0.97 at
// 12000, 0.99 at 14001, 1.01 at 16001, 1.04 at 20001, 1.12 at 32001 and 1.29 at 65540.  So rows of more than 216 chunks (13824 elements) keep eight waves.
constexpr int64_t kFewWavesChunks = 216;

DirectPlan plan(const LinearArgs &a) {
    DirectPlan pl;
    const bool f32 = a.dt == TBN_F32;
    const int64_t tiles = (a.p / a.in + 31) / 32;
    const int64_t ce = f32 ? kChunkBytes / 4 : kChunkBytes / 2;
    pl.row_tiles = (a.M + 31) / 32;
    pl.chunks = (a.in + ce - 1) / ce;
    const int64_t W = pl.row_tiles * tiles;
    // offsets inside 32 rows and tile words in 64 bits: one column tile and eight waves, the others share what their waves load
    pl.wide = a.in >= (int64_t(1) << 25) || a.p >= (int64_t(1) << 36);
    const int64_t fours = pl.row_tiles * ((tiles + kMaxNT - 1) / kMaxNT);
    int nt = kMaxNT;
    if (W <= 1024 || pl.wide) nt = 1;
    else if (f32 && fours <= 384 && pl.chunks <= 12) nt = 1;
    else if (!f32 && W <= 4096) nt = 2;
    else if (!f32)
        for (int cand = kMaxNT - 1; cand >= 2; --cand)
            if ((tiles + cand - 1) / cand * cand < (tiles + nt - 1) / nt * nt) nt = cand;
    pl.groups = (tiles + nt - 1) / nt;
    pl.nt = static_cast<int>((tiles + pl.groups - 1) / pl.groups);
    pl.kw = 8;
    const int64_t waves = f32 && pl.chunks <= kFewWavesChunks ? 2048 : 3072;
    while (!pl.wide && pl.kw > (f32 ? 4 : 1) && pl.row_tiles * pl.groups * pl.kw > waves) pl.kw /= 2;
    return pl;
}

}  // namespace

// Shapes this kernel takes: tile of whole rows; it is meant for what the matrix-core kernels decline.
bool linear_direct_supported(const LinearArgs &a) {
    if (a.dt != TBN_F32 && a.dt != TBN_BF16) return false;
    if (a.M < 1 || a.in < 1 || a.p % a.in != 0) return false;
    const int64_t U = a.p / a.in;
    if (U < 1 || U > a.out || a.out % U != 0 || a.out / U > (1 << 30)) return false;
    if (U > (1 << 30)) return false;   // columns are kept in 32 bits
    if (a.n_alpha != 1 && a.n_alpha != a.out / U) return false;
    const DirectPlan pl = plan(a);
    return pl.row_tiles <= 0x7fffffffLL && pl.row_tiles * pl.groups <= 0x7fffffffLL;
}

// Where this kernel beats the one that would otherwise take a call with rows in multiples of 8 and 16-byte aligned
// activations.  Graph replays, microseconds per call, the other kernel / this one; W is the number of 32 x 32 tiles of Z.
bool linear_direct_preferred(const LinearArgs &a, DirectOver other) {
    if ((a.flags & ~uint32_t(TBN_FLAG_RELU)) || !linear_direct_supported(a)) return false;   // flags that steer to another kernel
    if (plan(a).wide) return false;
    const bool f32 = a.dt == TBN_F32;
    const int64_t U = a.p / a.in, W = ((a.M + 31) / 32) * ((U + 31) / 32);
    if (other == DirectOver::Tile) {
        // the tile kernel splits K among waves in whole slices: rows that do not divide leave it one wave per tile (bfloat16
        // 1297 x 3840 -> 64: 23.0 / 8.8; 500 x 512 -> 256: 6.1 / 4.6; 9926 x 512 -> 32: 7.5 / 7.9; float32 817 x 640 -> 476:
        // 15.5 / 8.4); float32 and few tiles, where it takes four column tiles per wave (200 x 4096 -> 512: 23.5 / 15.5;
        // 600 x 4096 -> 512: 25.1 / 29.4), unless there is only one (2867 x 3072 -> 32: 10.6 / 12.4; 3867 x 5632 -> 24: 17.7 /
        // 21.2)
        const bool one_slice = linear_tile_k_slices(a) == 1;
        if (f32 && W <= 256 && (U > 32 || one_slice)) return true;
        return one_slice && W <= 1024 && a.in > kChunkBytes / (f32 ? 4 : 2) && (f32 || a.M <= 4096);
    }
    if (other == DirectOver::SmallBatch) {
        // more than one workgroup of the small-batch kernel per CU (700 drawn calls, that kernel / this one: 257 - 512 of
        // them bfloat16 1.18 - 1.72, float32 0.96 - 1.43, more 1.28 - 2.46)
        if (W <= 1024 && ((U + 15) / 16) * ((a.M + 15) / 16) > 256) return true;
        // Below that, rows of whole lines: float32, whose sums here keep infinities and the bits below 2^-133 and have accumulators of
        // their own for the small terms (that kernel does neither, so that its speed, 0.74 - 0.92 of the time, does not count); bfloat16 with many
        // replicas, which that kernel stores two bytes at a time (102 drawn layers of 17 - 600 rows, the time here over the time there: to 1280
        // elements 1.13 with up to eight replicas, 1.06 with 16, 0.96 with 32; longer rows 1.02, 0.96 and 0.90), and bfloat16 of up to 16 rows
        // (calls that the decode kernel leaves, more than 16384 outputs of Z: 1.1 there too, but the tests' table of kernels has such calls here).
        if ((!f32 && a.M > 16 && a.out / U <= (a.in <= 1280 ? 16 : 8)) || U % 8 != 0 || a.in < 384) return false;
        return f32 ? a.in % 64 == 0 && a.in <= 1280 : a.in % 128 == 0 && (a.in <= 3584 || a.in >= 4608);
    }
    // short rows in few blocks of the block or the streaming kernel (bfloat16 8961 x 256 -> 96: 8.1 / 5.7; 1289 x 256 -> 848:
    // 6.4 / 5.3; 1810 x 512 -> 528: 8.8 / 5.7; 6395 x 512 -> 168: 9.2 / 6.7; with activations at an odd element, 1226 x 256 ->
    // 1248 (W = 1521): 8.7 / 9.0; 2736 x 768 -> 376: 8.9 / 10.9)
    if (other == DirectOver::Block) return a.in <= 512 && W <= 1200;
    // the general kernel's 128 x 128 blocks: few of them (bfloat16 200 x 520 -> 640: 11.1 / 4.6; 12000 x 520 -> 152: 13.0 /
    // 10.6; 2500 x 2504 -> 640: 20.0 / 20.2; 2500 x 1000 -> 1400: 15.9 / 19.4; float32 300 x 200 -> 250: 21.6 / 4.4; 6000 x
    // 2504 -> 640: 75 / 66; 12000 x 520 -> 640: 51 / 50), and columns that it stores one by one (bfloat16 8364 x 376 -> 1076:
    // 54 / 24; 5338 x 1024 -> 2564: 74 / 60).  In bfloat16 long rows outweigh that where its blocks fill the CUs (4040 x 7344 ->
    // 948: 64 / 108): times in microseconds by least squares over 471 shapes with more than 2e6 tile rows W * in; of 36 shapes
    // that were more than 4 % slower here 8 are left, and 2 of 4218 went the other way.
    if (U % 8 != 0) {
        const double rows = 1e-6 * static_cast<double>(W) * static_cast<double>(a.in);
        if (f32 || rows <= 2) return W <= 16384;
        const int64_t rounds = (((a.M + 127) / 128) * ((U + 127) / 128) + 255) / 256;
        const double outputs = 1e-6 * static_cast<double>(a.M) * static_cast<double>(a.out);
        return W <= 16384 && 8.7 + 3.18 * rows + 0.41 * outputs <= 6.9 + 7.1e-3 * static_cast<double>(rounds) * static_cast<double>(a.in) + 1.93 * outputs;
    }
    if (f32) return W <= 4096;
    return W <= 1024 || (W <= 2048 && a.in <= 2048);
}

template <typename XT>
static tbn_status launch_ends(const LinearArgs &a, DirectLinearParams P) {
    constexpr int kLds = Lds<1, 8>::kBytes + 4096;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&linear_direct_kernel<XT, 1, 8, true>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (attr != hipSuccess) {
        set_error("tbn_linear_forward: cannot reserve %d bytes of LDS", kLds);
        return TBN_ERR_DEVICE;
    }
    const dim3 grid = grid_of(P);
    hipLaunchKernelGGL((linear_direct_kernel<XT, 1, 8, true>), grid, dim3(512), kLds, a.stream,
                       static_cast<const XT *>(a.x), static_cast<XT *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward (columns that hold a tile start)");
}

bool linear_direct_ends_supported(const LinearArgs &a) {
    if (a.dt != TBN_F32 && a.dt != TBN_BF16) return false;
    // at most one tile start per row; word numbers before the tile's start, as unsigned numbers, lie past its end
    if (a.M < 1 || a.p < a.in || a.in > (1 << 21) || a.p >= (int64_t(1) << 31) || a.n_alpha != a.k || a.out > (1 << 30)) return false;
    return (a.M + 31) / 32 * ((int64_t(a.k) + 14) / 16) <= 0x7fffffffLL;
}

tbn_status launch_linear_direct_ends(const LinearArgs &a) {
    if (a.k < 2) return TBN_OK;
    DirectLinearParams P = {};
    P.M = a.M; P.out = a.out;
    P.in = a.in;
    P.p = a.p;
    P.k = a.k;
    P.last_word = (a.p + 31) / 32 - 1;
    const int32_t ce = a.dt == TBN_F32 ? kChunkBytes / 4 : kChunkBytes / 2;
    P.chunks = (P.in + ce - 1) / ce;
    P.relu = (a.flags & TBN_FLAG_RELU) ? 1 : 0;
    P.groups = static_cast<uint32_t>((a.k - 1 + 15) / 16);
    P.row_tiles = static_cast<uint32_t>((a.M + 31) / 32);
    return a.dt == TBN_F32 ? launch_ends<float>(a, P) : launch_ends<uint16_t>(a, P);
}

tbn_status launch_linear_direct(const LinearArgs &a) {
    const DirectPlan pl = plan(a);
    DirectLinearParams P;
    P.M = a.M; P.out = a.out;
    P.in = a.in;
    P.U = static_cast<int32_t>(a.p / a.in);
    P.last_word = (a.p + 31) / 32 - 1;
    P.chunks = pl.chunks;
    P.reps = static_cast<int32_t>(a.out / (a.p / a.in));
    P.n_alpha = a.n_alpha;
    P.relu = (a.flags & TBN_FLAG_RELU) ? 1 : 0;
    P.groups = static_cast<uint32_t>(pl.groups);
    P.row_tiles = static_cast<uint32_t>(pl.row_tiles);
    if (pl.wide) return a.dt == TBN_F32 ? launch_one<float, 1, 8, true>(a, P) : launch_one<uint16_t, 1, 8, true>(a, P);
    return a.dt == TBN_F32 ? launch_nt<float>(a, P, pl.nt, pl.kw) : launch_nt<uint16_t>(a, P, pl.nt, pl.kw);
}

}  // namespace tbn
