// Fully-connected tiled-bit layer with binary activations (the paper's Conclusion names it as the first
// direction of future work and gives no formula; the reading built here: an activation becomes +1 or -1 by the
// rule Eq. 3 applies to a weight sum -- +1 where it is greater than zero -- and the layer operation stated after
// Eq. 8 is applied to those signs unchanged).  Activations travel as rows of sign bits, 32 per word.
//
// Kernels:
//   * sign_pack: real activations -> rows of sign bits (one pass over X, 16 bytes per lane where rows are whole
//     words, a wave ballot otherwise).
//   * binact_mfma (tile of whole weight rows, in % 256 == 0): Z = S T^T on the matrix cores in the 4-bit float
//     format (E2M1 holds +1 and -1 exactly; v_mfma_f32_32x32x64_f8f6f4 multiplies 64 elements of K per instruction, four
//     times the bfloat16 rate; the float32 sums of such products are exact).  A lane's operand for one instruction is 32 sign
//     bits in four registers of eight 4-bit values.  Both operands use the same assignment of K to lanes and registers, so a
//     dot product does not depend on what that assignment is.  The distinct columns are computed once and every replica is
//     written as alpha[t] * Z in whole 128-byte lines after a turn through LDS (Section "CNN Architectures": only one of the
//     tile computations needs to be executed); sign bits are formed in the accumulators' layout.  Two forms of the loop:
//       - STAGED (sign bits out, and long rows on many blocks): bits through LDS, one vector instruction per operand register (see
//         `operand`).  A wave issues an instruction every four cycles and a matrix instruction takes 32, so that seven vector
//         instructions per operand made 38 cycles of every product, and loads of 16 bytes from each of 32 rows, which the load path
//         takes 64 cycles for, made 55 - 62 by time stamps; here it is 47 with one workgroup per CU (five vector instructions per product, one of
//         them for the counts of set bits; 43 without the LDS reads).  What 12288 elements of K more take, over the products of a SIMD and
//         at 2.4 GHz: 50 cycles with one workgroup per CU (8192 x 4096 and 16384 -> 512, k = 1; 66 in the other form), 46 where two
//         share it (-> 8192; 73).  Graph replays on two cards: 8192 x 4096 -> 16384, k = 2: sign bits out 140 and 155
//         us before, 97 and 106 now, bfloat16 out 152 / 113 and 159 / 116 (eager calls 99 - 116 and 114 - 132, by how many follow one another: the clock
//         moves with the power); 8192 x 4096 -> 4096, k = 8, sign bits out 13.8 / 10.6 and 13.2 / 10.3 (the words formed
//         by comparisons and lane exchanges behind a turn through LDS took 4.7 of it, 1.9 now); 8192 x 256 -> 4096, k = 2, sign bits
//         out 11.9 / 8.4.  Tried: K dealt to two groups of four waves (37 cycles, but 1.1 us to add the sums and a later start: 12.2
//         us against 10.9 with sign bits out); 32-byte pieces of rows, whose LDS addresses are immediate (121 us against 113).
//       - else (real outputs of other rows): four shifts and and-ors, seven instructions, spread a word over four registers, the loads
//         go straight to registers and no wave waits for another: what staging adds per block costs short rows with real outputs
//         more than it gains (8192 x 256 -> 4096, k = 2, bfloat16 out 13.4 us and 15.8 staged).
//   * binact_staged: the same product for small and middle layers and for long rows up to 2048 blocks, in blocks of 64
//     x 64 whose four waves share K and whose bits pass through LDS (the reasons stand at the kernel, the line between
//     the two at binact_staged_preferred).
//   * binact_generic: every other legal shape, one thread per output, XOR and population count on whole words
//     where a word lies inside one tile copy, bit by bit where it crosses a tile end.
#include "tbn_common.h"

#include <type_traits>

namespace tbn {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // round to nearest even in hardware
}

// ---- sign bits ------------------------------------------------------------------------------------------

template <typename XT> struct Chunk;   // 16 bytes of activations -> one bit per element
template <> struct Chunk<float> {
    static constexpr int elems = 4;
    static __device__ __forceinline__ uint32_t bits(const u32x4_t &v) {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) m |= (__uint_as_float(v[i]) > 0.f ? 1u : 0u) << i;
        return m;
    }
};
template <> struct Chunk<uint16_t> {
    static constexpr int elems = 8;
    static __device__ __forceinline__ uint32_t bits(const u32x4_t &v) {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            m |= (__uint_as_float(v[i] << 16) > 0.f ? 1u : 0u) << (2 * i);
            m |= (__uint_as_float(v[i] & 0xffff0000u) > 0.f ? 1u : 0u) << (2 * i + 1);
        }
        return m;
    }
};

// Rows of whole words (in % 32 == 0): the rows of sign bits are then one bit stream over the flat activations.
// A lane takes 16 bytes; the 32 / elems lanes of a word OR their pieces together.
template <typename XT>
__global__ __launch_bounds__(256) void sign_pack_flat_kernel(const XT *__restrict__ x, uint32_t *__restrict__ xbits,
                                                             int64_t n_chunks) {
    constexpr int E = Chunk<XT>::elems, LPW = 32 / E;   // lanes per word: 8 (float32) or 4 (bfloat16)
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    // every lane of a wave runs the same number of rounds (the shuffles need all of them)
    const int64_t first = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t wave_first = first - (threadIdx.x & 63);
    for (int64_t base = wave_first; base < n_chunks; base += stride) {
        const int64_t c = base + (threadIdx.x & 63);
        uint32_t m = 0;
        if (c < n_chunks) {
            const u32x4_t v = *reinterpret_cast<const u32x4_t *>(reinterpret_cast<const unsigned char *>(x) + c * 16);
            m = Chunk<XT>::bits(v) << (E * static_cast<int>(c % LPW));
        }
#pragma unroll
        for (int d = 1; d < LPW; d <<= 1) m |= __shfl_xor(m, d);
        if (c < n_chunks && (c % LPW) == 0) xbits[c / LPW] = m;
    }
}

// Any row length: a wave takes 64 consecutive activations of one row; the ballot of "greater than zero" is the
// two words.  Lanes past the row's end vote 0, which is what the unused bits of a row's last word hold.
template <typename XT>
__global__ __launch_bounds__(256) void sign_pack_ballot_kernel(const XT *__restrict__ x, uint32_t *__restrict__ xbits,
                                                               int64_t M, int64_t in, int64_t groups, int64_t row_words) {
    const int lane = threadIdx.x & 63;
    const int64_t n_waves = int64_t(gridDim.x) * (blockDim.x >> 6);
    const int64_t total = M * groups;
    for (int64_t item = int64_t(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6); item < total; item += n_waves) {
        const int64_t m = item / groups, g = item - m * groups;
        const int64_t j = g * 64 + lane;
        const bool pos = j < in && ElemIO<XT>::load(x + m * in + j) > 0.f;
        const uint64_t vote = __ballot(pos);
        if (lane < 2 && 2 * g + lane < row_words)
            xbits[m * row_words + 2 * g + lane] = static_cast<uint32_t>(vote >> (32 * lane));
    }
}

// ---- shape-agnostic forward -----------------------------------------------------------------------------

struct BinactArgs {
    const uint32_t *xbits;
    void *y;
    int dt;
    int64_t M, in, out;
    const uint32_t *tile;
    int64_t p;
    int32_t k;
    const float *alpha;
    int32_t n_alpha;
    uint32_t flags;
    hipStream_t stream;
};

// One output of the layer.  The flat weight index of (o, j) is f = o*in + j: tile bit f % p, alpha[f / p].  The
// products of one tile copy are counted as integers (32 minus twice the differing bits per word) and scaled
// once; with one alpha, or a tile of whole rows, an output is a single product of a float and an integer.
__device__ __forceinline__ float binact_output(const uint32_t *__restrict__ xr, int64_t o, int64_t in, int64_t row_words,
                                               const uint32_t *__restrict__ tile, int64_t p, int64_t n_words,
                                               const float *__restrict__ alpha, int32_t n_alpha) {
    const int64_t f0 = o * in;
    int64_t q = f0 % p;          // tile position of the next weight
    int64_t c = f0 / p;          // tile copy it belongs to
    int32_t cnt = 0;             // sum of the +-1 products inside copy c so far
    float acc = 0.f;
    auto flush = [&]() {   // a tile copy ends; with one alpha for all copies the count simply runs on
        if (n_alpha != 1) {
            acc += alpha[c] * static_cast<float>(cnt);
            cnt = 0;
        }
        ++c;
        q = 0;
    };
    for (int64_t w = 0; w < row_words; ++w) {
        const uint32_t xw = xr[w];
        const int32_t nb = (in - 32 * w) < 32 ? static_cast<int32_t>(in - 32 * w) : 32;
        if (q + nb <= p) {
            const uint32_t win = tile_window32(tile, q, n_words);
            const uint32_t mask = nb == 32 ? 0xffffffffu : ((1u << nb) - 1u);
            cnt += nb - 2 * __popc((xw ^ win) & mask);
            q += nb;
            if (q == p) flush();
        } else {   // the word crosses a tile end
            for (int32_t b = 0; b < nb; ++b) {
                const uint32_t tb = (tile[q >> 5] >> (q & 31)) & 1u;
                cnt += (((xw >> b) & 1u) == tb) ? 1 : -1;
                if (++q == p) flush();
            }
        }
    }
    if (n_alpha == 1) acc = alpha[0] * static_cast<float>(cnt);
    else if (q != 0) acc += alpha[c] * static_cast<float>(cnt);   // the copy the row ends in
    return acc;
}

// one thread per output
template <typename YT>
__global__ __launch_bounds__(256) void binact_generic_kernel(const uint32_t *__restrict__ xbits, YT *__restrict__ y,
                                                             int64_t total, int64_t in, int64_t out, int64_t row_words,
                                                             const uint32_t *__restrict__ tile, int64_t p,
                                                             const float *__restrict__ alpha, int32_t n_alpha, int relu) {
    const int64_t n_words = (p + 31) / 32;
    for (int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; idx < total; idx += int64_t(gridDim.x) * blockDim.x) {
        const int64_t m = idx / out, o = idx - m * out;
        float acc = binact_output(xbits + m * row_words, o, in, row_words, tile, p, n_words, alpha, n_alpha);
        if (relu) acc = fmaxf(acc, 0.f);
        ElemIO<YT>::store(y + idx, acc);
    }
}

// sign bits out: one thread per word of 32 outputs
__global__ __launch_bounds__(256) void binact_generic_sign_kernel(const uint32_t *__restrict__ xbits, uint32_t *__restrict__ ybits,
                                                                  int64_t total_words, int64_t in, int64_t out, int64_t row_words,
                                                                  int64_t out_words, const uint32_t *__restrict__ tile, int64_t p,
                                                                  const float *__restrict__ alpha, int32_t n_alpha) {
    const int64_t n_words = (p + 31) / 32;
    for (int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; idx < total_words; idx += int64_t(gridDim.x) * blockDim.x) {
        const int64_t m = idx / out_words, wo = idx - m * out_words;
        uint32_t bits = 0;
        for (int b = 0; b < 32 && 32 * wo + b < out; ++b)
            bits |= (binact_output(xbits + m * row_words, 32 * wo + b, in, row_words, tile, p, n_words, alpha, n_alpha) > 0.f ? 1u : 0u) << b;
        ybits[idx] = bits;
    }
}

// ---- tile of whole rows, any row length: a thread per batch row and 32 distinct columns ---------------------
// For shapes the matrix-core kernel declines (rows that are no multiple of 256, numbers of distinct columns that are
// no multiple of 8).  With p a multiple of `in` only the U = p / in rows of the tile are distinct.  A workgroup owns
// 128 batch rows (one per thread) and 32 distinct columns, whose tile words pass through LDS, 128 words of K at a
// time (cut out of the tile at any bit offset, the last word of a row masked); a thread loads a word of its sign row
// once and counts the differing bits against the 32 columns' words, which every lane reads from the same LDS address:
// a word of 32 products costs an exclusive-or and a bit count.  Integer counts per output, one product with alpha per
// replica, as in binact_output.
constexpr int kDirCols = 32;
constexpr int kDirRows = 128;
constexpr int kDirStage = 128;   // words of K per pass

struct BinactDirectParams {
    int64_t M, in, out, U, row_words, n_words, out_words;
    int32_t reps, n_alpha, relu;
};

template <typename YT, bool SIGN>
__global__ __launch_bounds__(kDirRows) void binact_direct_kernel(const uint32_t *__restrict__ xbits, YT *__restrict__ y,
                                                                const uint32_t *__restrict__ tile,
                                                                const float *__restrict__ alpha, BinactDirectParams P) {
    __shared__ __attribute__((aligned(16))) uint32_t t_lds[kDirStage][kDirCols];
    const int tid = threadIdx.x;
    const int64_t m = int64_t(blockIdx.x) * kDirRows + tid;
    const int64_t u0 = int64_t(blockIdx.y) * kDirCols;
    const bool live = m < P.M;
    const uint32_t *xr = xbits + (live ? m : P.M - 1) * P.row_words;   // rows past M repeat the last one; never written
    const int32_t tail = static_cast<int32_t>(P.in & 31);               // bits in the last word of a row (0: all 32)

    int32_t cnt[kDirCols];   // differing bits
#pragma unroll
    for (int f = 0; f < kDirCols; ++f) cnt[f] = 0;

    for (int64_t w0 = 0; w0 < P.row_words; w0 += kDirStage) {
        const int32_t n = static_cast<int32_t>(P.row_words - w0 < kDirStage ? P.row_words - w0 : kDirStage);
        __syncthreads();   // the previous pass is done with the staged words
        for (int32_t i = tid; i < n * kDirCols; i += kDirRows) {
            const int32_t e = i / kDirCols, f = i % kDirCols;
            const int64_t u = u0 + f < P.U ? u0 + f : P.U - 1;   // columns past U repeat the last one; never written
            uint32_t tw = tile_window32(tile, u * P.in + 32 * (w0 + e), P.n_words);
            if (tail && w0 + e == P.row_words - 1) tw &= (1u << tail) - 1u;
            t_lds[e][f] = tw;
        }
        __syncthreads();
#pragma unroll 2
        for (int32_t e = 0; e < n; ++e) {
            uint32_t xw = xr[w0 + e];
            if (tail && w0 + e == P.row_words - 1) xw &= (1u << tail) - 1u;   // padding bits of a sign row do not count
            const uint4 *tv = reinterpret_cast<const uint4 *>(t_lds[e]);
#pragma unroll
            for (int g = 0; g < kDirCols / 4; ++g) {
                const uint4 t4 = tv[g];
                cnt[4 * g + 0] += __popc(xw ^ t4.x);
                cnt[4 * g + 1] += __popc(xw ^ t4.y);
                cnt[4 * g + 2] += __popc(xw ^ t4.z);
                cnt[4 * g + 3] += __popc(xw ^ t4.w);
            }
        }
    }

    if (!live) return;
    const int32_t in32 = static_cast<int32_t>(P.in);
    if constexpr (SIGN) {   // U is a multiple of 32: the 32 columns are one word of every replica
        uint32_t pos = 0, neg = 0;   // sum > 0, sum < 0
#pragma unroll
        for (int f = 0; f < kDirCols; ++f) {
            const int32_t z = in32 - 2 * cnt[f];
            pos |= (z > 0 ? 1u : 0u) << f;
            neg |= (z < 0 ? 1u : 0u) << f;
        }
        uint32_t *yr = reinterpret_cast<uint32_t *>(y) + m * P.out_words + (u0 >> 5);
        for (int32_t t = 0; t < P.reps; ++t) {
            const float al = alpha[P.n_alpha == 1 ? 0 : t];
            yr[int64_t(t) * (P.U >> 5)] = al > 0.f ? pos : (al < 0.f ? neg : 0u);
        }
    } else {
        YT *yr = y + m * P.out;
        for (int32_t t = 0; t < P.reps; ++t) {
            const float al = alpha[P.n_alpha == 1 ? 0 : t];
#pragma unroll
            for (int f = 0; f < kDirCols; ++f) {
                const int64_t u = u0 + f;
                if (u < P.U) {
                    float v = al * static_cast<float>(in32 - 2 * cnt[f]);
                    if (P.relu) v = fmaxf(v, 0.f);
                    ElemIO<YT>::store(yr + int64_t(t) * P.U + u, v);
                }
            }
        }
    }
}

// ---- matrix-core forward --------------------------------------------------------------------------------

constexpr int kTurnStride = 68;                   // floats per row of a wave's 64 x 64 sums in LDS
constexpr int kTurnBytes = 64 * kTurnStride * 4;  // per wave
// Stages of sign bits (STAGED), two super-steps of 256 batch and tile rows, 64 bytes a row, a ring of four.  Behind the loop the turn
// round, or the words of sign bits, take their place; the counts of set bits lie behind that.
constexpr int kStageBytes = 256 * 64;
constexpr int kRing = 4;
constexpr int count_off(bool sign) { return sign || kRing * kStageBytes > 4 * kTurnBytes ? kRing * kStageBytes : 4 * kTurnBytes; }
constexpr int mfma_lds(bool sign, bool staged) { return staged ? count_off(sign) + 256 * 4 : 4 * kTurnBytes; }

// s_waitcnt that waits for the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
// Reads of the stages are inline assembly: the compiler would make each wait for every global -> LDS load in flight.  The register is
// handed to the compiler by tie() behind the wait that covers the read.
template <int OFF>
__device__ __forceinline__ void lds_read16(u32x4_t &dst, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
template <int N>
__device__ __forceinline__ void lds_wait() {
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void tie(u32x4_t &r) { asm volatile("" : "+v"(r)); }
// An operand is formed, and a matrix instruction issued (the tie of its accumulators behind it), where it stands: left alone the compiler forms three
// operands in one slot and puts eight matrix instructions in a row.
__device__ __forceinline__ void pin(i32x8_t &f) {
    int f0 = f[0], f1 = f[1], f2 = f[2], f3 = f[3];
    asm volatile("" : "+v"(f0), "+v"(f1), "+v"(f2), "+v"(f3));
    f[0] = f0, f[1] = f1, f[2] = f2, f[3] = f3;
}
// A register that readlane reads later is loaded by every lane of the wave here: left alone the compiler may move the load to where it is
// read, behind a branch that the lanes which hold the wanted values did not take.
__device__ __forceinline__ void hold_in_all_lanes(float &v) { asm volatile("; held in all lanes: %0" : "+v"(v)); }
template <int V> using Int = std::integral_constant<int, V>;

struct BinactMfmaParams {
    int64_t M;
    int32_t in, out, U;
    int32_t reps;       // out / U
    int32_t n_alpha;
    int32_t tiles_n;    // column blocks of 128
    uint32_t tiles_m;   // row blocks of 128
    int32_t xcd_order;  // deal the column blocks of a row block to one XCD
    int32_t n_super;    // in / 256
    int32_t row_bytes;  // in / 8
};

// 256 threads = 4 waves in 2 x 2; a wave owns 64 batch rows x 64 distinct columns (2 x 2 MFMA tiles) over all of K.
// SIGN: the sign bits of the outputs are written instead of the outputs (U % 32 == 0; YT is then not used).
// STAGED: the bits pass through LDS as 64-byte pieces of rows, operands cost a vector instruction per register and half of them are
// counted; otherwise every lane loads for itself, seven vector instructions per operand, and no wave ever waits for another one,
// which is what short rows with real outputs want.
template <typename YT, bool RELU, bool SIGN, bool STAGED>
__global__ __launch_bounds__(256, 2) void binact_mfma_kernel(const uint32_t *__restrict__ xbits, YT *__restrict__ y,
                                                             const uint32_t *__restrict__ tile,
                                                             const float *__restrict__ alpha, BinactMfmaParams P) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, lh = lane >> 5;
    const uint32_t bid = blockIdx.x;
    // Workgroup ids are dealt round-robin to the 8 XCDs: the column blocks of one row block take consecutive slots of
    // one XCD, so that the rows of sign bits they share come from that XCD's L2 (the remaining row blocks: plain order).
    uint32_t tile_m, tile_n;
    {
        const uint32_t tiles_n = static_cast<uint32_t>(P.tiles_n), xcd = bid & 7, slot = bid >> 3;
        // (with real outputs and many column blocks the plain order measured 4 % faster: 8192 x 4096 -> 16384, k = 2 and 8)
        const uint32_t full = P.xcd_order ? (P.tiles_m / 8) * tiles_n : 0u;   // slots per XCD in the regular part
        if (slot < full) {
            const uint32_t q = slot / tiles_n;
            tile_n = slot - q * tiles_n;
            tile_m = q * 8 + xcd;
        } else {
            const uint32_t rest = bid - full * 8;
            const uint32_t q = rest / tiles_n;
            tile_n = rest - q * tiles_n;
            tile_m = (P.xcd_order ? (P.tiles_m / 8) * 8 : 0u) + q;
        }
    }
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t mb = int64_t(tile_m) * 128, m0 = mb + wm * 64;   // the block's and this wave's first batch row
    const int32_t nb = static_cast<int32_t>(tile_n) * 128, n0 = nb + wn * 64;   // and first distinct column

    // alpha of replica t in lane t (replicas past the 64th are fetched one by one in the epilogue)
    float alpha_lanes = alpha[P.n_alpha == 1 ? 0 : (lane < P.reps ? lane : P.reps - 1)];

    // The instruction leaves row 8*(r / 4) + 4*lh + r % 4 of its result in register r: with tile row column_of(l) from operand lane l,
    // register r of a lane is column 16*lh + r of the tile, sixteen adjacent columns.
    auto column_of = [](int l) { return 16 * ((l >> 2) & 1) + 4 * (l >> 3) + (l & 3); };
    // Operand t of either kind is the wave's batch rows 32*(t ^ row_turn) on, or its columns 32*(t ^ col_turn) on.
    const int row_turn = STAGED ? wn : 0, col_turn = STAGED ? wm : 0;
    f32x16_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
    float *const counts = reinterpret_cast<float *>(lds + count_off(SIGN));   // STAGED: 2 * set bits of the block's rows, then of its columns
    if constexpr (STAGED) {
        // ---- the sign bits of a stage: 16 wave-loads of 16 rows x 64 bytes, four per wave (waves 0 and 1: batch rows) -----
        // LDS row 128 + 64 w + 32 t + l holds distinct column 64 w + 32 t + column_of(l) of the block.  Rows past M and columns past U repeat the last one.  Piece c of LDS row r lies in slot c ^ (r / 4) % 4 of
        // the row's four: operand reads free of bank conflicts.
        const unsigned char *const src = wave < 2 ? reinterpret_cast<const unsigned char *>(xbits) + mb * P.row_bytes
                                                : reinterpret_cast<const unsigned char *>(tile) + int64_t(nb) * P.row_bytes;
        uint32_t from[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 64 * wn + 16 * j + (lane >> 2);   // LDS row, from the first batch row or the first tile row on
            const int64_t left = wave < 2 ? P.M - 1 - mb : int64_t(P.U - 1 - nb);
            const int want = wave < 2 ? r : (r & ~31) + column_of(r & 31);
            from[j] = static_cast<uint32_t>(want < left ? want : static_cast<int>(left)) * static_cast<uint32_t>(P.row_bytes);
        }
        const uint32_t piece = static_cast<uint32_t>((lane ^ (lane >> 4)) & 3) * 16u;
        const uint32_t last_piece = static_cast<uint32_t>(P.row_bytes) - 16u;
        auto fetch = [&](int32_t stage) __attribute__((always_inline)) {   // behind a row's end: its last piece, never used
            unsigned char *const dst = lds + (stage % kRing) * kStageBytes + wave * 4096;
            const uint32_t at = static_cast<uint32_t>(stage) * 64u + piece;
            const uint32_t off = at < last_piece ? at : last_piece;
#pragma unroll
            for (int j = 0; j < 4; ++j) __builtin_amdgcn_global_load_lds(src + (from[j] + off), dst + j * 1024, 16, 0, 0);
        };

        // ---- operands ---------------------------------------------------------------------------------------------------
        // Activations are the second operand, tile rows the first; operand 0 / 1 are the wave's batch rows 32*(t ^ row_turn) on, 2 / 3
        // its columns 32*(t ^ col_turn) on, so that each of the block's eight operands is the first of its kind in one wave, which
        // counts its bits.  A lane's words of a super-step are bytes 32*S + 16*lh .. + 15 of its row, and instruction c takes bits 4n + c of all four:
        //   c = 0, 1, 2: the bits where they are are the 4-bit floats 0.5, 1 and 2 (or 0), the block scales make every product of two set
        //                bits a 4: with s = 2a - 1 and t = 2b - 1 that is st = 4ab - 2a - 2b + 1, the rest from the counts of set bits;
        //   c = 3:       the bit is the sign of +-1 (0x2 or 0xA; a set bit gives -1 in both operands alike).
        // One vector instruction per register instead of seven per four.
        uint32_t rd[4];   // of a stage's first super-step; the second one's: ^ 32
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            auto at = [&](int r) { return static_cast<uint32_t>(r * 64 + ((lh ^ ((r >> 2) & 3)) << 4)); };
            rd[t] = at(64 * wm + 32 * (t ^ row_turn) + ln);
            rd[2 + t] = at(128 + 64 * wn + 32 * (t ^ col_turn) + ln);
        }
        uint32_t mask0 = 0x11111111u, mask1 = 0x22222222u, mask2 = 0x44444444u, mask3 = 0x88888888u, counted = 0x77777777u;
        asm volatile("" : "+v"(mask0), "+v"(mask1), "+v"(mask2), "+v"(mask3), "+v"(counted));   // registers: an and-or takes no constants of this size
        auto operand = [&](i32x8_t &f, const u32x4_t &w, auto c_c) __attribute__((always_inline)) {
            constexpr int C = decltype(c_c)::value;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                f[j] = static_cast<int>(C == 3 ? ((w[j] & mask3) | mask1) : (w[j] & (C == 0 ? mask0 : C == 1 ? mask1 : mask2)));
            pin(f);
        };

        uint32_t count[2] = {0, 0};      // set bits of operands 0 and 2, those of instruction 3 left out
        u32x4_t raw[2][4];
        i32x8_t F[2][4] = {};            // the upper four words of an operand are not read in this format
        // One super-step: four groups of four instructions.  In front of each instruction one operand of the next group is formed; the
        // words of the next super-step are requested in the first group and taken in the last one.
        auto step = [&](auto s_c, const uint32_t (&next)[4]) __attribute__((always_inline)) {   // S: half of the stage
            constexpr int S = decltype(s_c)::value, N = S ^ 1;
            auto group = [&](auto i_c) __attribute__((always_inline)) {
                constexpr int I = decltype(i_c)::value, C = (I + 1) & 3;
                uint32_t bits = 0;
                if constexpr (I == 3) lds_wait<0>();
                auto one = [&](auto q_c) __attribute__((always_inline)) {
                    constexpr int Q = decltype(q_c)::value;
                    if constexpr (I == 0) lds_read16<0>(raw[N][Q], next[Q]);
                    if constexpr (I == 3) tie(raw[N][Q]);
                    operand(F[(I & 1) ^ 1][Q], I < 3 ? raw[S][Q] : raw[N][Q], Int<C>{});
                    if constexpr ((Q & 1) == 0) bits = raw[S][Q][I] & counted;
                    else count[Q >> 1] += static_cast<uint32_t>(__builtin_popcount(bits));
                    asm volatile("" : "+v"(bits), "+v"(count[0]), "+v"(count[1]));
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int tm = Q >> 1, tn = Q & 1;
                    acc[tm][tn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(F[I & 1][2 + tn], F[I & 1][tm], acc[tm][tn], 4, 4, 0,
                                                                                  I == 0 ? 129 : I == 1 ? 128 : 0, 0, I == 0 ? 129 : I == 1 ? 128 : 0);
                    asm volatile("" : "+v"(acc[tm][tn]));   // issued here
                    __builtin_amdgcn_sched_barrier(0);
                };
                one(Int<0>{}); one(Int<1>{}); one(Int<2>{}); one(Int<3>{});
            };
            group(Int<0>{}); group(Int<1>{}); group(Int<2>{}); group(Int<3>{});
        };

        // Stage s + 1 is readable behind the barrier of stage s, which also frees the slot of stage s - 1 for stage s + 3.
        // (both scale operands zero: the form of the instruction without block scales, one issue slot instead of two)
        const int32_t n_stages = (P.n_super + 1) / 2;
        fetch(0);
        if (n_stages > 1) fetch(1);
        if (n_stages > 2) fetch(2);
        if (n_stages > 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));
        else if (n_stages > 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int f = 0; f < 4; ++f) lds_read16<0>(raw[0][f], rd[f]);
        lds_wait<0>();
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            tie(raw[0][f]);
            operand(F[0][f], raw[0][f], Int<0>{});
        }
        for (int32_t st = 0; st < n_stages; ++st) {
            if (st + 2 < n_stages) __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __builtin_amdgcn_s_barrier();
            if (st + 3 < n_stages) fetch(st + 3);
            const int32_t super = 2 * st;
            uint32_t here[4], next[4];
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                here[f] = (rd[f] ^ 32u) + static_cast<uint32_t>((st % kRing) * kStageBytes);
                next[f] = rd[f] + static_cast<uint32_t>(((st + 1) % kRing) * kStageBytes);
            }
            step(Int<0>{}, here);
            if (super + 1 < P.n_super) step(Int<1>{}, next);
        }

        // ---- counts of set bits ---------------------------------------------------------------------------------------
#pragma unroll
        for (int i = 0; i < 2; ++i) count[i] += static_cast<uint32_t>(__shfl_xor(static_cast<int>(count[i]), 32));
        if (lh == 0) {
            counts[64 * wm + 32 * wn + ln] = static_cast<float>(2 * count[0]);
            counts[128 + 64 * wn + 32 * wm + column_of(ln)] = static_cast<float>(2 * count[1]);
        }
        __syncthreads();   // the counts are there, and every wave is done with the stages
    } else {
        // Operand rows.  Activations (second operand): lane (ln, lh) supplies batch row 32*tm + ln.  Tile rows (first
        // operand): lane ln supplies distinct column 32*tn + column_of(ln).  K: bytes 32*S + 16*lh .. + 15 of the row for the
        // four instructions of super-step S, word i for instruction i.
        const unsigned char *a_row[2], *b_row[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            int64_t m = m0 + 32 * t + ln;
            m = m < P.M ? m : P.M - 1;
            a_row[t] = reinterpret_cast<const unsigned char *>(xbits) + m * P.row_bytes + 16 * lh;
            int32_t u = n0 + 32 * t + column_of(ln);
            u = u < P.U ? u : P.U - 1;
            b_row[t] = reinterpret_cast<const unsigned char *>(tile) + int64_t(u) * P.row_bytes + 16 * lh;
        }
        auto load = [&](u32x4_t (&r)[4], int32_t S) {
            r[0] = *reinterpret_cast<const u32x4_t *>(a_row[0] + S * 32);
            r[1] = *reinterpret_cast<const u32x4_t *>(a_row[1] + S * 32);
            r[2] = *reinterpret_cast<const u32x4_t *>(b_row[0] + S * 32);
            r[3] = *reinterpret_cast<const u32x4_t *>(b_row[1] + S * 32);
        };
        // 32 sign bits -> 32 four-bit floats: bit 4n + j becomes the sign of value n of register j (0x2 is +1.0, 0xA is -1.0).
        // A set bit gives -1 in both operands alike, so their products are those of the signs.
        uint32_t sign_bits = 0x88888888u, one_bits = 0x22222222u;
        asm volatile("" : "+v"(sign_bits), "+v"(one_bits));   // registers: an and-or takes no constants of this size
        auto expand = [&](i32x8_t &f, uint32_t word) {
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = static_cast<int>(((word << (3 - j)) & sign_bits) | one_bits);
        };


        // Sign bits are fetched two super-steps ahead into three rotating register sets (a super-step is 16
        // instructions, about a quarter of a microsecond: one would not cover a miss in the XCD's L2).
        const int32_t last = P.n_super - 1;
        u32x4_t raw[3][4];
        load(raw[0], 0);
        load(raw[1], 1 < last ? 1 : last);
        i32x8_t F[2][4] = {};   // [operand set][A0, A1, B0, B1]; the upper four words of an operand are not read in this format
#pragma unroll
        for (int f = 0; f < 4; ++f) expand(F[0][f], raw[0][f][0]);
        constexpr int kOne = 0;   // both scale operands zero: the compiler takes the form of the instruction without block scales
        // One super-step: four groups of four instructions.  In front of each instruction one operand of the next group is
        // expanded (seven vector instructions, 28 of the 32 cycles the matrix instruction before it runs).  The last
        // super-step loads itself once more and expands operands nobody multiplies: the body stays one straight line of code.
        auto step = [&](auto c_c, int32_t S) __attribute__((always_inline)) {
            constexpr int C = decltype(c_c)::value, N1 = (C + 1) % 3, N2 = (C + 2) % 3;
            load(raw[N2], S + 2 < last ? S + 2 : last);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = i & 1, n = s ^ 1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    constexpr int kOrder[4] = {0, 2, 3, 1};
                    const int f = kOrder[q];
                    expand(F[n][f], i < 3 ? raw[C][f][i + 1] : raw[N1][f][0]);
                    __builtin_amdgcn_sched_barrier(0);
                    const int tm = q >> 1, tn = q & 1;
                    acc[tm][tn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(F[s][2 + tn], F[s][tm], acc[tm][tn], 4, 4, 0, kOne, 0, kOne);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        int32_t S = 0;
        for (; S + 3 <= P.n_super; S += 3) {
            step(std::integral_constant<int, 0>{}, S);
            step(std::integral_constant<int, 1>{}, S + 1);
            step(std::integral_constant<int, 2>{}, S + 2);
        }
        if (S < P.n_super) {   // one or two super-steps are left; the register sets are back in their first roles
            step(std::integral_constant<int, 0>{}, S);
            if (S + 1 < P.n_super) step(std::integral_constant<int, 1>{}, S + 1);
        }
    }
    hold_in_all_lanes(alpha_lanes);   // rows past M and columns past U are left out below
    const float rest = 192.f * static_cast<float>(P.n_super);   // three quarters of K
    auto of_row = [&](int tm) __attribute__((always_inline)) { return rest - counts[64 * wm + 32 * (tm ^ row_turn) + ln]; };
    auto of_cols = [&](int tn, int a) __attribute__((always_inline)) {   // of columns 16*lh + 4*a .. + 3 of the tile
        return *reinterpret_cast<const f32x4_t *>(counts + 128 + 64 * wn + 32 * (tn ^ col_turn) + 16 * lh + 4 * a);
    };

    if constexpr (SIGN) {
        // alpha[t] * z is positive where z and alpha[t] have the same sign.  A lane shifts the signs of z ("negative") and of -z
        // ("positive") of its sixteen columns of a row into two halves of a register; the lane halves trade theirs, so that a lane
        // holds whole words of 32 columns, and every replica takes the "positive" or the "negative" word by the sign of its alpha
        // (zero or not a number: no bit).
        uint32_t *yb = reinterpret_cast<uint32_t *>(y);
        const int64_t out_words = P.out >> 5;
        const int32_t words_per_replica = P.U >> 5;
        uint32_t half[2][2];   // sixteen columns: "positive" in the low half, "negative" in the high half
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const float r = of_row(tm);
#pragma unroll
            for (int tn = 0; tn < 2; ++tn) {
                uint32_t pos = 0, neg = 0;
#pragma unroll
                for (int a = 3; a >= 0; --a) {
                    const f32x4_t c = of_cols(tn, a);
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        const float d = r - c[e], z = acc[tm][tn][4 * a + e] + d, minus = (c[e] - r) - acc[tm][tn][4 * a + e];   // (never -0)
                        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(z), 31);
                        pos = __builtin_amdgcn_alignbit(pos, __float_as_uint(minus), 31);
                    }
                }
                half[tm][tn] = pos | (neg << 16);
            }
        }
        // the lanes with lh = 0 take the words of the first row tile, those with lh = 1 those of the second; the block's words meet in LDS, [row][pos, neg][4 words], so that a store writes the 128 columns of a row and replica at once
        uint32_t *const words = reinterpret_cast<uint32_t *>(lds);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const auto v = __builtin_amdgcn_permlane32_swap(half[0][i], half[1][i], false, false);   // low columns, high columns
            const int row = 64 * wm + 32 * (lh ^ row_turn) + ln, word = 2 * wn + (i ^ col_turn);
            words[row * 8 + word] = (v[0] & 0xffffu) | (v[1] << 16);
            words[row * 8 + 4 + word] = (v[0] >> 16) | (v[1] & 0xffff0000u);
        }
        __syncthreads();
        const int row = tid & 127;
        const int64_t m = mb + row;
        if (m >= P.M) return;
        const u32x4_t wp = *reinterpret_cast<const u32x4_t *>(words + row * 8), wneg = *reinterpret_cast<const u32x4_t *>(words + row * 8 + 4);
        uint32_t *const yrow = yb + m * out_words + (nb >> 5);
        const int32_t left = (P.U - nb) >> 5;
        for (int32_t t = wave >> 1; t < P.reps; t += 2) {
            const float al = t < 64 ? __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha_lanes), t))
                                    : alpha[P.n_alpha == 1 ? 0 : t];
            const u32x4_t zero = {0u, 0u, 0u, 0u}, w = al > 0.f ? wp : (al < 0.f ? wneg : zero);
            uint32_t *dst = yrow + int64_t(t) * words_per_replica;
            if (left >= 4) {
                typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
                *reinterpret_cast<u32x4_a4 *>(dst) = w;
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (i < left) dst[i] = w[i];
            }
        }
        return;
    }

    // ---- turn the sums round through the wave's own LDS and write every replica ----------------------------
    float *zt = reinterpret_cast<float *>(lds + wave * kTurnBytes);
#pragma unroll
    for (int tm = 0; tm < 2; ++tm) {
        const int row = 32 * (tm ^ row_turn) + ln;
        const float r = STAGED ? of_row(tm) : 0.f;
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                f32x4_t v = {acc[tm][tn][4 * a], acc[tm][tn][4 * a + 1], acc[tm][tn][4 * a + 2], acc[tm][tn][4 * a + 3]};
                if constexpr (STAGED) {
                    const f32x4_t c = of_cols(tn, a);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += r - c[e];
                }
                *reinterpret_cast<f32x4_t *>(zt + row * kTurnStride + 32 * (tn ^ col_turn) + 16 * lh + 4 * a) = v;
            }
    }
    // a lane takes eight adjacent columns of one row; eight lanes cover the 64 columns of a row
    const int c8 = lane & 7, rsub = lane >> 3;
    const int32_t col = n0 + 8 * c8;
    if (col < P.U) {
#pragma unroll 1
        for (int q = 0; q < 8; ++q) {
            const int row = 8 * q + rsub;
            const int64_t m = m0 + row;
            if (m >= P.M) continue;
            const f32x4_t z0 = *reinterpret_cast<const f32x4_t *>(zt + row * kTurnStride + 8 * c8);
            const f32x4_t z1 = *reinterpret_cast<const f32x4_t *>(zt + row * kTurnStride + 8 * c8 + 4);
            YT *yrow = y + m * P.out + col;
            auto emit = [&](int32_t t, float al) __attribute__((always_inline)) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = al * z0[i];
                    v[4 + i] = al * z1[i];
                }
                if (RELU) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = fmaxf(v[i], 0.f);
                }
                if constexpr (sizeof(YT) == 4) {
                    f32x4_t o0 = {v[0], v[1], v[2], v[3]}, o1 = {v[4], v[5], v[6], v[7]};
                    *reinterpret_cast<f32x4_t *>(yrow + int64_t(t) * P.U) = o0;
                    *reinterpret_cast<f32x4_t *>(yrow + int64_t(t) * P.U + 4) = o1;
                } else {
                    u32x4_t o;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
                    *reinterpret_cast<u32x4_t *>(yrow + int64_t(t) * P.U) = o;
                }
            };
            const int32_t reps_in_lanes = P.reps < 64 ? P.reps : 64;
            for (int32_t t = 0; t < reps_in_lanes; ++t)
                emit(t, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha_lanes), t)));
            for (int32_t t = 64; t < P.reps; ++t) emit(t, alpha[P.n_alpha == 1 ? 0 : t]);
        }
    }
}

// ---- matrix-core forward of small and middle layers and of long rows: sign bits through LDS, K dealt to the waves ------------
// What bounds it: latency.  On small and middle layers there is one block per CU at most (or two), so a layer takes what one workgroup
// takes from its first load to its last store; long rows go through it in up to four rounds of two blocks per CU, whose stores and loads
// run under each other's products (8192 x 4096 -> 4096, k = 8, bfloat16 out: 1024 blocks, a wave multiplies 13 % of its time).
// binact_mfma_kernel's 128 x 128 block is 256 matrix instructions per wave behind loads that touch 32 lines each; here a block is 64 x 64,
// its four waves share K (64 instructions each at in = 4096), and the bits come as whole lines, once per workgroup, 32 KiB at a time
// through registers into one of two LDS slots, so that a stage's loads run under the products of the one before.  Stamps of 1024 x 4096 ->
// 4096, k = 8, sign bits out: 1.1 us to the first stage, 2.1 of products, 0.5 to exchange the sums, 1.5 for the words; kernel 13.1 us
// before and 6.3, one row 9.3 / 5.8; with operands and matrix instructions pinned to their places (see pin; the compiler put
// eight matrix instructions in a row behind their operands) 6.0, one row 5.4, 8192 x 4096 -> 4096, k = 8, bfloat16 out 17.9 against 17.2.  Tried: blocks of 128 x 128 with K dealt to two pairs of waves (13.6 us at any number of rows),
// products and expansions ordered instruction by instruction through inline assembly (6.2; at 8192 rows 16.7 against 16.3), LDS writes and
// loads dealt one behind each product (8.5).

struct BinactStagedParams {
    int64_t M;
    int32_t out, U;
    int32_t reps;       // out / U
    int32_t n_alpha;
    int32_t tiles_n;    // column blocks
    uint32_t tiles_m;   // row blocks
    int32_t n_super;    // in / 256
    int32_t row_bytes;  // in / 8
};

// A block of 64 batch rows x 64 distinct columns per workgroup; every wave takes all of it (2 x 2 MFMA tiles) over the
// super-steps (256 elements of K) congruent to its number (mod 4), and the four sums meet in LDS.
constexpr int kGroups = 4;                          // groups of waves that share K
constexpr int kStBM = 64, kStBN = 64;
constexpr int kStPieces = 4 * kGroups;                   // 16-byte pieces of a row per stage: two super-steps of every group
constexpr int kStStage = (kStBM + kStBN) * kStPieces * 16;   // 32 KiB
constexpr int kStStride = kStBN + 4;                // floats per row of a group's sums
constexpr int kStPlane = kStBM * kStStride;         // floats
constexpr int kStLds = kGroups * kStPlane * 4 > 2 * kStStage ? kGroups * kStPlane * 4 : 2 * kStStage;

// PIN: operands and matrix instructions stay where they stand, and sign bits' first alphas are fetched in front of the loop (387 drawn layers
// with sign bits out on 257 - 512 blocks, without / with: rows of 1280 - 2048 elements 0.98 in the mean, 2304 - 3072 0.99, 3328 - 4096
// 1.02, longer ones 1.06; with real outputs 1.00 - 1.04 at any length; from before the alphas came without branches, which gave either 1.02 - 1.04).
template <typename YT, bool RELU, bool SIGN, bool PIN>
__global__ __launch_bounds__(256, 2) void binact_staged_kernel(const uint32_t *__restrict__ xbits, YT *__restrict__ y,
                                                                            const uint32_t *__restrict__ tile,
                                                                            const float *__restrict__ alpha, BinactStagedParams P) {
    constexpr int TM = 2, TN = 2, BM = kStBM, BN = kStBN, NP = kStPieces, NF = TM + TN;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, lh = lane >> 5;
    const int grp = wave;                                  // K group
    const uint32_t bid = blockIdx.x;
    // Workgroup ids are dealt round-robin to the 8 XCDs: the column blocks of one row block take consecutive slots of
    // one XCD, so that the rows of sign bits they share come from that XCD's L2 (the remaining row blocks: plain order).
    uint32_t tile_m, tile_n;
    {
        const uint32_t tiles_n = static_cast<uint32_t>(P.tiles_n), xcd = bid & 7, slot = bid >> 3;
        const uint32_t full = (P.tiles_m / 8) * tiles_n;   // slots per XCD in the regular part
        if (slot < full) {
            const uint32_t q = slot / tiles_n;
            tile_n = slot - q * tiles_n;
            tile_m = q * 8 + xcd;
        } else {
            const uint32_t rest = bid - full * 8;
            const uint32_t q = rest / tiles_n;
            tile_n = rest - q * tiles_n;
            tile_m = (P.tiles_m / 8) * 8 + q;
        }
    }
    const int64_t m0 = int64_t(tile_m) * BM;
    const int32_t n0 = static_cast<int32_t>(tile_n) * BN;

    // ---- the sign bits of a stage: eight 16-byte pieces per thread, whole lines of a row ------------------------
    // LDS rows 0 .. BM - 1 are the batch rows, the BN behind them the tile rows; row BM + 32 t + l holds distinct column
    // 32 t + 16*((l >> 2) & 1) + 4*(l >> 3) + (l & 3): the instruction leaves row 8*(r / 4) + 4*lh + r % 4 of its result in
    // register r, so that register r of a lane is column 32 t + 16*lh + r, sixteen adjacent columns.  Rows past M and columns
    // past U repeat the last one.  Piece c of row r lies in slot c ^ swizzle(r) of the row: operand reads free of conflicts.
    constexpr int kPasses = (BM + BN) * NP / 256;          // 8
    static_assert(kPasses == 8 && BM * NP % 256 == 0, "a pass lies in the batch rows or in the tile rows");
    auto swizzle = [](int r) { return r & 15; };
    const unsigned char *src[2] = {reinterpret_cast<const unsigned char *>(xbits) + m0 * P.row_bytes,
                                   reinterpret_cast<const unsigned char *>(tile) + int64_t(n0) * P.row_bytes};
    uint32_t from[kPasses], to[kPasses];
    const int piece = tid % NP;
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
        const int r = i * (256 / NP) + tid / NP;
        const bool act = i < BM * NP / 256;
        const int l = r & 31, c = ((r - BM) & ~31) + 16 * ((l >> 2) & 1) + 4 * (l >> 3) + (l & 3);
        const int64_t left = act ? P.M - 1 - m0 : int64_t(P.U - 1 - n0);
        const int want = act ? r : c;
        from[i] = static_cast<uint32_t>(want < left ? want : static_cast<int>(left)) * static_cast<uint32_t>(P.row_bytes);
        to[i] = static_cast<uint32_t>(r * NP + (piece ^ swizzle(r))) * 16u;
    }
    const int32_t last_piece = P.row_bytes - 16;
    u32x4_t held[kPasses];   // the stage after the one in LDS
    auto fetch_all = [&](int32_t stage) __attribute__((always_inline)) {   // behind a row's end: its last piece, never used
        const int32_t at = stage * (NP * 16) + piece * 16;
        const uint32_t off = static_cast<uint32_t>(at < last_piece ? at : last_piece);
#pragma unroll
        for (int i = 0; i < kPasses; ++i)
            held[i] = *reinterpret_cast<const u32x4_t *>(src[i < BM * NP / 256 ? 0 : 1] + (from[i] + off));
    };
    auto put = [&](int i, uint32_t at) __attribute__((always_inline)) { *reinterpret_cast<u32x4_t *>(lds + at + to[i]) = held[i]; };
    auto lds_barrier = [] __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    // Operands of a super-step: piece 2 * (kGroups * j + grp) + lh of rows 32 t + ln, word i for instruction i.
    uint32_t op_row[NF];
    int op_swz[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int r = f < TM ? 32 * f + ln : BM + 32 * (f - TM) + ln;
        op_row[f] = static_cast<uint32_t>(r * NP * 16);
        op_swz[f] = swizzle(r);
    }
    auto read = [&](u32x4_t (&r)[NF], uint32_t at, int j) __attribute__((always_inline)) {
        const int c = 2 * (kGroups * j + grp) + lh;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            r[f] = *reinterpret_cast<const u32x4_t *>(lds + at + op_row[f] + static_cast<uint32_t>(c ^ op_swz[f]) * 16u);
    };
    // 32 sign bits -> 32 four-bit floats: bit 4n + j becomes the sign of value n of register j (0x2 is +1.0, 0xA is -1.0).
    // A set bit gives -1 in both operands alike, so their products are those of the signs.
    uint32_t sign_bits = 0x88888888u, one_bits = 0x22222222u;
    asm volatile("" : "+v"(sign_bits), "+v"(one_bits));   // registers: an and-or takes no constants of this size
    auto expand = [&](i32x8_t &f, uint32_t word) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = static_cast<int>(((word << (3 - j)) & sign_bits) | one_bits);
        if constexpr (PIN) pin(f);
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    const int32_t n_stages = (P.n_super + 2 * kGroups - 1) / (2 * kGroups);
    fetch_all(0);
#pragma unroll
    for (int i = 0; i < kPasses; ++i) put(i, 0);
    if (n_stages > 1) fetch_all(1);
    // alpha of replica t in lane t (replicas past the 64th are fetched one by one below); sign bits out: a lane's first eight
    // replicas (up to 16 replicas in all)
    float alpha_lanes = 0.f, al_own[8] = {};
    const int32_t last_alpha = P.n_alpha == 1 ? 0 : P.reps - 1;
    auto first_alphas = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int32_t t = lh + 2 * c;
            // (With the choice between one scalar and many made here, the compiler put a branch around every load and they came one after the
            // other: 2600 drawn layers with sign bits out 1.03 - 1.04 times as fast without, 16 x 512 -> 8192, k = 8 4.47 us / 4.2.)
            al_own[c] = alpha[t < last_alpha ? t : last_alpha];
        }
    };
    if constexpr (!SIGN) alpha_lanes = alpha[P.n_alpha == 1 ? 0 : (lane < P.reps ? lane : P.reps - 1)];
    else if constexpr (PIN) first_alphas();
    lds_barrier();
    u32x4_t raw[2][NF];
    read(raw[0], 0, 0);
    i32x8_t F[2][NF] = {};   // the upper four words of an operand are not read in this format
#pragma unroll
    for (int f = 0; f < NF; ++f) expand(F[0][f], raw[0][f][0]);
    constexpr int kOne = 0;   // both scale operands zero: the compiler takes the form of the instruction without block scales
    // One super-step: four groups of four instructions; in front of an instruction one operand of the next group is expanded.
    auto multiply = [&](const u32x4_t (&r)[NF], const u32x4_t (&r_next)[NF]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = i & 1, n = s ^ 1;
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                expand(F[n][q], i < 3 ? r[q][i + 1] : r_next[q][0]);
                __builtin_amdgcn_sched_barrier(0);
                const int tm = q >> 1, tn = q & 1;
                acc[tm][tn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(F[s][TM + tn], F[s][tm], acc[tm][tn], 4, 4, 0, kOne, 0, kOne);
                if constexpr (PIN) asm volatile("" : "+v"(acc[tm][tn]));   // issued here
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // Two LDS slots: stage s + 1 goes to LDS while the first half of stage s is multiplied; the barrier between the halves
    // publishes it and frees the slot of stage s (every wave's reads of it have arrived by then).
    uint32_t slot = 0;
    for (int32_t st = 0; st < n_stages; ++st) {
        const int32_t first = st * (2 * kGroups) + grp;
        const uint32_t other = slot ^ static_cast<uint32_t>(kStStage);
        read(raw[1], slot, 1);
        if (st + 1 < n_stages) {
#pragma unroll
            for (int i = 0; i < kPasses; ++i) put(i, other);
            if (st + 2 < n_stages) fetch_all(st + 2);
        }
        if (first < P.n_super) multiply(raw[0], raw[1]);
        lds_barrier();
        if (st + 1 < n_stages) read(raw[0], other, 0);
        if (first + kGroups < P.n_super) multiply(raw[1], raw[0]);
        slot = other;
    }

    // ---- the groups' sums meet in LDS (nothing reads the stages behind the last barrier); every replica is written --------
    float *planes = reinterpret_cast<float *>(lds);
    constexpr int STR = kStStride;
    {
        float *zt = planes + grp * kStPlane;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f32x4_t v = {acc[tm][tn][4 * a], acc[tm][tn][4 * a + 1], acc[tm][tn][4 * a + 2], acc[tm][tn][4 * a + 3]};
                    *reinterpret_cast<f32x4_t *>(zt + (32 * tm + ln) * STR + 32 * tn + 16 * lh + 4 * a) = v;
                }
    }
    hold_in_all_lanes(alpha_lanes);   // columns past U are left out below
    lds_barrier();
    // a wave takes a quarter of the rows
    if constexpr (SIGN) {
        // alpha[t] * z is positive where z and alpha[t] have the same sign: a lane adds up one column of a row, and the votes
        // "z > 0" and "z < 0" of the wave are the words of 64 columns.  A pass takes as many rows as make 32 words; lane l
        // stores word l % 32 of the pass for replicas l / 32, l / 32 + 2, ..., the "positive" or the "negative" word by the
        // sign of that replica's alpha (zero or not a number: no bit).
        uint32_t *yb = reinterpret_cast<uint32_t *>(y);
        const int64_t out_words = P.out >> 5;
        constexpr int WPR = BN / 32, RPP = 32 / WPR;          // words of a row, rows per pass
        if constexpr (!PIN) first_alphas();
        const int slot_w = lane & 31, t_first = lane >> 5;
        const int32_t colw = n0 + 32 * (slot_w % WPR);
        const int32_t words_per_replica = P.U >> 5;
#pragma unroll 1
        for (int q = 0; q < BM / 4 / RPP; ++q) {
            const int row0 = wave * (BM / 4) + q * RPP;
            uint64_t wp = 0, wn = 0;   // the words of 64 columns that this lane stores one of
            float part[RPP][BN / 64][kGroups];   // every read is issued before the first sum
#pragma unroll
            for (int r = 0; r < RPP; ++r)
#pragma unroll
                for (int h = 0; h < BN / 64; ++h)
#pragma unroll
                    for (int g = 0; g < kGroups; ++g) part[r][h][g] = planes[g * kStPlane + (row0 + r) * STR + 64 * h + lane];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < RPP; ++r) {
#pragma unroll
                for (int h = 0; h < BN / 64; ++h) {
                    float sum = part[r][h][0];
#pragma unroll
                    for (int g = 1; g < kGroups; ++g) sum += part[r][h][g];
                    const uint64_t pos = __ballot(sum > 0.f), neg = __ballot(sum < 0.f);
                    const bool mine = (slot_w >> 1) == r * (WPR / 2) + h;
                    wp = mine ? pos : wp;
                    wn = mine ? neg : wn;
                }
            }
            const int up = 32 * (slot_w & 1);
            const uint32_t sp = static_cast<uint32_t>(wp >> up), sn = static_cast<uint32_t>(wn >> up);
            const int64_t m = m0 + row0 + slot_w / WPR;
            if (m < P.M && colw < P.U) {
                uint32_t *dst = yb + m * out_words + (colw >> 5);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const int32_t t = t_first + 2 * c;
                    if (t < P.reps) dst[int64_t(t) * words_per_replica] = al_own[c] > 0.f ? sp : (al_own[c] < 0.f ? sn : 0u);
                }
                for (int32_t t = t_first + 16; t < P.reps; t += 2) {
                    const float al = alpha[P.n_alpha == 1 ? 0 : t];
                    dst[int64_t(t) * words_per_replica] = al > 0.f ? sp : (al < 0.f ? sn : 0u);
                }
            }
        }
        return;
    }
    // a lane takes eight adjacent columns of one row
    constexpr int LPR = BN / 8, RPP = 64 / LPR, PASSES = BM / 4 / RPP;   // lanes per row, rows per pass
    const int c8 = lane % LPR, rsub = lane / LPR;
    const int row_first = wave * (BM / 4) + rsub;
    auto sums = [&](int row, f32x4_t &z0, f32x4_t &z1) __attribute__((always_inline)) {
        const float *z = planes + row * STR + 8 * c8;
        z0 = *reinterpret_cast<const f32x4_t *>(z);
        z1 = *reinterpret_cast<const f32x4_t *>(z + 4);
#pragma unroll
        for (int g = 1; g < kGroups; ++g) {
            z0 += *reinterpret_cast<const f32x4_t *>(z + g * kStPlane);
            z1 += *reinterpret_cast<const f32x4_t *>(z + g * kStPlane + 4);
        }
    };
    const int32_t col = n0 + 8 * c8;
    if (col < P.U) {
#pragma unroll 1
        for (int q = 0; q < PASSES; ++q) {
            const int row = row_first + q * RPP;
            const int64_t m = m0 + row;
            if (m >= P.M) continue;
            f32x4_t z0, z1;
            sums(row, z0, z1);
            YT *yrow = y + m * P.out + col;
            auto emit = [&](int32_t t, float al) __attribute__((always_inline)) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = al * z0[i];
                    v[4 + i] = al * z1[i];
                }
                if (RELU) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = fmaxf(v[i], 0.f);
                }
                if constexpr (sizeof(YT) == 4) {
                    f32x4_t o0 = {v[0], v[1], v[2], v[3]}, o1 = {v[4], v[5], v[6], v[7]};
                    *reinterpret_cast<f32x4_t *>(yrow + int64_t(t) * P.U) = o0;
                    *reinterpret_cast<f32x4_t *>(yrow + int64_t(t) * P.U + 4) = o1;
                } else {
                    u32x4_t o;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
                    *reinterpret_cast<u32x4_t *>(yrow + int64_t(t) * P.U) = o;
                }
            };
            const int32_t reps_in_lanes = P.reps < 64 ? P.reps : 64;
            for (int32_t t = 0; t < reps_in_lanes; ++t)
                emit(t, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha_lanes), t)));
            for (int32_t t = 64; t < P.reps; ++t) emit(t, alpha[P.n_alpha == 1 ? 0 : t]);
        }
    }
}

template <typename YT, bool RELU, bool SIGN = false, bool PIN = true>
static tbn_status launch_staged_t(const BinactArgs &a, const BinactStagedParams &P) {
    static const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&binact_staged_kernel<YT, RELU, SIGN, PIN>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, kStLds);
    if (e != hipSuccess) {
        set_error("tbn_linear_forward_binact: the matrix-core kernel was refused %d bytes of LDS", kStLds);
        (void)hipGetLastError();
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL((binact_staged_kernel<YT, RELU, SIGN, PIN>), dim3(P.tiles_m * static_cast<uint32_t>(P.tiles_n)), dim3(256),
                       kStLds, a.stream, a.xbits, static_cast<YT *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward_binact (matrix-core kernel)");
}

static tbn_status launch_binact_staged(const BinactArgs &a) {
    const int64_t U = a.p / a.in;
    BinactStagedParams P;
    P.M = a.M;
    P.out = static_cast<int32_t>(a.out);
    P.U = static_cast<int32_t>(U);
    P.reps = static_cast<int32_t>(a.out / U);
    P.n_alpha = a.n_alpha;
    P.tiles_n = static_cast<int32_t>((U + kStBN - 1) / kStBN);
    P.tiles_m = static_cast<uint32_t>((a.M + kStBM - 1) / kStBM);
    P.n_super = static_cast<int32_t>(a.in / 256);
    P.row_bytes = static_cast<int32_t>(a.in / 8);
    const bool relu = (a.flags & TBN_FLAG_RELU) != 0;
    if (a.flags & TBN_FLAG_SIGN_OUT) return a.in > 3072 ? launch_staged_t<float, false, true>(a, P) : launch_staged_t<float, false, true, false>(a, P);
    if (a.dt == TBN_F32) return relu ? launch_staged_t<float, true>(a, P) : launch_staged_t<float, false>(a, P);
    return relu ? launch_staged_t<uint16_t, true>(a, P) : launch_staged_t<uint16_t, false>(a, P);
}

bool binact_mfma_supported(const BinactArgs &a) {
    if (a.p % a.in != 0 || a.in % 256 != 0) return false;
    const int64_t U = a.p / a.in;
    if (U % 8 != 0 || a.out % U != 0) return false;
    if ((a.flags & TBN_FLAG_SIGN_OUT) && U % 32 != 0) return false;   // a word of sign bits lies in one replica
    if (a.in > (int64_t(1) << 24) || a.out > (int64_t(1) << 30) || U > (int64_t(1) << 24)) return false;
    if ((reinterpret_cast<uintptr_t>(a.xbits) | reinterpret_cast<uintptr_t>(a.tile) | reinterpret_cast<uintptr_t>(a.y)) & 15u) return false;
    const int64_t blocks = ((a.M + 127) / 128) * ((U + 127) / 128);
    return blocks <= 0x7fffffffLL;
}

constexpr int64_t kCountedRows = int64_t(1) << 22;   // sums of four times the set bits both operands have are exact in float32 up to here

// Real outputs: long rows on more than one and a half blocks per CU take the 128 x 128 blocks with staged bits (205 drawn layers of more
// than 1024 blocks of 64 x 64, as graph replays against the other kernels: rows of 2304 - 3072 elements 1.02 - 1.11 in the mean, longer ones
// 1.08 - 1.23; up to 2048 elements 0.84 - 1.03, and on fewer blocks 0.91 - 1.0, with more than 4096 elements 1.04 - 1.14 there, where no line
// has been drawn: those stay with the blocks of 64 x 64).  Rows of Y that do not start on lines lose (4765 x 3328 -> 13184, k = 8, float32: 62.6 us
// and 70.4); U % 64 sees to that for both types, float32 with U % 64 == 32 was not drawn by itself and stays where it was.
bool binact_long_rows(const BinactArgs &a) {
    const int64_t U = a.p / a.in;
    return a.in > 2048 && a.in <= kCountedRows && U % 64 == 0 && ((a.M + 127) / 128) * ((U + 127) / 128) > 384;
}

// Where the staged kernel's blocks of 64 x 64 beat the 128 x 128 of binact_mfma_kernel (400 drawn layers of 1 - 8192 rows, 256 -
// 4096 elements and columns, k = 2, 4, 8, as graph replays): a workgroup takes a quarter of the time, so while there is a CU for
// each of them the larger blocks leave CUs idle (geometric mean 1.41 times as fast at up to 256 blocks, 1024 x 4096 -> 4096, k = 8,
// bfloat16 out 14.6 us against 7.1, sign bits 13.1 / 6.3).  With two per CU they still win with sign bits out
// of rows of more than 1024 elements or with column blocks of 128 to fill (4096 x 4096 13.6 / 9.0; shorter rows, 95 drawn layers of 257 - 512
// blocks: these take 1.18 times the 128 x 128 blocks' time up to 512 elements, 1.08 up to 1024; 1536 - 2048 0.9 in the mean; 1508 x 512 -> 5888,
// k = 8, 736 columns: 6.5 / 5.8) and, up to 384, with real outputs of at least three super-steps; beyond, what
// every block pays beside its products (the first stage, the four sums of each output through LDS) costs short rows more than the filling
// gains (8192 x 1024 -> 1024, k = 2: 8.0 / 9.5).  Drawn again, 381 layers inside these lines: 1.34 on the mean, one more than 3 % slower.  Real outputs of up to 64 short
// rows: 14 x 256 -> 1536, k = 4: 4.1 / 4.6.
bool binact_staged_preferred(const BinactArgs &a) {
    const int64_t U = a.p / a.in, blocks = ((a.M + kStBM - 1) / kStBM) * ((U + kStBN - 1) / kStBN);
    if (a.flags & TBN_FLAG_SIGN_OUT) {
        // Short rows whose columns fill blocks of 128, but not with eight replicas or more on 8 - 13 row blocks: eight are the fewest whose column blocks
        // share an XCD, which completes the lines of the many stores there; blocks of 128 reach that with twice the rows.  These blocks' time
        // over the others', 1400 drawn layers, by 8, 9, 10, 11, 12, 13 row blocks: rows of 1024 elements 0.88, 0.91, 0.95, 0.96, 0.99, 0.99, of 768
        // 0.91, 0.94, 0.96, 0.99, 0.99, 0.95, of 512 0.97, 0.98, 0.97, 1.05, 1.07, 1.10; up to seven 1.15 - 1.3, from 14 on 1.02 - 1.3, fewer replicas
        // 1.0 - 1.25 at any number (488 x 1024 -> 32768, k = 8: 5.9 us and 6.9).
        const int64_t row_blocks = (a.M + kStBM - 1) / kStBM;
        const bool eight = a.in >= 512 && a.out / U >= 8 && row_blocks >= 8 && row_blocks <= (a.in > 512 ? 13 : 10);
        return blocks <= (a.in > 1024 || U % 128 != 0 || eight ? 512 : 256) || a.in > kCountedRows;
    }
    if (binact_long_rows(a)) return false;
    if (a.in < 768) return a.M > 64 && blocks <= 256;
    if (blocks <= 384) return true;
    // Real outputs of long rows, 385 - 2048 blocks, by rounds of two blocks per CU (2 x 420 layers of 2048 - 16384 elements and 1 - 16
    // replicas, graph replays, 128 x 128 blocks / these, range and mean): from 4096 elements on float32 0.97 - 1.63, 1.22; bfloat16 with at
    // most half of the last round filled, where the larger blocks fill theirs as little, 0.97 - 1.59, 1.23, with more of it at eight replicas
    // 0.96 - 1.82, 1.27 (8192 x 4096 -> 4096, k = 8: 21.4 us / 19.8; fewer replicas 0.96 - 1.71, not taken).  3072 - 3840 elements: at eight
    // replicas and more 0.94 - 1.38, 1.10 over the layers taken; at fewer 0.76 - 1.38, mostly lost (1947 x 3328 -> 3392, k = 1, bfloat16: 16.8 us / 22.2).
    // Shorter: 0.74 - 1.38.  Of the 256 layers of both draws that these lines take six are more than 3 % slower, by 6 % at most.
    const int64_t reps = a.out / U;
    if (a.in < (reps >= 8 ? 3072 : 4096) || blocks > 2048) return false;
    return a.dt == TBN_F32 || (blocks - 1) % 512 < 256 || (a.in >= 4096 && reps >= 8);
}

// Does binact_mfma_kernel count set bits (its STAGED form)?
bool binact_counted(const BinactArgs &a) { return (a.flags & TBN_FLAG_SIGN_OUT) != 0 || binact_long_rows(a); }

template <typename YT, bool RELU, bool SIGN, bool STAGED>
static tbn_status launch_mfma_s(const BinactArgs &a, const BinactMfmaParams &P, unsigned blocks) {
    constexpr int bytes = mfma_lds(SIGN, STAGED);
    // the permission for more than 64 KiB of LDS, once per process
    static const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&binact_mfma_kernel<YT, RELU, SIGN, STAGED>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) {
        set_error("tbn_linear_forward_binact: the matrix-core kernel was refused %d bytes of LDS", bytes);
        (void)hipGetLastError();
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL((binact_mfma_kernel<YT, RELU, SIGN, STAGED>), dim3(blocks), dim3(256), bytes, a.stream, a.xbits,
                       static_cast<YT *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward_binact (matrix-core kernel)");
}
template <typename YT, bool RELU>
static tbn_status launch_mfma_t(const BinactArgs &a, const BinactMfmaParams &P, unsigned blocks) {
    return binact_counted(a) ? launch_mfma_s<YT, RELU, false, true>(a, P, blocks) : launch_mfma_s<YT, RELU, false, false>(a, P, blocks);
}

tbn_status launch_binact_mfma(const BinactArgs &a) {
    const int64_t U = a.p / a.in;
    BinactMfmaParams P;
    P.M = a.M;
    P.in = static_cast<int32_t>(a.in);
    P.out = static_cast<int32_t>(a.out);
    P.U = static_cast<int32_t>(U);
    P.reps = static_cast<int32_t>(a.out / U);
    P.n_alpha = a.n_alpha;
    P.tiles_n = static_cast<int32_t>((U + 127) / 128);
    P.tiles_m = static_cast<uint32_t>((a.M + 127) / 128);
    // (sign bits out with 64 column blocks: the same time in both orders, but the 4 MiB of tile rows of a row block then
    // pass through every XCD's L2 once per row block, 203 MB fetched instead of 40)
    P.xcd_order = P.tiles_n <= ((a.flags & TBN_FLAG_SIGN_OUT) ? 32 : 4) ? 1 : 0;
    P.n_super = static_cast<int32_t>(a.in / 256);
    P.row_bytes = static_cast<int32_t>(a.in / 8);
    const unsigned blocks = static_cast<unsigned>(((a.M + 127) / 128) * P.tiles_n);
    const bool relu = (a.flags & TBN_FLAG_RELU) != 0;
    if (a.flags & TBN_FLAG_SIGN_OUT) return launch_mfma_s<float, false, true, true>(a, P, blocks);
    if (a.dt == TBN_F32) return relu ? launch_mfma_t<float, true>(a, P, blocks) : launch_mfma_t<float, false>(a, P, blocks);
    return relu ? launch_mfma_t<uint16_t, true>(a, P, blocks) : launch_mfma_t<uint16_t, false>(a, P, blocks);
}

tbn_status launch_binact_generic(const BinactArgs &a) {
    if (a.flags & TBN_FLAG_SIGN_OUT) {
        const int64_t out_words = (a.out + 31) / 32, total_words = a.M * out_words;
        int64_t blocks = (total_words + 255) / 256;
        if (blocks > (1 << 20)) blocks = 1 << 20;
        hipLaunchKernelGGL(binact_generic_sign_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, a.stream, a.xbits,
                           static_cast<uint32_t *>(a.y), total_words, a.in, a.out, (a.in + 31) / 32, out_words, a.tile, a.p,
                           a.alpha, a.n_alpha);
        return check_launch("tbn_linear_forward_binact (generic kernel, sign bits out)");
    }
    const int64_t total = a.M * a.out;
    int64_t blocks = (total + 255) / 256;
    if (blocks > (1 << 20)) blocks = 1 << 20;
    const int relu = (a.flags & TBN_FLAG_RELU) ? 1 : 0;
    const int64_t row_words = (a.in + 31) / 32;
    if (a.dt == TBN_F32)
        hipLaunchKernelGGL(binact_generic_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, a.stream, a.xbits,
                           static_cast<float *>(a.y), total, a.in, a.out, row_words, a.tile, a.p, a.alpha, a.n_alpha, relu);
    else
        hipLaunchKernelGGL(binact_generic_kernel<uint16_t>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, a.stream,
                           a.xbits, static_cast<uint16_t *>(a.y), total, a.in, a.out, row_words, a.tile, a.p, a.alpha,
                           a.n_alpha, relu);
    return check_launch("tbn_linear_forward_binact (generic kernel)");
}

bool binact_direct_supported(const BinactArgs &a) {
    if (a.M < 1 || a.p % a.in != 0 || a.in >= (int64_t(1) << 31)) return false;
    const int64_t U = a.p / a.in;
    if (U < 1 || U > a.out || a.out % U != 0 || a.out / U > (1 << 30)) return false;
    if (a.n_alpha != 1 && a.n_alpha != a.out / U) return false;
    if ((a.flags & TBN_FLAG_SIGN_OUT) && U % 32 != 0) return false;   // a word of sign bits lies in one replica
    return (a.M + kDirRows - 1) / kDirRows <= 0x7fffffffLL && (U + kDirCols - 1) / kDirCols <= 65535;
}

tbn_status launch_binact_direct(const BinactArgs &a) {
    BinactDirectParams P;
    P.M = a.M; P.in = a.in; P.out = a.out;
    P.U = a.p / a.in;
    P.row_words = (a.in + 31) / 32;
    P.n_words = (a.p + 31) / 32;
    P.out_words = (a.out + 31) / 32;
    P.reps = static_cast<int32_t>(a.out / P.U);
    P.n_alpha = a.n_alpha;
    P.relu = (a.flags & TBN_FLAG_RELU) ? 1 : 0;
    const dim3 grid(static_cast<unsigned>((a.M + kDirRows - 1) / kDirRows), static_cast<unsigned>((P.U + kDirCols - 1) / kDirCols));
    if (a.flags & TBN_FLAG_SIGN_OUT)
        hipLaunchKernelGGL((binact_direct_kernel<float, true>), grid, dim3(kDirRows), 0, a.stream, a.xbits,
                           static_cast<float *>(a.y), a.tile, a.alpha, P);
    else if (a.dt == TBN_F32)
        hipLaunchKernelGGL((binact_direct_kernel<float, false>), grid, dim3(kDirRows), 0, a.stream, a.xbits,
                           static_cast<float *>(a.y), a.tile, a.alpha, P);
    else
        hipLaunchKernelGGL((binact_direct_kernel<uint16_t, false>), grid, dim3(kDirRows), 0, a.stream, a.xbits,
                           static_cast<uint16_t *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward_binact (direct kernel)");
}

enum class BinactKernel { Staged, MatrixCore, Direct, Generic };

BinactKernel choose_binact(const BinactArgs &a) {
    if (!(a.flags & TBN_FLAG_FORCE_GENERIC)) {
        if (binact_mfma_supported(a)) return binact_staged_preferred(a) ? BinactKernel::Staged : BinactKernel::MatrixCore;
        // (at small batches with short rows one thread per output is level or ahead: 64 rows of 1000 bits 12.7 us
        // against 22.4)
        if ((a.M > 64 || a.in >= 2048) && binact_direct_supported(a)) return BinactKernel::Direct;
    }
    return BinactKernel::Generic;
}

}  // namespace

tbn_status launch_sign_pack(const void *x, int dt, int64_t M, int64_t in, uint32_t *xbits, hipStream_t stream) {
    const int64_t row_words = (in + 31) / 32;
    if (in % 32 == 0 && !(reinterpret_cast<uintptr_t>(x) & 15u)) {
        const int64_t n_chunks = M * in / (dt == TBN_F32 ? 4 : 8);
        int64_t blocks = (n_chunks + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        if (dt == TBN_F32)
            hipLaunchKernelGGL(sign_pack_flat_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                               static_cast<const float *>(x), xbits, n_chunks);
        else
            hipLaunchKernelGGL(sign_pack_flat_kernel<uint16_t>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                               static_cast<const uint16_t *>(x), xbits, n_chunks);
        return check_launch("tbn_sign_pack");
    }
    const int64_t groups = (in + 63) / 64;
    int64_t blocks = (M * groups + 3) / 4;
    if (blocks > 16384) blocks = 16384;
    if (dt == TBN_F32)
        hipLaunchKernelGGL(sign_pack_ballot_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                           static_cast<const float *>(x), xbits, M, in, groups, row_words);
    else
        hipLaunchKernelGGL(sign_pack_ballot_kernel<uint16_t>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                           static_cast<const uint16_t *>(x), xbits, M, in, groups, row_words);
    return check_launch("tbn_sign_pack");
}

tbn_status launch_linear_binact(const uint32_t *xbits, void *y, int dt, int64_t M, int64_t in, int64_t out,
                                const uint32_t *tile, int64_t p, int32_t k, const float *alpha, int32_t n_alpha,
                                uint32_t flags, hipStream_t stream) {
    const BinactArgs a{xbits, y, dt, M, in, out, tile, p, k, alpha, n_alpha, flags, stream};
    switch (choose_binact(a)) {
        case BinactKernel::Staged: return launch_binact_staged(a);
        case BinactKernel::MatrixCore: return launch_binact_mfma(a);
        case BinactKernel::Direct: return launch_binact_direct(a);
        case BinactKernel::Generic: break;
    }
    return launch_binact_generic(a);
}

const char *linear_binact_kernel_name(const uint32_t *xbits, const void *y, int dt, int64_t M, int64_t in, int64_t out, int64_t p,
                                      int32_t k, int32_t n_alpha, uint32_t flags) {
    switch (choose_binact(BinactArgs{xbits, const_cast<void *>(y), dt, M, in, out, nullptr, p, k, nullptr, n_alpha, flags, nullptr})) {
        case BinactKernel::Staged: return "staged";
        case BinactKernel::MatrixCore: return "matrix-core";
        case BinactKernel::Direct: return "direct";
        case BinactKernel::Generic: break;
    }
    return "generic";
}

bool linear_binact_counted(const uint32_t *xbits, const void *y, int dt, int64_t M, int64_t in, int64_t out, int64_t p, int32_t k,
                           int32_t n_alpha, uint32_t flags) {
    const BinactArgs a{xbits, const_cast<void *>(y), dt, M, in, out, nullptr, p, k, nullptr, n_alpha, flags, nullptr};
    return choose_binact(a) == BinactKernel::MatrixCore && binact_counted(a);
}

}  // namespace tbn
