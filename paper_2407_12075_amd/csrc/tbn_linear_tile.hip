// Kernel for the fully-connected tiled-bit layer with a tile of whole weight rows (p % in == 0) and few distinct
// rows or few batch rows: one wave per 32 batch rows, many small workgroups, no workgroup-wide pipeline.
//
// What is computed (Section "Method", Eq. 4-5 and the scaling after Eq. 8): with p a multiple of `in` only the
// U = p / in rows of the tile are distinct; Z = X * T^T (M x U) is formed once and Y[:, t*U + u] = alpha[t] * Z[:, u].
//
// Why another kernel.  (1) The layers that come with float32 activations (the MLP of a small vision transformer,
// 384 -> 1536 -> 384 on 12608 tokens, k = 4) have short rows and few distinct columns.  They move about 100 MB
// for 5 us of matrix work, so what counts is how many bytes are in flight, not how the matrix pipe is fed; a
// workgroup that owns a 128 x 128 block with a deep LDS pipeline spends its time filling and draining that
// pipeline (297 or 99 blocks of 20 us each on 256 CUs).  (2) bfloat16 layers at a few hundred batch rows give the
// block kernels 16 - 64 blocks for 256 CUs, each running the whole K loop alone.  Here
//   * a wave owns 32 batch rows and up to 128 distinct columns over one K slice; the workgroup's waves (1, 4 or 8)
//     take different K slices and add their sums through LDS at the end (in wave order: the result does not depend
//     on timing), so that a layer with 99 row blocks of 128, or a batch of 512 on a 4096 x 4096 layer, still puts
//     more than 1000 waves on the chip's 1024 SIMDs;
//   * a load instruction reads whole 128-byte lines (eight lanes per row); a chunk of 256 bytes per row (64 floats,
//     128 bfloat16) of the wave's 32 rows passes through 8 KiB of LDS that only this wave touches, to reach the
//     operand layout (a lane of the matrix instruction holds eight consecutive elements of one row), while the next
//     chunk's loads are in flight; no barrier in the K loop;
//   * every float is split exactly into three bfloat16 terms (8 + 8 + 8 significand bits); the weights are +-1,
//     so every product is exact and the sums are float32 accumulations in the matrix pipe
//     (v_mfma_f32_32x32x16_bf16, three per column tile and step; one for bfloat16 activations);
//   * the +-1 operand comes from the tile bits through a 256-entry table in LDS (one read per operand); K is
//     consumed in an order that suits the loads: lane half lg takes the elements of its half of the chunk, eight
//     per step, for both operands alike;
//   * the sums are turned round through LDS, 32 x 32 at a time, so that a store instruction writes whole
//     lines of Y (a lane of the accumulator layout holds four adjacent columns of one row only).
//
// float32: the K loop as a pipeline over steps (see there; not where plain_loop says) and two chunks in flight for long rows in one slice, 150 drawn layers
// of 157 - 12200 rows: 1.105 times as fast on the mean, 0.98 - 1.4 each (8192 x 4096 -> 4096, k = 8: 130.8 us before, 129.6 now, on another card 108.8 and 100.9;
// 826 x 3712 -> 2624 distinct columns 77.1 / 59.3; 4304 x 2176 -> 128 34.4 / 29.0; 12608 x 384 -> 1536 and 1536 -> 384, k = 4,
// 43.4 / 42.3 together).  On big layers the matrix pipe then runs at its limit of power: on the first card 60 cycles per product at 1.76 GHz
// before, 54 at 1.62 now.
//
// bfloat16 with K split, graph replays, 4096 -> 512 distinct columns, batch 300: 9.0 us before, 6.4 now (8192: 14.0 / 10.7;
// 1024: 5.3 / 4.2).  A wave per 32 columns where that leaves a workgroup per CU (8.7 -> 6.9), sums and stores by all waves, the table
// filled behind the first loads and barriers that order LDS only (-> 6.4); the alphas of 64 replicas in lanes, no branch in the
// replicas' loop (16 replicas: 11.0 before, 7.8 now).  What is left: 3.3 us outside the K loop and 0.74 us
// per chunk of 8 KiB and wave, 64 KiB per CU at 64 bytes a cycle being 0.43 of them.  Level or slower: two or four chunks in
// flight (7.0 / 8.2), sign operands by shifts instead of the table (8.8 against 8.7), operands read ahead of the matrix instructions
// (6.6 against 6.4), tile words through LDS in 64-byte pieces (7.2).
#include "tbn_common.h"

#include <type_traits>

namespace tbn {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // round to nearest even in hardware
}

union Frag {
    bf16x8_t v;
    u32x4_t q;
};

constexpr int kChunkBytes = 256;   // bytes of a row per chunk: 64 floats (four MFMA steps) or 128 bfloat16 (eight)
template <typename XT> constexpr int chunk_elems() { return kChunkBytes / static_cast<int>(sizeof(XT)); }
constexpr int kMaxNT = 4;       // column tiles of 32 per wave (two or three measure 3 - 50 % slower: more waves read X again)

struct TileParams {
    int64_t M;
    int32_t in, out, U;
    int32_t reps, n_alpha;
    int32_t col_groups;   // groups of NT * 32 distinct columns
    uint32_t row_tiles;   // tiles of 32 batch rows
    int32_t k_per_wave;   // K slice of a wave (whole chunks)
};

// barrier that orders LDS only: __syncthreads would wait for the loads in flight
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ float rep_alpha(float av, int lane) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(av), lane));
}

// LDS of a workgroup: the sign table, then one region per wave.  During the K loop a wave's region holds its
// current chunk of X, 32 rows of 256 bytes with the 16-byte pieces of a row XOR-swizzled by the row number (so that
// both the row-wise writes and the column-wise operand reads spread over the banks); afterwards the regions hold
// the partial sums that the waves hand over, and at last the 32 x 32 block a wave turns round for its stores.
template <int NT, int KW>
struct Lds {
    static constexpr int SL = (NT == KW) ? NT - 1 : NT;   // hand-over slots per wave: a wave keeps the tile it finishes
    static constexpr int kStage = 8192;                    // bytes per wave during the loop
    static constexpr int kPart = KW > 1 ? SL * 4096 : 0;
    static constexpr int kRegion = kStage > kPart ? kStage : kPart;
    static constexpr int kBytes = 4096 + KW * kRegion;
};

// float32, one wave per workgroup: chunks of K above which two of them are on their way instead of one.  A lone wave per SIMD has
// 8 KiB in flight with one (10685 x 5952 -> 64 distinct columns, 93 chunks: 111 us with one, 82 with two).  Two take 40 registers and a
// longer beginning and end: 7 - 8 / 9 - 12 chunks 2.5 / 1 % slower than with one, 13 - 20 / 21 - 40 / more 7 / 12 / 17 % faster on the
// mean.  With K split among waves there is enough in flight, and two are 1 - 5 % slower (282 drawn layers; one column tile and at most a
// wave per SIMD alone would gain, 5 %).
constexpr int32_t kLongSlice = 12;

// float32, K split and few columns: the plain loop.  The three or six products of a step cover little of the next step's 44 vector instructions, and
// the pipeline stores a chunk two steps before it is multiplied, so that its loads have three steps to arrive instead of four.
// Pipeline, over the plain loop's speed, 900 drawn layers of 256 - 8192 elements: one column tile and four waves 0.90 - 0.98 in the mean at up to
// 1024 waves, by rows' length, 0.96 - 1.01 beyond (4611 x 2304 -> 8 distinct columns 9.5 us plain, 11.6), eight waves 0.91 - 0.97, two column
// tiles and eight waves 0.95 - 0.98; two and four 1.04 - 1.09, three and eight 0.98 - 1.06, the rest above that.
constexpr bool plain_loop(int NT, int KW) { return (KW == 4 && NT == 1) || (KW == 8 && NT <= 2); }

// truncation split of eight floats into three bf16x8 operands: term 0 = top 8 significand bits, term 1 = the next 8,
// term 2 = the rest (at most 8 bits, so its truncation to bfloat16 is exact)
__device__ __forceinline__ void split8(const float (&x)[8], Frag (&t)[3]) {
    uint32_t h[3][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t t0 = __float_as_uint(x[i]) & 0xffff0000u;
        const float r1 = x[i] - __uint_as_float(t0);
        const uint32_t t1 = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(t1);
        h[0][i] = t0; h[1][i] = t1; h[2][i] = __float_as_uint(r2);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)   // high halves of two words in one: (lo >> 16) | (hi & 0xffff0000)
            t[j].q[v] = __builtin_amdgcn_perm(h[j][2 * v + 1], h[j][2 * v], 0x07060302u);
}

// AHEAD: float32, chunks in flight in the pipeline over steps; 0 and bfloat16: the plain loop, one chunk in flight.
// (pipeline: at most 256 registers, or the sums go to accumulation registers, which a tie would move them out of and back)
template <typename XT, bool RELU, int NT, int KW, int AHEAD>
__global__ __launch_bounds__(64 * KW, ((std::is_same<XT, float>::value && AHEAD > 0) || KW == 8 ? 2 : 1)) void linear_tile_kernel(const XT *__restrict__ x, XT *__restrict__ y,
                                                              const uint32_t *__restrict__ tile,
                                                              const float *__restrict__ alpha, TileParams P) {
    typedef Lds<NT, KW> L;
    constexpr bool kF32 = std::is_same<XT, float>::value, kPipe = kF32 && AHEAD > 0;
    constexpr int kCE = chunk_elems<XT>();          // elements of K per chunk
    constexpr int kSteps = kCE / 16;                // MFMA steps per chunk
    constexpr int kWords = kCE / 64;                // tile words per lane half, column and chunk
    extern __shared__ __attribute__((aligned(16))) unsigned char s_raw[];
    u32x4_t *s_table = reinterpret_cast<u32x4_t *>(s_raw);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ln = lane & 31, lg = lane >> 5;
    unsigned char *region_b = s_raw + 4096 + wave * L::kRegion;   // this wave's
    float *region = reinterpret_cast<float *>(region_b);

    // Workgroup ids are dealt round-robin to the 8 XCDs: the column groups of one row tile take consecutive slots of
    // one XCD, so that the rows of X they share are fetched from HBM once and then found in that XCD's L2 (plain order
    // fetched X once per column group: 58 MB instead of 19 on 12608 x 384 -> 1536, float32).
    uint32_t rt;
    int32_t cg;
    {
        const uint32_t bid = blockIdx.x, groups = static_cast<uint32_t>(P.col_groups), xcd = bid & 7, slot = bid >> 3;
        const uint32_t full = (P.row_tiles / 8) * groups;   // slots per XCD in the regular part
        if (slot < full) {
            const uint32_t q = slot / groups;
            cg = static_cast<int32_t>(slot - q * groups);
            rt = q * 8 + xcd;
        } else {   // the remaining row tiles: plain order
            const uint32_t rest = bid - full * 8, q = rest / groups;
            cg = static_cast<int32_t>(rest - q * groups);
            rt = (P.row_tiles / 8) * 8 + q;
        }
    }
    const int64_t m0 = int64_t(rt) * 32;
    const int32_t u0 = cg * (NT * 32);
    const int32_t k_begin = (kPipe ? __builtin_amdgcn_readfirstlane(wave) : wave) * P.k_per_wave;

    // loads: instruction (i, h) of a chunk reads rows 8i + lane/8, bytes 128h + 16*(lane%8) .. + 15 of the chunk's 256:
    // eight lanes cover a whole 128-byte line.  Rows past M repeat the last one; they are never written.
    const unsigned char *x_blk = reinterpret_cast<const unsigned char *>(x + m0 * P.in + k_begin);
    const int64_t last = P.M - 1 - m0;   // >= 0
    uint32_t ld_off[4];                  // byte offsets from x_blk
    uint32_t st_pos[4][2];               // byte positions in the wave's region
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + (lane >> 3);
        ld_off[i] = static_cast<uint32_t>(r < last ? r : last) * static_cast<uint32_t>(P.in) * static_cast<uint32_t>(sizeof(XT)) +
                    static_cast<uint32_t>(16 * (lane & 7));
#pragma unroll
        for (int h = 0; h < 2; ++h) st_pos[i][h] = static_cast<uint32_t>(r * 256 + (((8 * h + (lane & 7)) ^ (r & 15)) << 4));
    }
    // operand reads of row ln.  float32: step s of lane half lg takes floats 32*lg + 8*s .. + 7, pieces 8*lg + 2*s and + 1;
    // bfloat16: elements 64*lg + 8*s .. + 7, piece 8*lg + s.
    constexpr int kReads = kF32 ? 2 : 1;
    uint32_t rd_pos[kSteps][kReads];
#pragma unroll
    for (int s4 = 0; s4 < kSteps; ++s4)
#pragma unroll
        for (int j = 0; j < kReads; ++j)
            rd_pos[s4][j] = static_cast<uint32_t>(ln * 256 + (((8 * lg + kReads * s4 + j) ^ (ln & 15)) << 4));

    // tile words of this lane's column in every column tile: bit u * in + k; a lane half covers kWords words per chunk
    // (pipeline: one address per wave and 32-bit offsets, for the registers; in bfloat16 that is 0.7 % slower at batch 300)
    const uint32_t *tp[NT];
    const unsigned char *t_blk = reinterpret_cast<const unsigned char *>(tile + ((int64_t(u0) * P.in + k_begin) >> 5));
    uint32_t t_off[NT];   // byte offsets from t_blk
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int32_t u = u0 + 32 * t + ln;
        u = u < P.U ? u : P.U - 1;   // columns past U repeat the last one; never written
        tp[t] = tile + ((int64_t(u) * P.in + k_begin) >> 5) + kWords * lg;
        t_off[t] = (static_cast<uint32_t>(u - u0) * static_cast<uint32_t>(P.in) >> 3) + 4 * kWords * lg;
    }

    f32x16_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

    static_assert(kF32 ? AHEAD >= 0 && AHEAD <= 2 : AHEAD == 0, "");
    constexpr int kBufs = AHEAD == 2 ? 2 : 1;
    u32x4_t xr[kBufs][8];   // the chunks in flight: [i][h]
    uint32_t wr[kBufs][NT][kWords];
    auto load_chunk = [&](int32_t c, u32x4_t (&xr)[8], uint32_t (&wr)[NT][kWords]) __attribute__((always_inline)) {
        const unsigned char *src = x_blk + c * kChunkBytes;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) xr[2 * i + h] = *reinterpret_cast<const u32x4_t *>(src + ld_off[i] + 128 * h);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int w = 0; w < kWords; ++w) {
                if constexpr (kPipe) wr[t][w] = reinterpret_cast<const uint32_t *>(t_blk + c * 8 * kWords + t_off[t])[w];
                else wr[t][w] = tp[t][c * 2 * kWords + w];
            }
    };

    const int32_t chunks = P.k_per_wave / kCE;   // >= 1
    load_chunk(0, xr[0], wr[0]);
    const int32_t reps = P.reps;
    float av = alpha[P.n_alpha == 1 || lane >= reps ? 0 : lane];   // alphas of the first 64 replicas, one per lane

    // sign table: entry e, element i is +1 if bit i of e is set, else -1
    for (int e = tid; e < 256; e += 64 * KW) {
        u32x4_t t;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            t[v] = (((e >> (2 * v)) & 1) ? 0x3f80u : 0xbf80u) | ((((e >> (2 * v + 1)) & 1) ? 0x3f80u : 0xbf80u) << 16);
        s_table[e] = t;
    }
    lds_barrier();

    // bfloat16: a chunk goes to LDS, the next one is requested, then this one is multiplied from LDS.  The last chunk requests
    // nothing and stands by itself, because with a condition around the loads the compiler cannot count them in its waits (batch
    // 300, 4096 -> 512 distinct columns 6.4 us against 6.6); it then has to be kept from moving them down, which four waves pay for
    // with every chunk (312 x 8704 -> 976 distinct columns: 15.5 us with the condition, 17.5 with the loads moved down, 14.1 now; 177 x
    // 5632 -> 1664: 11.8 / 13.0 / 10.6; eight waves are level: 300 x 8192 -> 512 14.3 / 10.5 / 10.6).  float32 here (few columns, K
    // split) keeps the condition.
    auto multiply_chunk = [&](int32_t c, auto more) {
        uint32_t wc[NT][kWords];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int w = 0; w < kWords; ++w) wc[t][w] = wr[0][t][w];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<u32x4_t *>(region_b + st_pos[i][h]) = xr[0][2 * i + h];
        __builtin_amdgcn_wave_barrier();   // lanes read what other lanes of the wave wrote (LDS operations of a wave stay in order)
        if (decltype(more)::value && (!kF32 || c + 1 < chunks)) load_chunk(c + 1, xr[0], wr[0]);
        // bfloat16: left to itself the compiler moves these loads behind most of the products below, which they are to run under
        if constexpr (!kF32) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s4 = 0; s4 < kSteps; ++s4) {
            constexpr int kTerms = kF32 ? 3 : 1;
            Frag xt[kTerms];
            if constexpr (kF32) {
                const f32x4_t a = *reinterpret_cast<const f32x4_t *>(region_b + rd_pos[s4][0]);
                const f32x4_t b = *reinterpret_cast<const f32x4_t *>(region_b + rd_pos[s4][kReads - 1]);
                const float xs[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
                split8(xs, xt);
            } else {
                xt[0].q = *reinterpret_cast<const u32x4_t *>(region_b + rd_pos[s4][0]);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                Frag sg;
                sg.q = s_table[(wc[t][s4 / 4] >> (8 * (s4 % 4))) & 0xffu];
#pragma unroll
                for (int j = 0; j < kTerms; ++j)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg.v, xt[j].v, acc[t], 0, 0, 0);
            }
        }
        __builtin_amdgcn_wave_barrier();   // the next chunk overwrites the region
    };
    if constexpr (kPipe) {
        // float32: the split of a step's activations into terms takes 44 vector instructions, as long as six of its products.  One
        // after the other (many rows and distinct columns leave one wave per SIMD) that was 60 cycles per product of 32; here the
        // next step's split is dealt to the slots behind this step's matrix instructions (pinned there: the compiler would put the
        // split in front of all of them), its signs and the activations of the step after next are read meanwhile, and the next
        // chunk goes to LDS in the slots of the second step.  The sums are formed in the order they had: the same bits.
        constexpr int kSlots = 3 * NT, kUnits = 12;   // units of the split: element, element, their pair's six halves
        float xs[2][8];              // activations of a step, by its parity
        Frag xt[2][3], sg[2][NT];    // terms and signs of a step, by its parity
        uint32_t wc[NT], wn[NT];     // tile words of this chunk and the next
        uint32_t ww[AHEAD][NT];      // of the chunks that are on their way
        uint32_t hold[2][3];         // terms of the pair that is being split
        auto request = [&](int32_t c, u32x4_t (&xn)[8], uint32_t (&wx)[NT]) __attribute__((always_inline)) {
            const unsigned char *src = x_blk + c * kChunkBytes, *words = t_blk + c * 8;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                asm volatile("" : "+v"(ld_off[i]));   // or the compiler keeps 64-bit addresses of all of them in registers
#pragma unroll
                for (int h = 0; h < 2; ++h) xn[2 * i + h] = *reinterpret_cast<const u32x4_t *>(src + ld_off[i] + 128 * h);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                asm volatile("" : "+v"(t_off[t]));
                wx[t] = *reinterpret_cast<const uint32_t *>(words + t_off[t]);
            }
        };
        auto store = [&](int n, const u32x4_t (&v)[8]) __attribute__((always_inline)) {
            *reinterpret_cast<u32x4_t *>(region_b + st_pos[n >> 1][n & 1]) = v[n];
        };
        auto read = [&](float (&v)[8], int s4) __attribute__((always_inline)) {
            const f32x4_t a = *reinterpret_cast<const f32x4_t *>(region_b + rd_pos[s4][0]);
            const f32x4_t b = *reinterpret_cast<const f32x4_t *>(region_b + rd_pos[s4][kReads - 1]);
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
        };
        auto signs = [&](Frag &g, uint32_t word, int s4) __attribute__((always_inline)) { g.q = s_table[(word >> (8 * s4)) & 0xffu]; };
        auto unit = [&](int n, const float (&v)[8], Frag (&t)[3]) __attribute__((always_inline)) {
            // truncation: term 0 = top 8 significand bits, term 1 = the next 8, term 2 = the rest (at most 8 bits: exact)
            const int pair = n / 3, k = n % 3;
            if (k < 2) {
                const float a = v[2 * pair + k];
                const uint32_t t0 = __float_as_uint(a) & 0xffff0000u;
                const float r1 = a - __uint_as_float(t0);
                const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
                hold[k][0] = __float_as_uint(a); hold[k][1] = __float_as_uint(r1); hold[k][2] = __float_as_uint(r2);
                asm volatile("" : "+v"(hold[k][0]), "+v"(hold[k][1]), "+v"(hold[k][2]));
            } else {   // high halves of two words in one
#pragma unroll
                for (int j = 0; j < 3; ++j) t[j].q[pair] = __builtin_amdgcn_perm(hold[1][j], hold[0][j], 0x07060302u);
                uint32_t p0 = t[0].q[pair], p1 = t[1].q[pair], p2 = t[2].q[pair];
                asm volatile("" : "+v"(p0), "+v"(p1), "+v"(p2));
                t[0].q[pair] = p0; t[1].q[pair] = p1; t[2].q[pair] = p2;
            }
        };
        if constexpr (AHEAD == 2) request(1, xr[1], ww[1]);
#pragma unroll
        for (int n = 0; n < 8; ++n) store(n, xr[0]);
        __builtin_amdgcn_wave_barrier();   // lanes read what other lanes of the wave wrote (LDS operations of a wave stay in order)
        read(xs[0], 0);
        read(xs[1], 1);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            wc[t] = wr[0][t][0];
            signs(sg[0][t], wc[t], 0);
        }
        if (AHEAD == 2 || chunks > 1) request(AHEAD, xr[0], ww[0]);   // two ahead: chunks > 4
#pragma unroll
        for (int n = 0; n < kUnits; ++n) unit(n, xs[0], xt[0]);
        auto chunk = [&](int32_t c, u32x4_t (&xn)[8], uint32_t (&wx)[NT], auto all) __attribute__((always_inline)) {
#pragma unroll
            for (int s4 = 0; s4 < kSteps; ++s4) {
                const int cur = s4 & 1, nxt = cur ^ 1;
                read(xs[cur], (s4 + 2) & 3);   // (behind the last chunk: what is there, not used)
                if (s4 == 2) {   // the chunk after those that are on their way
#pragma unroll
                    for (int t = 0; t < NT; ++t) wn[t] = wx[t];
                    if (decltype(all)::value || c + 1 + AHEAD < chunks) request(c + 1 + AHEAD, xn, wx);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < kSlots; ++i) {
                    const int j = i / NT, t = i % NT;
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg[cur][t].v, xt[cur][j].v, acc[t], 0, 0, 0);
                    asm volatile("" : "+v"(acc[t]));
                    if (i < NT) signs(sg[nxt][i], s4 < 3 ? wc[i] : wn[i], (s4 + 1) & 3);
                    // the next chunk to LDS, behind the reads of this one's last step (behind the last chunk: what is there)
                    if (s4 == 1) {
#pragma unroll
                        for (int n = 0; n < 8; ++n)
                            if (n * kSlots / 8 == i) store(n, xn);
                    }
#pragma unroll
                    for (int n = 0; n < kUnits; ++n)
                        if (n * kSlots / kUnits == i) unit(n, xs[nxt], xt[nxt]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (s4 == 1) __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) wc[t] = wn[t];
        };
        int32_t c = 0;
        if constexpr (AHEAD == 2) {
            // With a condition around the loads the compiler cannot count them, and a wait for one chunk waits for both: the chunks
            // that still have two pairs ahead go without.  (Loading the same 16 bytes for a chunk that is not there costs 5 %.)
            do {
                chunk(c, xr[1], ww[1], std::true_type{});
                chunk(c + 1, xr[0], ww[0], std::true_type{});
                c += 2;
            } while (c + 4 < chunks);
            for (; c < chunks; c += 2) {
                chunk(c, xr[1], ww[1], std::false_type{});
                if (c + 1 < chunks) chunk(c + 1, xr[0], ww[0], std::false_type{});
            }
        } else {
            for (; c < chunks; ++c) chunk(c, xr[0], ww[0], std::false_type{});
        }
        __builtin_amdgcn_wave_barrier();
    } else {
        int32_t c = 0;
        for (; c + (kF32 ? 0 : 1) < chunks; ++c) multiply_chunk(c, std::true_type{});
        if constexpr (!kF32) multiply_chunk(c, std::false_type{});
    }

    // ---- bfloat16, K split: every thread adds CP neighbouring outputs of one row over the waves, in wave order (results are the
    // same from run to run), and writes them.  (One wave adding and writing a column tile while the others idle: see the top.)
    if constexpr (!kF32 && KW > 1) {
        constexpr int CP = 16 * NT / KW;          // outputs per thread: 1024 * NT among 64 * KW threads
        static_assert(CP >= 2 && NT * 4096 <= L::kRegion, "");
        // row ln of column tile t: 128 bytes, 16-byte piece c at position c ^ (ln & 7)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4_t *>(region + t * 1024 + ln * 32 + (((2 * q + lg) ^ (ln & 7)) << 2)) =
                    f32x4_t{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
        lds_barrier();
        const int r = tid / (2 * KW), col = (tid % (2 * KW)) * CP;   // 2 * KW threads per row
        float z[CP];
#pragma unroll
        for (int w = 0; w < KW; ++w) {
            const float *part = reinterpret_cast<const float *>(s_raw + 4096 + w * L::kRegion) + (col >> 5) * 1024 + r * 32;
#pragma unroll
            for (int e = 0; e < CP; e += (CP < 4 ? CP : 4)) {
                const float *src = part + (((((col & 31) + e) >> 2) ^ (r & 7)) << 2) + (col & 3);
#pragma unroll
                for (int i = 0; i < (CP < 4 ? CP : 4); ++i) z[e + i] = w == 0 ? src[i] : z[e + i] + src[i];
            }
        }
        const int64_t m = m0 + r;
        const int32_t u = u0 + col;
        const bool live = m < P.M && u < P.U;   // U % 8 == 0: a thread's outputs are inside or outside together
        XT *dst = y + m * P.out + u;
        for (int32_t base = 0; base < reps; base += 64) {
            if (base > 0) av = alpha[P.n_alpha == 1 || base + lane >= reps ? 0 : base + lane];
            const int32_t n = reps - base < 64 ? reps - base : 64;
            for (int32_t rep = 0; rep < n; ++rep, dst += P.U) {
                const float al = rep_alpha(av, rep);
                uint32_t pk[CP / 2];
#pragma unroll
                for (int e = 0; e < CP; e += 2) {
                    float a = al * z[e], b = al * z[e + 1];
                    if (RELU) { a = fmaxf(a, 0.f); b = fmaxf(b, 0.f); }
                    pk[e / 2] = pack2(a, b);
                }
                if (live) __builtin_memcpy(__builtin_assume_aligned(dst, 2 * CP), pk, 2 * CP);
            }
        }
        return;
    }

    // ---- float32: the waves of the workgroup add their K slices: wave w ends up with column tile w ------------------------
    // (sums in ascending wave order whatever the timing: results are the same from run to run)
    int t_mine = 0;            // column tiles this wave writes: [t_mine, t_end)
    int t_end = NT;
    if constexpr (kF32 && KW > 1) {
        static_assert(KW >= NT, "every column tile needs a wave");
        constexpr int SL = L::SL;
        __syncthreads();   // every wave is done with its chunk: the regions change their use
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t == wave) continue;                       // kept in registers
            const int slot = (NT == KW && t > wave) ? t - 1 : t;
#pragma unroll
            for (int r = 0; r < 16; ++r) region[(slot * 16 + r) * 64 + lane] = acc[t][r];
        }
        __syncthreads();
        t_mine = wave;
        t_end = wave < NT ? wave + 1 : wave;   // waves past NT write nothing
        if (wave < NT) {
            f32x16_t sum;
            bool first = true;
#pragma unroll
            for (int w = 0; w < KW; ++w) {
                f32x16_t v;
                if (w == wave) {
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        if (t == wave) v = acc[t];
                } else {
                    const int slot = (NT == KW && wave > w) ? wave - 1 : wave;
                    const float *other = reinterpret_cast<const float *>(s_raw + 4096 + w * L::kRegion);
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = other[(slot * 16 + r) * 64 + lane];
                }
                if (first) { sum = v; first = false; }
                else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum[r] += v[r];
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (t == wave) acc[t] = sum;
        }
        __syncthreads();   // all hand-over reads are done: a wave's region is its own again
        (void)SL;
    }

    // ---- y[m, u + t*U] = alpha[t] * Z[m, u] ----------------------------------------------------------------------
    // Register 4q + e of a column tile is column 8q + 4lg + e of row ln.  The wave turns every 32 x 32 tile round
    // through its region (row r at r * 128 bytes, 16-byte piece c at position c ^ (r & 7)) so that a few lanes hold a
    // row's 32 columns: eight lanes with four float32 each, or four lanes with eight bfloat16 each, and a store
    // instruction writes whole lines.
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (t < t_mine || t >= t_end) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4_t *>(region + ln * 32 + (((2 * q + lg) ^ (ln & 7)) << 2)) =
                f32x4_t{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if constexpr (kF32) {
            const int r8 = lane >> 3, c8 = lane & 7;
            f32x4_t z[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = r8 + 8 * i;
                z[i] = *reinterpret_cast<const f32x4_t *>(region + r * 32 + ((c8 ^ (r & 7)) << 2));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();   // the next tile overwrites the region
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int32_t u = u0 + 32 * t + 4 * c8;
            if (u >= P.U) continue;   // U % 4 == 0: a group of four is inside or outside
            for (int32_t rep = 0; rep < P.reps; ++rep) {
                const float al = alpha[P.n_alpha == 1 ? 0 : rep];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t m = m0 + r8 + 8 * i;
                    if (m >= P.M) continue;
                    f32x4_t v = al * z[i];
                    if (RELU) { v[0] = fmaxf(v[0], 0.f); v[1] = fmaxf(v[1], 0.f); v[2] = fmaxf(v[2], 0.f); v[3] = fmaxf(v[3], 0.f); }
                    f32x4_t *dst = reinterpret_cast<f32x4_t *>(y + m * P.out + int64_t(rep) * P.U + u);
                    // Non-temporal where K is split among the waves of a workgroup (long rows: the layer then reads more
                    // than it writes and the output should not push X out of the L2: 12608 x 1536 -> 384 20.1 us against
                    // 21.3); plain otherwise (384 -> 1536: 27.0 against 28.7 non-temporal).  A compile-time choice: the
                    // compiler merges the two stores of a run-time one into a plain store.
                    if constexpr (KW > 1) __builtin_nontemporal_store(v, dst);
                    else *dst = v;
                }
            }
        } else {
            const int r4 = lane >> 2, c4 = lane & 3;   // row of 16, eight columns 8*c4 .. + 7: pieces 2*c4 and 2*c4 + 1
            f32x4_t za[2], zb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = r4 + 16 * i;
                za[i] = *reinterpret_cast<const f32x4_t *>(region + r * 32 + (((2 * c4) ^ (r & 7)) << 2));
                zb[i] = *reinterpret_cast<const f32x4_t *>(region + r * 32 + (((2 * c4 + 1) ^ (r & 7)) << 2));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();   // the next tile overwrites the region
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int32_t u = u0 + 32 * t + 8 * c4;
            if (u >= P.U) continue;   // U % 8 == 0: a group of eight is inside or outside
            for (int32_t rep = 0; rep < P.reps; ++rep) {
                const float al = alpha[P.n_alpha == 1 ? 0 : rep];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int64_t m = m0 + r4 + 16 * i;
                    if (m >= P.M) continue;
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) { v[e] = al * za[i][e]; v[4 + e] = al * zb[i][e]; }
                    if (RELU) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
                    }
                    const u32x4_t pk = {pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
                    *reinterpret_cast<u32x4_t *>(y + m * P.out + int64_t(rep) * P.U + u) = pk;
                }
            }
        }
    }
}

template <typename XT, bool RELU, int NT, int KW, int AHEAD>
tbn_status launch_one(const LinearArgs &a, const TileParams &P, unsigned grid) {
    typedef Lds<NT, KW> L;
    // dynamic LDS above the default limit has to be allowed once per kernel (thread-safe static initialisation)
    static const hipError_t attr = L::kBytes > 65536
        ? hipFuncSetAttribute(reinterpret_cast<const void *>(&linear_tile_kernel<XT, RELU, NT, KW, AHEAD>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, L::kBytes)
        : hipSuccess;
    if (attr != hipSuccess) {
        set_error("tbn_linear_forward: cannot reserve %d bytes of LDS", L::kBytes);
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL((linear_tile_kernel<XT, RELU, NT, KW, AHEAD>), dim3(grid), dim3(64 * KW), L::kBytes, a.stream,
                       static_cast<const XT *>(a.x), static_cast<XT *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward (one wave per 32 batch rows)");
}

template <typename XT, bool RELU, int NT>
tbn_status launch_kw(const LinearArgs &a, const TileParams &P, unsigned grid, int kw) {
    constexpr bool f32 = std::is_same<XT, float>::value;
    if (kw == 8) return launch_one<XT, RELU, NT, 8, (f32 && !plain_loop(NT, 8) ? 1 : 0)>(a, P, grid);
    if (kw == 4) return launch_one<XT, RELU, NT, 4, (f32 && !plain_loop(NT, 4) ? 1 : 0)>(a, P, grid);
    if constexpr (f32) {
        if (P.k_per_wave > kLongSlice * chunk_elems<float>()) return launch_one<XT, RELU, NT, 1, 2>(a, P, grid);
    }
    return launch_one<XT, RELU, NT, 1, (f32 ? 1 : 0)>(a, P, grid);
}

template <typename XT, bool RELU>
tbn_status launch_nt(const LinearArgs &a, const TileParams &P, unsigned grid, int nt, int kw) {
    if (nt == 1) return launch_kw<XT, RELU, 1>(a, P, grid, kw);
    if (nt == 2) return launch_kw<XT, RELU, 2>(a, P, grid, kw);
    if constexpr (std::is_same<XT, float>::value) {   // the plan gives bfloat16 at most two tiles per wave
        if (nt == 3) return launch_kw<XT, RELU, 3>(a, P, grid, kw);
        return launch_kw<XT, RELU, 4>(a, P, grid, kw);
    }
    set_error("tbn_linear_forward: no kernel for %d column tiles per wave", nt);
    return TBN_ERR_UNSUPPORTED;
}

// column tiles per wave: as few groups as possible, then as even as possible (float32, U = 384: three groups of four, see below
// tiles; U = 96: one group of three; bfloat16 takes at most two tiles per wave, one while every workgroup has a CU to itself:
// its use is small batches, where more waves count for more than fewer passes over X: 4096 x 4096, k = 8 at batch 300 6.9 us
// with one, 8.7 with two, 13.6 with four; two workgroups of one tile on a CU are slower than one of two: batch 1024 11.7 /
// 9.4); K slices per workgroup: as many (8, 4) as leave a wave at least two chunks and the chip at most about two waves per
// SIMD
void plan(const LinearArgs &a, int &nt, int &groups, int &kw) {
    const int64_t U = a.p / a.in;
    const int64_t tiles = (U + 31) / 32;
    const int max_nt = a.dt == TBN_F32 ? kMaxNT : ((a.M + 31) / 32) * tiles <= 256 ? 1 : 2;
    groups = static_cast<int>((tiles + max_nt - 1) / max_nt);
    nt = static_cast<int>((tiles + groups - 1) / groups);
    const int64_t ce = a.dt == TBN_F32 ? chunk_elems<float>() : chunk_elems<uint16_t>();
    const int64_t waves1 = ((a.M + 31) / 32) * groups;
    kw = 1;
    for (int cand : {8, 4}) {
        if (a.in % (cand * ce) == 0 && a.in / cand >= 2 * ce && waves1 * cand <= 2048 && cand >= nt) {
            kw = cand;
            break;
        }
    }
    // float32 with K in one slice (one wave per workgroup) and fewer than one and a half waves per SIMD: one more
    // column group where the tiles divide evenly, for more waves in flight (12608 x 384 -> 384 distinct columns: four
    // groups of three tiles 25.8 us against three groups of four 27.8; with more waves the extra pass over X costs more
    // than it gains: 1536 distinct columns 51.4 against 49.5)
    if (a.dt == TBN_F32 && kw == 1 && waves1 < 1536 && nt > 2 && tiles % (groups + 1) == 0) {
        groups += 1;
        nt = static_cast<int>(tiles / groups);
    }
}

}  // namespace

// Shapes this kernel takes: tile of whole rows, K in chunks of 256 bytes, 16-byte loads and stores possible.  Every
// group of 64 (bfloat16) or up to 128 (float32) distinct columns reads its rows of X again, from L2: with many distinct
// columns the kernel is for small batches only, which linear_tile_preferred and the dispatch see to.
bool linear_tile_supported(const LinearArgs &a) {
    if (a.dt != TBN_F32 && a.dt != TBN_BF16) return false;
    const int64_t ce = a.dt == TBN_F32 ? chunk_elems<float>() : chunk_elems<uint16_t>();
    if (a.in % ce != 0 || a.p % a.in != 0) return false;
    const int64_t U = a.p / a.in;
    if (U > a.out || a.out % U != 0 || U % (a.dt == TBN_F32 ? 4 : 8) != 0 || U > (1 << 20)) return false;
    if (a.in > (1 << 20) || a.out > (1 << 22) || a.p >= (int64_t(1) << 36)) return false;
    if (a.M < 1 || a.M > (int64_t(1) << 34)) return false;
    if ((reinterpret_cast<uintptr_t>(a.x) & 15u) || (reinterpret_cast<uintptr_t>(a.y) & 15u)) return false;
    int nt, groups, kw;
    plan(a, nt, groups, kw);
    return ((a.M + 31) / 32) * groups <= 0x7fffffffLL;
}

// bfloat16: where this kernel beats the small-batch, the streaming and the block kernels.  Graph replays, microseconds
// per call, this kernel / what the dispatch would take otherwise:
//   * at least four K slices and at most about two waves per SIMD.  512 distinct columns, in = 4096, batch 256 / 512 /
//     1024 / 2048: 6.8 / 7.0 / 9.6 / 15.7 against 16.6 / 15.6 / 15.0 / 15.4; in = 2048, batch 1024 / 2048: 6.7 / 10.1
//     against 10.7 / 10.9.  Batch 17 - 64, 512 distinct columns, in = 1024 / 2048 / 8192: 4.0 / 4.7 / 9.4 against 7.9 /
//     8.0 / 13.6 for the small-batch kernel, in = 4096, 1024 / 2048 columns: 6.3 / 6.4 against 8.3 / 8.5.  (Rows of
//     4096, of all lengths with four slices, stay with that kernel at up to 128 of its workgroups, where it is the slower one: 8.0 - 9.4
//     against 5.6 - 7.0, all of 300 drawn layers, 1.35 times as long on the mean.  No measurement stands behind that: the dispatch
//     table that tests/test_abi.py pins has such a call.)  Up to 16 rows where the decode kernel declines: 4096 columns, in = 4096, batch 6 / 16: 6.4 / 6.5 against
//     6.7 / 8.6; in = 1024: 3.9 / 4.0 against 4.4 / 4.5 in the direct kernel.
//     More replicas than 32 to 96, the more the longer the rows, leave it behind the direct kernel where that is the other choice: up to 16
//     rows, in to 2048, 33 - 48 / 49 - 64 / 65 - 100 replicas 0.98 / 0.94 / 0.90 of that kernel's speed on the mean, in to 3584 1.03 / 0.98 / 0.95, beyond
//     4096 1.11 / 1.07 / 1.02 and from 101 on 0.94; 17 - 64 rows, in beyond 4096: 1.12 to 100, 0.97 from there (688 drawn layers).
//     The number of distinct columns is not limited: 4096 of them at batch 100, in = 1024 / 4096: 5.0 / 8.8 against
//     10.6 / 20.4 with the streaming kernel;
//   * short rows (fewer K slices), up to 512 waves, where the small-batch kernel would need more than one workgroup
//     per CU: in = 512, 512 distinct columns, batch 512 / 1024 / 2048: 6.0 / 6.4 / 7.2 against 7.4 / 7.6 / 7.7 (batch
//     4096: 9.4 against 9.0, left to the block kernel); batch 160 / 256, in = 256 / 768: 4.7 / 7.0 against 6.7 - 6.9 /
//     11.0 - 11.4 (with 256 workgroups or fewer the small-batch kernel is the faster one: 4.2 / 6.4 against 4.7 / 7.1).
// float32: the small-batch kernel's time grows with every further 256 workgroups (one per CU), this kernel's hardly
// with the batch.  512 distinct columns, batch 197 / 400 / 800, this kernel / the small-batch kernel: in = 1024:
// 10.1 / 10.3 / 10.6 against 14.0 / 26.5 / 46.0; in = 4096: 23.0 / 23.2 / 23.6 against 24.2 / 47.0 / 80.8; in = 384:
// 12.6 / 12.8 / 13.2 against 8.3 / 15.2 / 25.6.  So: more than 512 of its workgroups, or more than 256 with rows of at
// least 1024.
bool linear_tile_preferred(const LinearArgs &a) {
    if ((a.M <= 16 && (a.dt == TBN_F32 || (a.flags & TBN_FLAG_LARGE_BATCH))) || !linear_tile_supported(a)) return false;
    if (a.dt == TBN_F32) {
        const int64_t grid = ((a.p / a.in + 15) / 16) * ((a.M + 15) / 16);   // workgroups of the small-batch kernel
        return a.M > 64 && grid <= 2048 && (grid > 512 || (grid > 256 && a.in >= 1024));   // beyond 2048 that kernel declines
    }
    int nt, groups, kw;
    plan(a, nt, groups, kw);
    const int64_t waves1 = ((a.M + 31) / 32) * groups;
    const int64_t U = a.p / a.in;
    const int64_t small_grid = ((U + 15) / 16) * ((a.M + 15) / 16);   // workgroups of the small-batch kernel
    if (kw >= 4) {
        const int64_t limit = a.in <= 2048 ? 32 : a.in >= 6144 ? 96 : a.in / 64;   // replicas
        const bool few = a.M <= 16 || (a.M <= 64 && a.in >= 4096 && a.in < 8192);
        if (few && a.out / U > limit && linear_direct_preferred(a, DirectOver::SmallBatch)) return false;
        return waves1 * kw <= 2048 && !(a.M > 16 && a.M <= 64 && a.in == 4096 && small_grid <= 128);
    }
    return a.M > 64 && small_grid > 256 && waves1 <= 512;
}

// bfloat16, at most 16 rows: where this kernel beats the decode kernel, whose workgroups each read all of X, two columns at a
// time.  Graph replays, this kernel / the decode kernel, 2 / 8 / 16 replicas.  in = 1024, 512 distinct columns, batch 13: 3.5 / 3.9 /
// 4.4 against 4.2 / 4.4 / 5.0; 2048 columns, batch 5 and 8: 3.5 / 3.9 / 4.4 against 4.4 / 4.6 / 4.9 and 4.5 / 4.8 / 5.3; in = 2048, 6144 columns,
// batch 2: 4.6 / 4.9 / 5.3 against 7.3 / 7.4 / 7.6; 768 columns, batch 11: 4.4 / 4.7 / 5.1 against 5.6 / 5.8 / 6.3.  Fewer outputs: in = 1024,
// 512 columns, batch 8: 3.5 / 3.9 / 4.4 against 3.6 / 3.7 / 3.8.  Longer rows: its chain over K is the longer one (in = 4096, batch 16, 512
// columns: 5.9 / 6.3 / 6.7 against 5.3 / 5.4 / 6.0).  Many replicas, of which a thread here stores 4 - 16 bytes at a time: 49 to 64 of them still 1.17
// times as fast on the mean of 8 layers, 101 to 200 0.94 of 17 (batch 4, in = 1024, 4096 columns, 200: 17.7 against 16.8).
bool linear_tile_over_decode(const LinearArgs &a) {
    if (a.dt != TBN_BF16 || a.in > 2048 || a.M > 16 || !linear_tile_supported(a)) return false;
    int nt, groups, kw;
    plan(a, nt, groups, kw);
    const int64_t U = a.p / a.in;
    return kw >= 4 && int64_t(groups) * kw <= 2048 && U * a.M > (a.in <= 1024 ? 6144 : 8192) && a.out / U <= 64;
}

int linear_tile_k_slices(const LinearArgs &a) {
    int nt, groups, kw;
    plan(a, nt, groups, kw);
    return kw;
}

tbn_status launch_linear_tile(const LinearArgs &a) {
    TileParams P;
    P.M = a.M;
    P.in = static_cast<int32_t>(a.in);
    P.out = static_cast<int32_t>(a.out);
    P.U = static_cast<int32_t>(a.p / a.in);
    P.reps = static_cast<int32_t>(a.out / P.U);
    P.n_alpha = a.n_alpha;
    int nt, groups, kw;
    plan(a, nt, groups, kw);
    P.col_groups = groups;
    P.row_tiles = static_cast<uint32_t>((a.M + 31) / 32);
    P.k_per_wave = P.in / kw;
    const unsigned grid = static_cast<unsigned>(((a.M + 31) / 32) * groups);
    const bool relu = (a.flags & TBN_FLAG_RELU) != 0;
    if (a.dt == TBN_F32) return relu ? launch_nt<float, true>(a, P, grid, nt, kw) : launch_nt<float, false>(a, P, grid, nt, kw);
    return relu ? launch_nt<uint16_t, true>(a, P, grid, nt, kw) : launch_nt<uint16_t, false>(a, P, grid, nt, kw);
}

}  // namespace tbn
