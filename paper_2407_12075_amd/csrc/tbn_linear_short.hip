// Fully-connected tiled-bit layer in bfloat16 with short rows and many distinct columns (the product of a column-tiled layer
// after its fold, first layers, the projections of small models): the activations of a row block stay in LDS.
//
// What is computed (Section "Method", Eq. 4-5 and the scaling after Eq. 8): with p a multiple of `in` the weight is
// the U = p / in rows of the tile stacked k times, copy t scaled by alpha[t]; Z = X * T^T is formed once and
// Y[:, t*U + u] = alpha[t] * Z[:, u].
//
// What bounds it: with K = 512 a 128 x 128 block of Z is four rounds of the block kernel, whose pipeline fill, hand-over of
// partial sums and barriers then take as long as its multiplications.  Here a workgroup loads the whole rows of its 128 (or
// 64) batch rows into LDS once and its eight waves walk the columns without ever meeting again: a wave multiplies all rows
// with 64 columns at a time over all of K, so there are no partial sums to hand over, and per eight matrix instructions a
// wave reads four operands from LDS and expands two from the tile bits in registers (18 vector instructions).  The two waves of a
// SIMD start at the same barrier and do equal passes, so they store at about the same time: only what they drift apart
// lets one wave's stores run under the other's multiplications, and nothing runs under those of the last pass.
//   * Rows in LDS are padded with zeros to whole chunks of 64 elements and by 16 bytes, which spreads the operand reads of 16
//     rows over all banks.
//   * In a chunk of 64 elements of K lane half lg takes elements 32 lg + 8 s .. + 7 in step s, so that its tile bits of a
//     column are one 32-bit window (any bit position: two words and a funnel shift).  The words come four at a time, two chunks
//     per load: a load of the words touches a line per column whatever its width, 64 cycles of the CU's load path, and word
//     by word the 16 loads of a wave's first chunks took 3 us and those of a pass as long as its multiplications.
//   * The +-1 operand is the row operand of v_mfma_f32_32x32x16_bf16 with its lanes numbered so that a lane ends up with eight
//     adjacent columns of one row of Y; two register sets trade halves (v_permlane16_swap) so that a store instruction
//     writes 64 bytes of 16 rows, without another pass through LDS.
// 8192 x 512 -> 4096, k = 1 (the product of a column-tiled layer of 4096 x 4096, k = 8): 48 - 51 us in the block kernel; here, with
// word loads / now, 37 / 34 in calls through the wrapper and 41.5 / 39.3 in graph replays, which leave no gaps and run at a lower clock: 3 us to start
// and load the rows, 25 of multiplications (a pass keeps the matrix pipe 94 % busy, at 1.5 - 1.7 GHz: the power limit), the rest stores
// that nothing runs under.  8192 x 128 / 256 / 320 / 576 -> 4096, graph replays: 20.5 / 24.5 / 26.7 / 41.0 before, 17.6 / 22.2 / 24.2 / 37.5 now;
// 2000 x 384 -> 4096 16.7 / 14.1; with two replicas of 4096 columns of 256 elements
// 34.6 / 34.3 (36.3 with all waves starting together).
// Tried: 64 rows per workgroup (55 us: twice the vector instructions per matrix instruction), non-temporal stores and wave
// priorities (no difference).
#include "tbn_common.h"

#include <type_traits>

namespace tbn {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_t u32x4_a4_t __attribute__((aligned(4)));   // at any word of the tile
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512, kWaves = 8;
constexpr int TM = 4, kRows = 32 * TM;   // rows per workgroup, all of them taken by every wave
constexpr int kCols = 64;         // columns per wave and pass
constexpr int kLdsMax = 160 * 1024;
// Two replicas, rows of at most this many chunks: wave after wave starts (80 drawn layers, together / one after another: 64 - 256 elements 1.05
// times as fast on the mean, to 384 0.98 - 1.16, 544 and 576 0.94 - 0.99; 8192 x 256 -> 8192 36.3 us / 34.3, 10531 x 96 -> 8192 41.3 / 33.9)
constexpr int kStaggerChunks = 6;

union Frag {
    bf16x8_t v;
    u32x4_t q;
};

struct ShortParams {
    int64_t M;
    int32_t in, out, U, reps, n_alpha;
    uint32_t last_word;    // of the tile
    int32_t chunks;        // of 64 elements of K
    uint32_t row_blocks, splits;   // workgroups: row blocks x column ranges
    int32_t groups;        // groups of 64 columns
    int32_t groups_per_split;
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // round to nearest even in hardware
}

// The +-1 operand from byte S of an inverted window (bit set: -1): the byte is replicated, each half shifted so that bits
// 2v and 2v + 1 land on the two sign positions, and the pattern of 1.0 merged in.
template <int S>
__device__ __forceinline__ void expand(uint32_t win, uint32_t signs, uint32_t ones, Frag &b) {
    const uint32_t rep = __builtin_amdgcn_perm(win, win, 0x01010101u * S);
    const u16x2_t r2 = __builtin_bit_cast(u16x2_t, rep);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const u16x2_t sh = {static_cast<uint16_t>(15 - 2 * v), static_cast<uint16_t>(14 - 2 * v)};
        b.q[v] = (__builtin_bit_cast(uint32_t, static_cast<u16x2_t>(r2 << sh)) & signs) | ones;
    }
}

template <bool RELU>
__global__ __launch_bounds__(kThreads, 2) void linear_short_kernel(const uint16_t *__restrict__ x, uint16_t *__restrict__ y,
                                                                   const uint32_t *__restrict__ tile,
                                                                   const float *__restrict__ alpha, ShortParams P) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_x[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, lg = lane >> 5;

    // workgroups that share rows take consecutive slots of one XCD (ids are dealt round-robin to the eight of them)
    uint32_t rb, sp;
    {
        const uint32_t bid = blockIdx.x, xcd = bid & 7, slot = bid >> 3, full = (P.row_blocks / 8) * P.splits;
        if (slot < full) {
            const uint32_t q = slot / P.splits;
            sp = slot - q * P.splits;
            rb = q * 8 + xcd;
        } else {
            const uint32_t rest = bid - full * 8, q = rest / P.splits;
            sp = rest - q * P.splits;
            rb = (P.row_blocks / 8) * 8 + q;
        }
    }
    const int64_t m0 = int64_t(rb) * (kRows);
    const int rows = static_cast<int>(P.M - m0 < kRows ? P.M - m0 : kRows);
    const uint32_t stride = static_cast<uint32_t>(P.chunks) * 128u + 16u;   // bytes per row in LDS

    const int32_t g_end = static_cast<int32_t>(sp + 1) * P.groups_per_split < P.groups ? static_cast<int32_t>(sp + 1) * P.groups_per_split : P.groups;
    // tile words of chunk c for a lane's two columns: operand lane l of column tile tn supplies column
    // 16*(l/8) + 8*((l/4)%2) + 4*tn + l%4 of the 64
    struct Cols { uint32_t word[2], sh[2]; };
    auto columns = [&](int32_t g) {
        Cols k;
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) {
            int32_t u = g * kCols + 16 * (ln >> 3) + 8 * ((ln >> 2) & 1) + 4 * tn + (ln & 3);
            u = u < P.U ? u : P.U - 1;   // columns past U repeat the last one; never written
            const uint64_t bit = uint64_t(u) * static_cast<uint32_t>(P.in) + static_cast<uint32_t>(32 * lg);
            k.word[tn] = static_cast<uint32_t>(bit >> 5);
            k.sh[tn] = static_cast<uint32_t>(bit & 31);
        }
        return k;
    };
    // the four words from 2 c on: chunks c and c + 1 (even c).  Past the row's end any value will do, past the tile's nothing may
    // be read: a lane there takes the last four words and moves them down.
    auto load_words = [&](const Cols &k, int32_t c, u32x4_t (&w)[2]) {
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) {
            const uint32_t i = k.word[tn] + static_cast<uint32_t>(2 * c), end = P.last_word - 3u;
            w[tn] = *reinterpret_cast<const u32x4_a4_t *>(tile + (i < end ? i : end));
        }
        if (__any(k.word[0] + static_cast<uint32_t>(2 * c) > P.last_word - 3u || k.word[1] + static_cast<uint32_t>(2 * c) > P.last_word - 3u)) {
#pragma unroll
            for (int tn = 0; tn < 2; ++tn) {
                const uint32_t i = k.word[tn] + static_cast<uint32_t>(2 * c), end = P.last_word - 3u, past = i > end ? i - end : 0u;
                if (past & 1u) w[tn] = u32x4_t{w[tn][1], w[tn][2], w[tn][3], w[tn][3]};
                if (past & 2u) w[tn] = u32x4_t{w[tn][2], w[tn][3], w[tn][3], w[tn][3]};
            }
        }
    };
    // inverted windows of chunks 0 .. kAhead - 1 of the next pass, formed before the stores of this one are issued: a load
    // behind the stores can only be waited for together with them (one counter, in issue order)
    constexpr int kAhead = 4;
    uint32_t first[kAhead][2];
    u32x4_t ring[kAhead / 2][2];   // [pair of chunks][column]
    Cols cols;
    auto form = [&](const Cols &k, int d, uint32_t (&win)[2]) {   // chunk d of the four in the ring
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) win[tn] = ~__funnelshift_r(ring[d >> 1][tn][2 * (d & 1)], ring[d >> 1][tn][2 * (d & 1) + 1], k.sh[tn]);
    };
    // (the first pass's words are requested in front of the rows: behind the barrier they keep the waves waiting)
    int32_t g = static_cast<int32_t>(sp) * P.groups_per_split + wave;
    cols = columns(g);
#pragma unroll
    for (int h = 0; h < kAhead / 2; ++h) load_words(cols, 2 * h, ring[h]);

    // ---- the rows: eight threads per 128 bytes of a row; rows past M repeat the last one (never written) --------------
    {
        const unsigned char *src = reinterpret_cast<const unsigned char *>(x + m0 * P.in);
        constexpr int kPasses = kRows / (kThreads / 8);   // rows per thread
        constexpr int kDepth = 8;                           // chunks of 128 bytes requested together
        uint32_t from[kPasses], to[kPasses];
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            const int r = tid / 8 + i * (kThreads / 8);
            from[i] = static_cast<uint32_t>(r < rows ? r : rows - 1) * static_cast<uint32_t>(P.in) * 2u;
            to[i] = static_cast<uint32_t>(r) * stride + static_cast<uint32_t>(tid & 7) * 16u;
        }
        const int32_t last = P.in * 2 - 16;   // in % 8 == 0: a piece is inside the row or outside
        for (int32_t c0 = 0; c0 < P.chunks; c0 += kDepth) {
            u32x4_t v[kDepth][kPasses];
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                if (c0 + d >= P.chunks) break;
                const int32_t at = (c0 + d) * 128 + (tid & 7) * 16;
#pragma unroll
                for (int i = 0; i < kPasses; ++i)
                    v[d][i] = *reinterpret_cast<const u32x4_t *>(src + (from[i] + static_cast<uint32_t>(at < last ? at : last)));
            }
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                if (c0 + d >= P.chunks) break;
                const int32_t at = (c0 + d) * 128 + (tid & 7) * 16;
#pragma unroll
                for (int i = 0; i < kPasses; ++i)
                    *reinterpret_cast<u32x4_t *>(s_x + (to[i] + static_cast<uint32_t>(c0 + d) * 128u)) = at <= last ? v[d][i] : u32x4_t{0u, 0u, 0u, 0u};
            }
        }
    }
    __syncthreads();

    // Two replicas: the waves' stores are as long as their multiplications, and only those that start apart run under another
    // wave's.  (The word by word loads of tile bits had spread the waves by the time they queued.)
    if (P.reps > 1 && P.chunks <= kStaggerChunks)
        for (int i = 0; i < wave; ++i) __builtin_amdgcn_s_sleep(16);   // 1024 cycles each

    uint32_t signs = 0x80008000u, ones = 0x3f803f80u;
    asm volatile("" : "+s"(signs), "+s"(ones));   // scalar registers: an and-or takes no constants of this size
    const unsigned char *a_ptr = s_x + static_cast<uint32_t>(ln) * stride + static_cast<uint32_t>(lg) * 64u;
#pragma unroll
    for (int d = 0; d < kAhead; ++d) form(cols, d, first[d]);
    for (; g < g_end; g += kWaves) {
        f32x16_t acc[TM][2];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < 2; ++tn)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[tm][tn][e] = 0.f;
        // The operands of a step are requested (activations) and expanded (signs) during the step before.
        Frag av[2][TM], bv[2][2];
        auto read = [&](const unsigned char *src, Frag (&a)[TM]) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) a[tm].q = *reinterpret_cast<const u32x4_t *>(src + static_cast<uint32_t>(32 * tm) * stride);
        };
        read(a_ptr, av[0]);
        expand<0>(first[0][0], signs, ones, bv[0][0]);
        expand<0>(first[0][1], signs, ones, bv[0][1]);
        const unsigned char *a_chunk = a_ptr;
        auto multiply = [&](const uint32_t (&win)[2], const uint32_t (&win_next)[2]) {
            auto step = [&](auto s_c) {
                constexpr int S = decltype(s_c)::value, cur = S & 1, nx = cur ^ 1;
                read(a_chunk + (S < 3 ? 16 * (S + 1) : 128), av[nx]);   // behind the row's last chunk: its padding, never used
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int tn = 0; tn < 2; ++tn) expand<(S + 1) & 3>(S < 3 ? win[tn] : win_next[tn], signs, ones, bv[nx][tn]);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < 2; ++tn)
                        acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[cur][tn].v, av[cur][tm].v, acc[tm][tn], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 2 * TM; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);               // a matrix instruction
                    __builtin_amdgcn_sched_group_barrier(0x2, 3, 0); // vector instructions in its shadow
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
            a_chunk += 128;
        };
        uint32_t win[2] = {first[0][0], first[0][1]}, next[2];
        auto chunk = [&](int32_t c, auto d_c, const uint32_t (&ready)[2], bool formed) {
            constexpr int D = decltype(d_c)::value;
            if (formed) { next[0] = ready[0]; next[1] = ready[1]; }
            else form(cols, (D + 1) % kAhead, next);
            if (D % 2 == 0 && c + kAhead < P.chunks) load_words(cols, c + kAhead, ring[D / 2]);   // both chunks of the pair have been formed
            multiply(win, next);
            win[0] = next[0]; win[1] = next[1];
        };
        using std::integral_constant;
        chunk(0, integral_constant<int, 0>{}, first[1], true);
        if (P.chunks > 1) chunk(1, integral_constant<int, 1>{}, first[2], true);
        if (P.chunks > 2) chunk(2, integral_constant<int, 2>{}, first[3], true);
        if (P.chunks > 3) chunk(3, integral_constant<int, 3>{}, first[3], false);
        for (int32_t c = kAhead; c < P.chunks; c += kAhead) {
            chunk(c, integral_constant<int, 0>{}, first[0], false);
            if (c + 1 < P.chunks) chunk(c + 1, integral_constant<int, 1>{}, first[0], false);
            if (c + 2 < P.chunks) chunk(c + 2, integral_constant<int, 2>{}, first[0], false);
            if (c + 3 < P.chunks) chunk(c + 3, integral_constant<int, 3>{}, first[0], false);
        }
        if (g + kWaves < g_end) {
            cols = columns(g + kWaves);
#pragma unroll
            for (int h = 0; h < kAhead / 2; ++h) load_words(cols, 2 * h, ring[h]);
#pragma unroll
            for (int d = 0; d < kAhead; ++d) {
                form(cols, d, first[d]);
                asm volatile("" : "+v"(first[d][0]), "+v"(first[d][1]) : : "memory");   // not moved behind the stores
            }
        }
        // Registers 4q .. 4q + 3 of tiles 0 and 1: columns 16q + 8 lg .. + 7 of row 32 tm + ln.  The lanes of rows 16 .. 31
        // of q = 2h trade with those of rows 0 .. 15 of q = 2h + 1: one register set then holds 32 columns of rows
        // 0 .. 15 (lanes 0 .. 15: columns 0 - 7, 32 .. 47: 8 - 15, 16 .. 31: 16 - 23, 48 .. 63: 24 - 31), the other of rows 16 .. 31.
        const int row16 = ln & 15, col = 16 * (ln >> 4) + 8 * lg;
        for (int32_t rep = 0; rep < P.reps; ++rep) {
            const float al = alpha[P.n_alpha == 1 ? 0 : rep];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    u32x4_t pk[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        float v[8];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v[e] = al * acc[tm][0][4 * (2 * h + j) + e];
                            v[4 + e] = al * acc[tm][1][4 * (2 * h + j) + e];
                        }
                        if (RELU) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
                        }
                        pk[j] = u32x4_t{pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const auto r = __builtin_amdgcn_permlane16_swap(pk[0][e], pk[1][e], false, false);
                        pk[0][e] = r[0];
                        pk[1][e] = r[1];
                    }
                    if (g * kCols + 32 * h + col >= P.U) continue;   // U % 8 == 0
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int r = 32 * tm + 16 * j + row16;
                        if (r < rows)
                            *reinterpret_cast<u32x4_t *>(y + (m0 + r) * P.out + (int64_t(rep) * P.U + g * kCols + 32 * h + col)) = pk[j];
                    }
                }
            }
        }
    }
}

template <bool RELU>
tbn_status launch_one(const LinearArgs &a, const ShortParams &P, int lds) {
    static const hipError_t attr =   // thread-safe static initialisation: set once per process
        hipFuncSetAttribute(reinterpret_cast<const void *>(&linear_short_kernel<RELU>), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
    if (attr != hipSuccess) {
        set_error("tbn_linear_forward: cannot reserve %d bytes of LDS", lds);
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL(linear_short_kernel<RELU>, dim3(P.row_blocks * P.splits), dim3(kThreads), lds, a.stream,
                       static_cast<const uint16_t *>(a.x), static_cast<uint16_t *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward (short rows)");
}

// (the read behind the last chunk of a row, whose data is never used: lane half 1 of the last row reads up to 80 bytes past
// its chunks, 64 past the 16 of its padding)
int64_t lds_bytes(int64_t in) { return kRows * (((in + 63) / 64) * 128 + 16) + 128; }

// Column ranges per row block: a workgroup costs about 4 us to start and load its rows and 10.6 us per pass over K = 512
// (two waves per SIMD, 64 columns each), its stores 1.2 us per pass and replica; one workgroup per CU at a time.  (Drawn with tile words
// one by one.  A fit to 200 layers since gives 4.8 us, 8.6 us and, stores, 4.0 us; three of them would get other ranges by it.)
int64_t column_splits(int64_t row_blocks, int64_t passes, int64_t in, int64_t reps) {
    const double pass = 0.0207 * static_cast<double>(in) + 1.2 * static_cast<double>(reps);
    int64_t best = 1;
    double best_cost = 0;
    for (int64_t s = 1; s <= passes && s <= 256; ++s) {
        const double cost = static_cast<double>((row_blocks * s + 255) / 256) * (4.0 + static_cast<double>((passes + s - 1) / s) * pass);
        if (s == 1 || cost < best_cost) { best = s; best_cost = cost; }
    }
    return best;
}

}  // namespace

// Shapes this kernel takes: whole rows of the tile, 16-byte loads and stores, 128 rows in LDS.
bool linear_short_supported(const LinearArgs &a) {
    if (a.dt != TBN_BF16 || a.in % 8 != 0 || a.p % a.in != 0 || a.in > 576 || a.p < 128 || lds_bytes(a.in) > kLdsMax) return false;
    const int64_t U = a.p / a.in;
    if (U > a.out || a.out % U != 0 || U % 8 != 0 || a.out > (1 << 22) || a.p >= (int64_t(1) << 36)) return false;
    if ((reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.y)) & 15u) return false;
    // (a launch has fewer than 2^32 threads along x)
    return a.M >= 1 && (a.M + kRows - 1) / kRows * ((U + kCols - 1) / kCols) < (int64_t(1) << 32) / kThreads;
}

// Where this kernel beats the block and the general kernel (graph replays, microseconds per call, the other kernel / this
// one with tile words one by one; 200 drawn layers since: the other kernel takes 1.37 times as long on the mean with one replica and 1.19 with two,
// and three layers 0.89 - 0.97 times): the share of the chip's wave passes (256 CUs, eight waves each) that have columns to work on must not be small.
// One replica: 8192 x 128 / 256 / 320 / 512 / 576 -> 4096 columns 30 / 20, 37 / 24, 41 / 27, 50 / 40 - 45, 56 / 43;
// 12638 x 72 -> 824 15.6 / 9.7; 6853 x 448 -> 2616 (share 0.54) 29.4 / 28.2; 2049 x 512 -> 3912 (0.51) 17.4 / 18.4.  Two
// replicas: 12000 x 200 -> 1400 29.2 / 24.7; 7815 x 576 -> 2584 (0.62) 44 / 40; 13011 x 504 -> 1344 (0.52) 35.6 / 37.0.  With
// more the stores bind either kernel: four, 8192 x 128 / 256 / 512 -> 4096 53.4 / 52.4, 62 / 53, 66 / 64; eight, 8192 x 256 ->
// 4096 109 / 128.  The line is drawn below four, where the one shape that gains 15 % stays with the general kernel.
bool linear_short_preferred(const LinearArgs &a) {
    if ((a.flags & ~uint32_t(TBN_FLAG_RELU)) || !linear_short_supported(a)) return false;   // flags that steer to another kernel
    const int64_t U = a.p / a.in, reps = a.out / U;
    if (reps > 2) return false;
    const int64_t row_blocks = (a.M + kRows - 1) / kRows, groups = (U + kCols - 1) / kCols, passes = (groups + kWaves - 1) / kWaves;
    const int64_t splits = column_splits(row_blocks, passes, a.in, reps);
    const int64_t slots = (row_blocks * splits + 255) / 256 * 256 * ((passes + splits - 1) / splits) * kWaves;
    return row_blocks * groups * 10 >= slots * (reps == 1 && a.in < 512 ? 5 : 6);
}

tbn_status launch_linear_short(const LinearArgs &a) {
    ShortParams P;
    P.M = a.M;
    P.in = static_cast<int32_t>(a.in);
    P.out = static_cast<int32_t>(a.out);
    P.U = static_cast<int32_t>(a.p / a.in);
    P.reps = P.out / P.U;
    P.n_alpha = a.n_alpha;
    P.last_word = static_cast<uint32_t>((a.p + 31) / 32 - 1);
    P.chunks = (P.in + 63) / 64;
    P.row_blocks = static_cast<uint32_t>((a.M + kRows - 1) / kRows);
    P.groups = (P.U + kCols - 1) / kCols;
    const int64_t passes = (P.groups + kWaves - 1) / kWaves, splits = column_splits(P.row_blocks, passes, a.in, P.reps);
    P.groups_per_split = static_cast<int32_t>((passes + splits - 1) / splits) * kWaves;
    P.splits = static_cast<uint32_t>((P.groups + P.groups_per_split - 1) / P.groups_per_split);
    const int lds = static_cast<int>(lds_bytes(a.in));
    return (a.flags & TBN_FLAG_RELU) ? launch_one<true>(a, P, lds) : launch_one<false>(a, P, lds);
}

}  // namespace tbn
