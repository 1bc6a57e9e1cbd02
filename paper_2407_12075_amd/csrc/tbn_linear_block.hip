// Matrix-core kernel for the fully-connected tiled-bit layer with bfloat16 activations, one 128 x 128 block of Z per
// workgroup or several one after the other, with separate load waves; for tiles that hold whole weight rows
// (p % in == 0) and, in the windowed form (WIN), rows of any length in multiples of 8 and tiles that end inside rows.
//
// What is computed (Section "Method", Eq. 4-5 and the scaling after Eq. 8): with p a multiple of `in` the
// (out x in) weight is the U = p / in rows of the tile stacked k times, copy t scaled by alpha[t].  So
// Z = X * T^T (M x U, T the +-1 rows of the tile) is formed once and Y[:, t*U + u] = alpha[t] * Z[:, u]
// ("only one of the tile computations needs to be executed", Section "CNN Architectures", applied to
// matrix columns).
//
// Layout on gfx950 and why (every point is a measurement on the chip):
//   * A wave issues one instruction every four cycles at best and a v_mfma_f32_32x32x16_bf16 occupies the
//     matrix pipe for 32, so what bounds the main loop is the number of other instructions the MFMA waves
//     have to issue -- and above all the global -> LDS wave-loads, which block the wave's whole instruction
//     stream whenever the CU's load path is busy.  The workgroup therefore has eight waves: four MFMA waves
//     (one per SIMD) that only read LDS and multiply, and four load waves that issue every wave-load of the
//     main loop and otherwise sleep at the round's barrier (with the MFMA waves loading for themselves, one
//     wave-load in an MFMA slot each, the same kernel measured 46.1 us against 42.6 on 8192 x 4096 -> 4096).
//   * MFMA wave (g, h) owns 128 rows x 64 columns of the block over the K stages congruent to g (mod 2):
//     4 x 2 MFMA tiles, the +-1 rows as the row operand, six LDS operand reads per eight MFMAs.  The two
//     K groups add their partial sums through LDS at the end.
//   * Activations go global -> LDS directly (16 bytes per lane, four ring slots of one stage for both K
//     groups, XOR-swizzled so that operand reads are free of bank conflicts).  The chunk of the packed tile
//     that the block's 128 tile rows need for two rounds travels the same way in coalesced 16-byte pieces;
//     an MFMA wave then takes the 64 window bits of its two columns with one LDS instruction per round.
//     Tile bits are never fetched lane by lane from global memory.
//   * A byte of tile bits becomes the +-1 bf16 MFMA operand through a 256-entry table in LDS.
//   * The replicated, alpha-scaled output is most of the bytes this kernel moves (eight ninths at k = 8).  It
//     is written with 16-byte stores that cover whole 128-byte lines (the sums are turned round through LDS
//     first).  With one block per workgroup the MFMA waves write it themselves with plain stores: all workgroups
//     store at the same time and the last-level cache takes the burst (8192 x 4096 -> 4096, k = 8: 37.7 us
//     against 42.4 with non-temporal stores).
//   * Grids of more blocks than CUs (PERSIST): one workgroup per CU walks blocks, and the stores of a block run
//     under the K loop of the next one.  Of waves 4 .. 7 two load (two quarters of a round each) and two store: the
//     MFMA waves leave the sums of a finished block in LDS, a store wave takes two 64 x 64 quarters into 128
//     registers and writes them, scaled, a few (replica, quarter, 32 rows) units per round, with non-temporal
//     stores (next to a running loop, plain stores push the activations that the other column blocks of the same
//     rows still need out of the XCD's L2: 16384 x 4096 -> 4096, k = 8: 81 us against 65).  Stores and loads have
//     waves of their own because the vector-memory counter counts both, in issue order: a wave that did both
//     waited for its stores whenever it waited for a round of loads (8192 x 4096 -> 16384, k = 8: block loops of
//     28.7 us against 24.7).  The first two rounds of the next block are issued inside the last rounds of the
//     current one, into the two ring slots behind its last round, which are free by then; between two loops lie 2.2 us (the K groups add their
//     sums, the store waves take them over).  8192 x 4096 -> 16384, k = 2 / 4 / 8 / 16: 410 / 211 / 117 / 86 us
//     against 410 / 216 / 127 / 97 with the stores after each loop; 32768 x 4096 -> 4096, k = 8: 137 against 152.
//     What stays exposed is the stores of a workgroup's last block.
//   * Rows of any length in multiples of 8 and tiles that end inside rows (WIN = true): the tile bits of a chunk begin at any
//     position, so the words that hold them come to LDS as they are and are shifted into the layout above by waves that do
//     not multiply; the zeros behind a row's end come from a piece of zeros in memory; alphas may differ from column to
//     column.  The MFMA waves' loop is the same.  8192 x 3000 -> 3072, k = 9 (1024 distinct columns, two blocks per CU): 55 us
//     against 61 in the general kernel, whose MFMA waves load and fetch windows for themselves; what is left to the aligned
//     form (8192 x 3072: 47) is the loads of rows that start inside lines, and 7 % for fetching the words.
//   * Split K (SPLIT = true, for grids that would leave most CUs idle and callers that bring a workspace):
//     the K loop of a block is dealt to S workgroups; each writes its float32 partial sums of the 128 x 128
//     block to the workspace, [split][M][U], and a second kernel adds the S partial sums of every output in
//     ascending split order (no atomics: the result is the same bit for bit from run to run), scales by
//     alpha and writes the replicas.
#include "tbn_common.h"

#include <type_traits>

namespace tbn {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

union Frag {
    bf16x8_t v;
    u32x4_t q;
};

constexpr int kBM = 128, kBN = 128;      // block of Z per workgroup
constexpr int kBK = 64;                  // K elements per K group and round
constexpr int kNB = 4;                   // ring slots
constexpr int kSlotBytes = 2 * kBM * kBK * 2;   // [K group][128 rows][128 bytes]
constexpr int kTileSlots = 3;            // ring of tile chunks, one chunk = two rounds
constexpr int kTileSlotBytes = 4096;     // [16-byte piece (= round parity)][128 columns][16 bytes]
constexpr int kBias = 3 * 1024;          // keeps the lane offsets of the wave-loads non-negative

// LDS map.  The sign table sits at address 0 so that a table read needs no base.
constexpr int kTableOff = 0;             // 256 entries of 16 bytes
constexpr int kRingOff = 4096;
constexpr int kTileOff = kRingOff + kNB * kSlotBytes;
constexpr int kLdsBytes = kTileOff + kTileSlots * kTileSlotBytes;
// WIN: the words of three chunks as they come from memory, in the layout of the tile chunks; the alphas.  Chunk c (rounds 2c and
// 2c + 1) has raw slot c % 3 and is read by put_tile of chunks c and c - 1 (the fifth words), pieces that another load wave
// brought among them.  So between the last read of a slot and the next fetch into it lies a barrier:
//   one block per workgroup   put_tile(0) (slots 0, 1)           | "round 0 readable"        | fetch of chunk 3 (slot 0)
//                             put_tile(2) (slots 1, 2)           | the same and round 0's    | fetch of chunk 4 (slot 1)
//                             chunk c, behind round 2c - 3's     | round 2c - 2's            | fetch of chunk c + 3
//   PERSIST                   chunk 0, behind the last round's   | the block's first         | fetch of chunk 3
//                             chunk 1, behind the block's first  | round 0's                 | fetch of chunk 4
//                             chunk c, behind round 2c - 3's     | round 2c - 2's            | fetch of chunk c + 3
//                             last chunk                         | round n - 4's             | the next block's fetches of chunks 0 and 1
// (tests/test_window_schedule.py walks the statements of these waves and checks this for every access.)
constexpr int kRawSlots = 3;
constexpr int kRawOff = kLdsBytes;
constexpr int kAlphaOff = kRawOff + kRawSlots * kTileSlotBytes;
constexpr int kMaxWinAlphas = (160 * 1024 - kAlphaOff) / 4;
constexpr int kXchgOff = kRingOff;       // after the main loop the ring holds the partial sums handed over (4 x 16 KiB)
static_assert(kLdsBytes <= 160 * 1024, "LDS budget of a gfx950 workgroup");

struct BlockParams {
    int64_t M;
    int32_t in, out, U;
    int32_t reps;         // out / U = k replicas of every distinct column
    int32_t n_alpha;
    int32_t tiles_n;      // column blocks of U
    uint32_t tiles_m;
    int32_t n_rounds;     // rounds of 128 elements of K per workgroup (even): in / 128, or in / 128 / splits
    int32_t splits;       // workgroups that share the K loop of a block (1: none)
    uint32_t vrows;       // tiles_m * splits: (row block, split) pairs
    float *partial;       // split K: [split][M][U] float32 partial sums
    // WIN
    int32_t p;            // tile bits
    int32_t alpha_step;   // tile copies per replica: alpha of column u + t*U is that of column u, t * alpha_step on
};

// s_waitcnt immediate that waits for the vector-memory counter only (gfx9 encoding: vmcnt in bits
// 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// All LDS traffic of this kernel is written as inline assembly: the compiler would otherwise make every
// LDS access wait for all global -> LDS loads in flight.  The waits are explicit; a register that a read
// fills is handed to the compiler only through tie() after the wait that covers it
// (paper_2407_12075_amd/asm_check.py verifies on the generated assembly that nothing touches such a
// register earlier).
template <int OFF>
__device__ __forceinline__ void lds_read16(u32x4_t &dst, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
// two 8-byte reads 512 bytes apart: registers 0-1 from addr, 2-3 from addr + 512
__device__ __forceinline__ void lds_read2x8(u32x4_t &dst, uint32_t addr) {
    asm volatile("ds_read2_b64 %0, %1 offset0:0 offset1:64" : "=v"(dst) : "v"(addr));
}
template <int OFF>
__device__ __forceinline__ void lds_write16(uint32_t addr, const u32x4_t &v) {
    asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(addr), "v"(v), "n"(OFF) : "memory");
}
template <int N>
__device__ __forceinline__ void lds_wait() {
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void tie(u32x4_t &r) { asm volatile("" : "+v"(r)); }

// wave-load J of a group of four that share an LDS base: the immediate offset is added to the LDS
// address and to the global address alike (the per-lane offset takes it back out, see a_off)
template <int J>
__device__ __forceinline__ void wave_load(const unsigned char *src, uint32_t off, unsigned char *dst) {
    __builtin_amdgcn_global_load_lds(src + off, dst, 16, J * 1024, 0);
}

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // round to nearest even in hardware
}

template <int V> using Int = std::integral_constant<int, V>;

__device__ __forceinline__ void lds_read4(uint32_t &dst, uint32_t addr) {
    asm volatile("ds_read_b32 %0, %1" : "=v"(dst) : "v"(addr));
}
__device__ __forceinline__ void tie(uint32_t &r) { asm volatile("" : "+v"(r)); }

// x / p and x % p for 0 <= x < 2^43 and 1 <= p < 2^31
__device__ __forceinline__ uint32_t divide(uint64_t x, uint32_t p, uint32_t &rest) {
    uint64_t q = static_cast<uint64_t>(static_cast<double>(x) / static_cast<double>(p));
    int64_t r = static_cast<int64_t>(x - q * p);
    if (r < 0) { --q; r += p; }
    if (r >= static_cast<int64_t>(p)) { ++q; r -= p; }
    rest = static_cast<uint32_t>(r);
    return static_cast<uint32_t>(q);
}
__device__ __align__(16) const uint32_t kZeroPiece[4] = {0u, 0u, 0u, 0u};   // what lies behind the end of a row

// 16-byte store to a scalar base plus a 32-bit lane offset (NT: non-temporal)
template <bool NT>
__device__ __forceinline__ void global_store16(unsigned char *base, uint32_t off, const u32x4_t &v) {
    if constexpr (NT) asm volatile("global_store_dwordx4 %0, %1, %2 nt" : : "v"(off), "v"(v), "s"(base) : "memory");
    else asm volatile("global_store_dwordx4 %0, %1, %2" : : "v"(off), "v"(v), "s"(base) : "memory");
}

// Workgroups that share rows of X are given consecutive slots on one XCD (workgroup ids are dealt
// round-robin to the 8 XCDs), so the later column blocks find X in that XCD's L2.
// With split K the unit that shares data is a (row block, split) pair: vrow counts those.
__device__ __forceinline__ void block_coords(const BlockParams &P, uint32_t bid, uint32_t &vrow, uint32_t &tile_n) {
    const uint32_t xcd = bid & 7, slot = bid >> 3;
    const uint32_t tiles_n = static_cast<uint32_t>(P.tiles_n);
    const uint32_t per_xcd_full = (P.vrows / 8) * tiles_n;   // slots per XCD in the regular part
    if (slot < per_xcd_full) {
        const uint32_t q = slot / tiles_n;
        tile_n = slot - q * tiles_n;
        vrow = q * 8 + xcd;
    } else {  // remaining row blocks: plain order
        const uint32_t rest = bid - per_xcd_full * 8;
        const uint32_t q = rest / tiles_n;
        tile_n = rest - q * tiles_n;
        vrow = (P.vrows / 8) * 8 + q;
    }
}

// RELU: fused max(0, .) of Algorithm 1.  SPLIT: the workgroup takes one of P.splits equal parts of K and writes
// float32 partial sums to P.partial instead of Y.  512 threads: waves 0 .. 3 multiply, waves 4 .. 7 load (and, PERSIST, store).
// PERSIST (grids of more blocks than CUs; at least four rounds): the workgroup walks blocks blockIdx.x, + gridDim.x, ...;
// waves 4 and 5 load, waves 6 and 7 write the replicas of the block before.  The
// first rounds of the next block start in the ring slot behind the current block's last round, and the hand-over uses
// the slots of the last two rounds.
// WIN (any row length in multiples of 8, tile starts anywhere): the loads of the last rounds take zeros for what lies behind
// a row's end; the load waves bring the words that hold a chunk's tile bits to one of three raw slots in LDS as they are
// (fetch_tile), three chunks ahead of the chunk that is multiplied, and put_tile shifts them into the chunk's slot, so that the
// MFMA waves see aligned chunks.  put_tile is the load waves' with one block per workgroup and the store waves' under PERSIST;
// behind the barrier of round 2c - 3 for chunk c, so that round 2c - 2's publishes it, and which barrier frees a raw slot
// stands at kRawSlots.  Alphas come from LDS, column by column.
template <bool RELU, bool SPLIT, bool PERSIST, bool WIN>
__global__ __launch_bounds__(512, 1) void linear_block_bf16_kernel(const uint16_t *__restrict__ x,
                                                                                     uint16_t *__restrict__ y,
                                                                                     const uint32_t *__restrict__ tile,
                                                                                     const float *__restrict__ alpha,
                                                                                     BlockParams P) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = wave & 3;     // MFMA wave: which quarter of the block it owns
    const int grp = li >> 1;     // K group
    const int wn = li & 1;       // column half
    const int ln = lane & 31;    // operand lane inside a 32 x 32 tile
    const int lg = lane >> 5;    // K half of the operand registers

    static_assert(!(SPLIT && PERSIST), "a split grid never has more workgroups than CUs");
    // Ring slot of round g of a block: (g + ph) % 4.  ph is 0 with one block per workgroup; a persistent workgroup
    // starts a block in the slot after the last one of the block before, ph' = (ph + rounds) % 4 (0 or 2: rounds come
    // in pairs).  Hand-over area: with one block per workgroup the start of the ring; PERSIST: the slots of a block's
    // last two rounds, which are the two slots behind those that take the first two rounds of the next block.
    auto xchg_base = [&](int32_t phase) -> uint32_t {
        return PERSIST ? static_cast<uint32_t>(kRingOff + ((P.n_rounds - 2 + phase) & 3) * kSlotBytes) : static_cast<uint32_t>(kXchgOff);
    };
    // Waves 4 .. 7.  One block per workgroup: four load waves, each issues a quarter of a round's loads (quarter q:
    // K group q / 2, row-slot half q % 2; WIN: and puts its quarter of the tile chunks in place).  PERSIST: waves 4 and 5 load
    // (two quarters each: K group = wave - 4), waves 6 and 7 write the replicas of the block before (the quarters of MFMA
    // waves 2*(wave - 6) and + 1; WIN: and put two quarters of the tile chunks in place).
    constexpr int NQ = PERSIST ? 2 : 1;   // quarters per load wave (and per store wave)
    const int first_q = PERSIST ? 2 * (wave & 1) : (wave & 3);
    const int32_t n_rounds = P.n_rounds;
    const uint32_t n_blocks = P.vrows * static_cast<uint32_t>(P.tiles_n);
    uint32_t bid = blockIdx.x;

    // ---- the loads of a round, a quarter at a time ------------------------------------------------------
    // Activations: wave-load j of quarter q fills 1 KiB of K group q / 2's 16 KiB: piece 8*(q % 2) + j, row slot
    // sr = 8*piece + lane/8, chunk slot lane%8.  Row-slot block sr/32 holds row block (sr/32 + 2*grp) % 4 of the
    // block (so that each K group ends with the sums it keeps in its first accumulators), chunk slot s of row
    // slot sr holds 16-byte chunk s ^ ((sr >> 1) & 7) of the round's 128 bytes of that row.  Rows past M repeat
    // row M - 1.  Tile chunk (two rounds: 256 bits = two 16-byte pieces per tile row): lane i of quarter q fills
    // slot S = 64*q + i of the chunk's 256: piece S / 128, LDS row S % 128; LDS row 64*h + 32*tn + l holds the
    // tile row that operand lane l of column half h supplies for MFMA tile tn, i.e. column
    // 64*h + 16*(l/8) + 8*((l/4)%2) + 4*tn + l%4 of the block (with this numbering a lane ends up with eight
    // adjacent columns of one row of Y).
    uint32_t split = 0;
    int64_t m0 = 0;
    int32_t n0 = 0;
    const unsigned char *x_blk[NQ] = {};
    const unsigned char *tile_bytes = nullptr;
    uint32_t a_off[NQ][8];
    uint32_t t_off[NQ];   // WIN: tile position of the lane's piece in the next chunk to fetch
    auto set_block = [&](uint32_t b) __attribute__((always_inline)) {
        uint32_t tile_m, tile_n;
        block_coords(P, b, tile_m, tile_n);
        split = 0;
        if (SPLIT) {
            const uint32_t vrow = tile_m;
            tile_m = vrow / static_cast<uint32_t>(P.splits);
            split = vrow - tile_m * static_cast<uint32_t>(P.splits);
        }
        const uint32_t round0 = split * static_cast<uint32_t>(P.n_rounds);   // first round of this workgroup's part of K (even)
        m0 = int64_t(tile_m) * kBM;
        n0 = static_cast<int32_t>(tile_n) * kBN;
        tile_bytes = reinterpret_cast<const unsigned char *>(tile) + round0 * 16u;
        const int64_t last = P.M - 1 - m0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int lq = first_q + q, gq = lq >> 1, hq = lq & 1;
            x_blk[q] = reinterpret_cast<const unsigned char *>(x) + m0 * P.in * 2 + (gq * 128 - kBias) + round0 * 256u;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int sr = 8 * (8 * hq + j) + (lane >> 3);
                const int r = ((((sr >> 5) + 2 * gq) & 3) << 5) + (sr & 31);
                const uint32_t rw = static_cast<uint32_t>(r < last ? r : last);
                const int chunk = (lane & 7) ^ ((sr >> 1) & 7);
                a_off[q][j] = rw * static_cast<uint32_t>(P.in) * 2u + static_cast<uint32_t>(chunk * 16 + kBias - (j & 3) * 1024);
            }
            const int S = 64 * lq + lane, rho = S & 127, l = rho & 31;
            int32_t u = n0 + (rho & 64) + 16 * (l >> 3) + 8 * ((l >> 2) & 1) + 4 * ((rho >> 5) & 1) + (l & 3);
            u = u < P.U ? u : P.U - 1;   // columns past U repeat the last one; they are never written
            if constexpr (WIN) {
                divide(uint64_t(static_cast<uint32_t>(u)) * static_cast<uint32_t>(P.in), static_cast<uint32_t>(P.p), t_off[q]);
                t_off[q] += static_cast<uint32_t>((S >> 7) * 128);
                if (t_off[q] >= static_cast<uint32_t>(P.p)) t_off[q] -= static_cast<uint32_t>(P.p);
            } else {
                t_off[q] = static_cast<uint32_t>(u) * (static_cast<uint32_t>(P.in) >> 3) + static_cast<uint32_t>((S >> 7) * 16);
            }
        }
    };
    set_block(bid);
    // issue order per round, which the wait counts rely on: eight activation wave-loads per quarter, then (even
    // rounds) a quarter's share of the tile chunk of this round and the next
    // tail: part of the round lies behind the rows' ends (WIN)
    auto issue_x = [&](auto q_c, auto j_c, auto tail_c, int32_t round_, int32_t phase) __attribute__((always_inline)) {
        constexpr int Q = decltype(q_c)::value, J = decltype(j_c)::value;
        const int lq = first_q + Q;
        unsigned char *const ring_q = lds_raw + kRingOff + (lq >> 1) * 16384 + (lq & 1) * 8192;
        const unsigned char *src = x_blk[Q] + static_cast<uint32_t>(round_) * 256u;   // wave-uniform
        asm volatile("" : "+s"(src));   // one scalar base, the lane offset stays a 32-bit register
        uint32_t off = a_off[Q][J];
        asm volatile("" : "+v"(off));
        unsigned char *dst = ring_q + ((round_ + phase) & (kNB - 1)) * kSlotBytes + (J >> 2) * 4096;
        if constexpr (decltype(tail_c)::value) {   // in % 8 == 0: a piece lies inside the row or outside
            const int piece = (lane & 7) ^ ((4 * J + (lane >> 4)) & 7);
            const bool inside = round_ * 128 + 64 * (lq >> 1) + 8 * piece < P.in;
            const unsigned char *from = inside ? src + off : reinterpret_cast<const unsigned char *>(kZeroPiece) - (J & 3) * 1024;
            __builtin_amdgcn_global_load_lds(from, dst, 16, (J & 3) * 1024, 0);
        } else {
            wave_load<(J & 3)>(src, off, dst);
        }
    };
    // WIN: the chunk of the tile that round_ (even) and the next take.  fetch_tile brings the four words that a piece's 128 bits
    // begin in to LDS as they are (by registers the compiler would wait for every load in flight), put_tile, later, shifts
    // them into place; its fifth word is the first of the row's next piece, so that the chunk behind has to be there too.
    auto fetch_tile = [&](int32_t round_) __attribute__((always_inline)) {
        const uint32_t last = ((static_cast<uint32_t>(P.p) + 31u) >> 5) - 4u;
        unsigned char *const raw = lds_raw + kRawOff + ((round_ >> 1) % kRawSlots) * kTileSlotBytes;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t w = t_off[q] >> 5;
            __builtin_amdgcn_global_load_lds(tile + (w < last ? w : last), raw + (first_q + q) * 1024, 16, 0, 0);
            t_off[q] += 256u;
            if (t_off[q] >= static_cast<uint32_t>(P.p)) t_off[q] -= static_cast<uint32_t>(P.p);
        }
    };
    uint32_t t_put[NQ];   // the position of the lane's piece in the next chunk to put in place
    auto start_tile = [&]() __attribute__((always_inline)) {   // of a block's first chunk
#pragma unroll
        for (int q = 0; q < NQ; ++q) t_put[q] = t_off[q];
    };
    auto put_tile = [&](int32_t round_) __attribute__((always_inline)) {
        const uint32_t bits = static_cast<uint32_t>(P.p);
        const uint32_t raw = static_cast<uint32_t>(kRawOff + ((round_ >> 1) % kRawSlots) * kTileSlotBytes);
        const uint32_t raw_next = static_cast<uint32_t>(kRawOff + (((round_ >> 1) + 1) % kRawSlots) * kTileSlotBytes);
        u32x4_t lo[NQ];
        uint32_t hi[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t S = static_cast<uint32_t>(64 * (first_q + q) + lane);
            lds_read16<0>(lo[q], raw + S * 16u);
            lds_read4(hi[q], (S < 128u ? raw : raw_next) + (S ^ 128u) * 16u);
        }
        lds_wait<0>();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            tie(lo[q]);
            tie(hi[q]);
            const uint32_t pos = t_put[q], word[5] = {lo[q][0], lo[q][1], lo[q][2], lo[q][3], hi[q]};
            u32x4_t v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbit(word[i + 1], word[i], pos & 31u);
            if (pos + 288u > bits) {   // the tile's end lies in this piece or the next: from memory, going on at the tile's first bit
                const uint32_t last = (bits - 1u) >> 5;
#pragma unroll 1
                for (int i = 0; i < 4; ++i) {
                    uint32_t b = pos + 32u * static_cast<uint32_t>(i);
                    b = b >= bits ? b - bits : b;
                    const uint32_t k = b >> 5, left = bits - b;
                    uint32_t r = __builtin_amdgcn_alignbit(tile[k < last ? k + 1 : last], tile[k], b & 31u);
                    if (left < 32u) r = (r & ((1u << left) - 1u)) | (tile[0] << left);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = e == i ? r : v[e];
                }
            }
            lds_write16<0>(static_cast<uint32_t>(kTileOff + (first_q + q) * 1024 + lane * 16 + ((round_ >> 1) % kTileSlots) * kTileSlotBytes), v);
            t_put[q] = pos + 256u;
            if (t_put[q] >= bits) t_put[q] -= bits;
        }
    };
    auto issue_tile = [&](auto q_c, int32_t round_) {   // round_ is even
        constexpr int Q = decltype(q_c)::value;
        const unsigned char *src = tile_bytes + static_cast<uint32_t>(round_) * 16u;   // 128 bits per round
        asm volatile("" : "+s"(src));
        uint32_t off = t_off[Q];
        asm volatile("" : "+v"(off));
        __builtin_amdgcn_global_load_lds(src + off, lds_raw + kTileOff + (first_q + Q) * 1024 + ((round_ >> 1) % kTileSlots) * kTileSlotBytes, 16, 0, 0);
    };
    auto issue_quarter = [&](auto q_c, int32_t round_, int32_t phase) __attribute__((always_inline)) {
        auto pieces = [&](auto tail_c) __attribute__((always_inline)) {
            issue_x(q_c, Int<0>{}, tail_c, round_, phase); issue_x(q_c, Int<1>{}, tail_c, round_, phase);
            issue_x(q_c, Int<2>{}, tail_c, round_, phase); issue_x(q_c, Int<3>{}, tail_c, round_, phase);
            issue_x(q_c, Int<4>{}, tail_c, round_, phase); issue_x(q_c, Int<5>{}, tail_c, round_, phase);
            issue_x(q_c, Int<6>{}, tail_c, round_, phase); issue_x(q_c, Int<7>{}, tail_c, round_, phase);
        };
        if constexpr (WIN) {
            if (round_ * 128 + 128 > P.in) {
                pieces(std::true_type{});
                return;
            }
        }
        pieces(std::false_type{});
    };
    auto issue_round = [&](int32_t round_, int32_t phase = 0) {
        issue_quarter(Int<0>{}, round_, phase);
        if constexpr (NQ == 2) issue_quarter(Int<1>{}, round_, phase);
        if ((round_ & 1) == 0) {
            issue_tile(Int<0>{}, round_);
            if constexpr (NQ == 2) issue_tile(Int<1>{}, round_);
        }
    };
    // loads of an odd and of an even round per load wave
    constexpr int kOdd = 8 * NQ, kEven = 9 * NQ;
    // WIN: alpha of a lane's eight columns from col on, replica 0
    auto alpha_index = [&](int32_t col, uint32_t (&idx)[8]) __attribute__((always_inline)) -> bool {   // all the same in the wave?
        uint32_t rest, i = 0;
        if (P.n_alpha > 1) i = divide(uint64_t(static_cast<uint32_t>(col)) * static_cast<uint32_t>(P.in), static_cast<uint32_t>(P.p), rest);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            idx[e] = i;
            if (P.n_alpha > 1) {
                rest += static_cast<uint32_t>(P.in);
                if (rest >= static_cast<uint32_t>(P.p)) { rest -= static_cast<uint32_t>(P.p); ++i; }
            }
        }
        return __all(idx[0] == static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(idx[0]))) && idx[0] == idx[7]);
    };
    // (columns past U and replicas past `out` may name an alpha that does not exist: the last one is read for them)
    auto alphas_of = [&](const uint32_t (&idx)[8], int32_t t, float (&al)[8]) __attribute__((always_inline)) {
        uint32_t raw[8];
        const uint32_t step = static_cast<uint32_t>(t) * static_cast<uint32_t>(P.alpha_step), last = static_cast<uint32_t>(P.n_alpha) - 1u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t i = idx[e] + step;
            lds_read4(raw[e], static_cast<uint32_t>(kAlphaOff) + (i < last ? i : last) * 4u);
        }
        lds_wait<0>();
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            tie(raw[e]);
            al[e] = __uint_as_float(raw[e]);
        }
    };

    // a lane's place in the stores of a replica: eight lanes per row of Y, eight adjacent columns each
    const int g8 = lane & 7, rr = lane >> 3;
    const uint32_t z_lane = (static_cast<uint32_t>(rr) * static_cast<uint32_t>(P.out) + static_cast<uint32_t>(8 * g8)) * 2u;
    const uint32_t out_bytes8 = static_cast<uint32_t>(P.out) * 16u;   // eight rows of Y in bytes
    const uint32_t rep_bytes = static_cast<uint32_t>(P.U) * 2u;

    // =================================================================================================
    // store waves (PERSIST)
    // =================================================================================================
    // MFMA wave q leaves the sums of its 64 x 64 quarter of a finished block in the hand-over area; a store wave
    // takes two quarters into registers (128 per lane) and writes them, scaled, one (replica, quarter, 32 rows)
    // unit after the other, spread evenly over the rounds in which the MFMA waves multiply the next block: the
    // matrix pipe does not wait for the stores, which are most of the bytes this kernel moves.  The stores have
    // waves of their own because the vector-memory counter counts loads and stores alike and in issue order: a
    // wave that did both would wait for its stores whenever it waits for a round of loads.
    if (PERSIST && wave >= 6) {
        float alpha_lanes = 0.f;
        if constexpr (!WIN) {
            const int t = P.n_alpha == 1 ? 0 : (lane < P.reps ? lane : P.reps - 1);
            const uint32_t off = static_cast<uint32_t>(t) * 4u;
            asm volatile("global_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)" : "=v"(alpha_lanes) : "v"(off), "s"(alpha) : "memory");
        }
        // WIN: of the eight columns of a lane in either quarter, replica 0; where all columns of a quarter have the same one (and
        // there are at most 64 replicas), its value for replica t in lane t (a read of LDS per unit cost 4 %)
        uint32_t alpha_at[2][8];
        bool alpha_same[2] = {false, false};
        float alpha_q[2] = {0.f, 0.f};
        int32_t st_col0 = 0;
        float zr[2][2][4][8];   // [quarter][32-row half][row rr + 8*i][column 8*g8 + e]
        unsigned char *st_base = nullptr;   // &Y[first row of quarter 0][first column of quarter 0], replica 0
        int64_t st_rows = 0;          // rows of the quarters that exist (may be <= 0)
        bool st_col_ok[2] = {false, false};
        int32_t st_rot = 0;           // the replica a block starts with: workgroups that store at the same time write different ones
        int32_t st_next = 0, st_total = 0, st_credit = 0;   // units written / to write; spreads them over the rounds
        auto store_unit = [&](int32_t uidx) __attribute__((always_inline)) {
            const int32_t sub = uidx & 3, half = sub & 1, q = sub >> 1;
            int32_t t = (uidx >> 2) + st_rot;
            t = t >= P.reps ? t - P.reps : t;
            float al[8];
            bool exists = true;
            if constexpr (WIN) {
                if (q == 0 ? alpha_same[0] : alpha_same[1]) {
                    const float one = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, q == 0 ? alpha_q[0] : alpha_q[1]), t));
#pragma unroll
                    for (int e = 0; e < 8; ++e) al[e] = one;
                } else if (q == 0) {
                    alphas_of(alpha_at[0], t, al);
                } else {
                    alphas_of(alpha_at[1], t, al);
                }
                exists = st_col0 + 64 * q + 8 * g8 + t * P.U < P.out;
            } else {
                const float one = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha_lanes), t));
#pragma unroll
                for (int e = 0; e < 8; ++e) al[e] = one;
            }
            unsigned char *dst = st_base + static_cast<uint32_t>(t) * rep_bytes + static_cast<uint32_t>(half) * 4u * out_bytes8 + static_cast<uint32_t>(q) * 128u;
            const int64_t rows_left = st_rows - 32 * half;
            auto emit = [&](auto q_c, auto half_c) __attribute__((always_inline)) {
                constexpr int Q = decltype(q_c)::value, H = decltype(half_c)::value;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        v[e] = al[e] * zr[Q][H][i][e];
                        if (RELU) v[e] = fmaxf(v[e], 0.f);
                    }
                    const u32x4_t pk = {pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
                    if (st_col_ok[Q] && exists && rr + 8 * i < rows_left) global_store16<true>(dst, z_lane + static_cast<uint32_t>(i) * out_bytes8, pk);
                }
            };
            if (sub == 0) emit(Int<0>{}, Int<0>{});
            else if (sub == 1) emit(Int<0>{}, Int<1>{});
            else if (sub == 2) emit(Int<1>{}, Int<0>{});
            else emit(Int<1>{}, Int<1>{});
        };
        int32_t ph = 0;
        if constexpr (WIN) {
            __builtin_amdgcn_s_barrier();   // the words of the first chunks are there
            start_tile();
            put_tile(0);
            lds_wait<0>();
        }
        for (;;) {
            const int64_t cur_m0 = m0;
            const int32_t cur_n0 = n0;
            const uint32_t next = bid + gridDim.x;
            const bool more = next < n_blocks;
            __builtin_amdgcn_s_barrier();   // the block's first barrier
            if constexpr (WIN) put_tile(2);
            for (int32_t g = 0; g < n_rounds; ++g) {
                if constexpr (WIN) lds_wait<0>();
                __builtin_amdgcn_s_barrier();
                if constexpr (WIN) {   // the words were there by this barrier; the next one publishes what they become
                    if ((g & 1) && g + 3 < n_rounds) {
                        put_tile(g + 3);
                    } else if (g + 1 == n_rounds && more) {
                        bid = next;
                        set_block(bid);
                        start_tile();
                        put_tile(0);
                    }
                }
                st_credit += st_total;
                for (; st_credit >= n_rounds && st_next < st_total; st_credit -= n_rounds) store_unit(st_next++);
            }
            while (st_next < st_total) store_unit(st_next++);
            if (!WIN && more) {
                bid = next;
                set_block(bid);
            }
            if constexpr (WIN) lds_wait<0>();
            __builtin_amdgcn_s_barrier();   // the two barriers of the hand-over
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_s_barrier();   // the sums of the finished block are in the hand-over area
            // the same turn-round as in the epilogue of the MFMA waves below: eight lanes take one row's 64 columns
            {
                const int ch_a = 2 * g8 + (g8 >> 2), ch_b = 2 * g8 + 1 - (g8 >> 2);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t area = xchg_base(ph) + static_cast<uint32_t>((first_q + q) * 16384);
                    u32x4_t za[2][4], zb[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = rr + 8 * i;
                            const int s_r = ((r >> 1) & 7) ^ (2 * (r & 1));
                            lds_read16<0>(za[h][i], area + static_cast<uint32_t>(h * 8192 + r * 256 + ((ch_a ^ s_r) << 4)));
                            lds_read16<0>(zb[h][i], area + static_cast<uint32_t>(h * 8192 + r * 256 + ((ch_b ^ s_r) << 4)));
                        }
                    lds_wait<0>();
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            tie(za[h][i]);
                            tie(zb[h][i]);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                zr[q][h][i][e] = __uint_as_float(g8 < 4 ? za[h][i][e] : zb[h][i][e]);
                                zr[q][h][i][4 + e] = __uint_as_float(g8 < 4 ? zb[h][i][e] : za[h][i][e]);
                            }
                        }
                }
            }
            {
                const int64_t row0 = cur_m0 + 64 * (first_q >> 1);
                st_base = reinterpret_cast<unsigned char *>(y) + (row0 * P.out + cur_n0) * 2;
                st_rows = P.M - row0;
                st_col_ok[0] = cur_n0 + 8 * g8 < P.U;
                st_col_ok[1] = cur_n0 + 64 + 8 * g8 < P.U;
                st_rot = static_cast<int32_t>(static_cast<uint32_t>(cur_m0 >> 7) % static_cast<uint32_t>(P.reps));
                st_next = 0;
                if constexpr (WIN) {
                    st_col0 = cur_n0;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        alpha_same[q] = alpha_index(cur_n0 + 64 * q + 8 * g8, alpha_at[q]) && P.reps <= 64;
                        float al[8];
                        alphas_of(alpha_at[q], lane, al);
                        alpha_q[q] = al[0];
                    }
                }
                st_total = 4 * P.reps;
                st_credit = 0;
                ph = (ph + n_rounds) & 3;
            }
            if (!more) {
                while (st_next < st_total) store_unit(st_next++);
                return;
            }
        }
    }

    // =================================================================================================
    // load waves
    // =================================================================================================
    if constexpr (WIN) {
        if (wave >= 4) {
        // The rounds of the loops below, two at a time (even, odd).  The words of a chunk are fetched behind the activations of
        // the even round before and put in place two rounds later (PERSIST: by the store waves; two load waves
        // that did it were late for the barriers: 8192 x 3000 -> 1024 distinct columns 56 us against 54); the barrier after that
        // publishes them.  Chunks past the end of a row are fetched and never used.
        auto issue_round_x = [&](int32_t round_, int32_t phase) __attribute__((always_inline)) {
            issue_quarter(Int<0>{}, round_, phase);
            if constexpr (NQ == 2) issue_quarter(Int<1>{}, round_, phase);
        };
        if constexpr (PERSIST) {
            fetch_tile(0);
            fetch_tile(2);
            fetch_tile(4);
            issue_round_x(0, 0);
            issue_round_x(1, 0);
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kOdd));
            __builtin_amdgcn_s_barrier();   // the words are there
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));   // round 0
            int32_t ph = 0;
            for (;;) {
                __builtin_amdgcn_s_barrier();   // meets the MFMA waves' "round 0 readable; the hand-over area is free"
                issue_round_x(2, ph);
                fetch_tile(6);
                const int32_t ph_next = (ph + n_rounds) & 3;
                const uint32_t next = bid + gridDim.x;
                const bool more = next < n_blocks;
                for (int32_t g = 0; g < n_rounds; g += 2) {
                    if (g + 2 < n_rounds || more) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kEven));
                    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                    __builtin_amdgcn_s_barrier();
                    if (g + 3 < n_rounds) issue_round_x(g + 3, ph);
                    else if (more) issue_round_x(1, ph_next);   // (set_block and round 0 of the next block: below)
                    if (g + 3 < n_rounds) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));
                    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kOdd));   // the words of the next block's first two chunks, older than its rounds 0 and 1
                    __builtin_amdgcn_s_barrier();
                    if (g + 4 < n_rounds) {
                        issue_round_x(g + 4, ph);
                        fetch_tile(g + 8);
                    } else if (more) {
                        if (g + 4 == n_rounds) {
                            bid = next;
                            set_block(bid);
                            fetch_tile(0);
                            fetch_tile(2);
                            issue_round_x(0, ph_next);
                        } else {
                            fetch_tile(4);
                        }
                    }
                }
                __builtin_amdgcn_s_barrier();   // the two barriers of the hand-over
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_s_barrier();   // the store waves take the sums of the finished block
                if (!more) return;
                ph = ph_next;
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // rounds 0 and 1 of the next block, the words of its third chunk
            }
        } else {
            start_tile();
            fetch_tile(0);
            fetch_tile(2);
            fetch_tile(4);
            issue_round_x(0, 0);
            issue_round_x(1, 0);
            if (n_rounds > 2) {
                issue_round_x(2, 0);
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * kOdd));
            } else {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kOdd));
            }
            __builtin_amdgcn_s_barrier();   // the words are there
            put_tile(0);
            if (n_rounds > 2) put_tile(2);
            if (n_rounds > 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kOdd));   // round 0
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));
            lds_wait<0>();
            __builtin_amdgcn_s_barrier();   // meets the MFMA waves' "table written, round 0 readable"
            fetch_tile(6);   // into the slot of chunk 0, which every load wave has put in place by that barrier
            for (int32_t g = 0; g < n_rounds; g += 2) {
                if (g + 2 < n_rounds) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kEven));
                else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                lds_wait<0>();
                __builtin_amdgcn_s_barrier();
                if (g + 3 < n_rounds) {
                    issue_round_x(g + 3, 0);
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));
                }
                __builtin_amdgcn_s_barrier();
                if (g + 4 < n_rounds) {
                    issue_round_x(g + 4, 0);
                    fetch_tile(g + 8);
                    put_tile(g + 4);
                }
            }
            __builtin_amdgcn_s_barrier();   // the two barriers of the hand-over
            __builtin_amdgcn_s_barrier();
            return;
        }
        }
    } else if (wave >= 4) {
        if constexpr (PERSIST) {
            // One workgroup walks blocks.  The last three rounds of a block load nothing for it, and the two ring slots behind its last round
            // are free by then: the activations of the next block's rounds 0 and 1 are issued there, one round each,
            // and its first tile chunk behind the last round's barrier (that slot of the tile ring is read until then),
            // so the hand-over between two blocks waits for no load to be issued.
            issue_round(0);
            issue_round(1);
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));   // round 0 and its tile chunk; round 1's loads are younger
            int32_t ph = 0;
            for (;;) {
                __builtin_amdgcn_s_barrier();   // meets the MFMA waves' "round 0 readable; the hand-over area is free"
                issue_round(2, ph);
                const int32_t ph_next = (ph + n_rounds) & 3;
                const uint32_t next = bid + gridDim.x;
                const bool more = next < n_blocks;
                for (int32_t g = 0; g < n_rounds; ++g) {
                    // round g + 1 has to be readable when the MFMA waves pass this barrier; what was issued after its
                    // loads may stay in flight: round g + 2 (with the tile chunk if that round is even), or, at the end of
                    // a block, the next block's round 0
                    if (g + 2 < n_rounds) {
                        if (g & 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));
                        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(kEven));
                    } else if (!more) {
                        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                    } else if (g + 2 == n_rounds) {
                        __builtin_amdgcn_s_waitcnt(vmcnt_imm(8 * NQ));
                    }
                    __builtin_amdgcn_s_barrier();
                    if (g + 3 < n_rounds) {
                        issue_round(g + 3, ph);
                    } else if (more) {
                        if (g + 3 == n_rounds) {
                            bid = next;
                            set_block(bid);
                            issue_quarter(Int<0>{}, 0, ph_next);
                            issue_quarter(Int<1>{}, 0, ph_next);
                        } else if (g + 2 == n_rounds) {
                            issue_quarter(Int<0>{}, 1, ph_next);
                            issue_quarter(Int<1>{}, 1, ph_next);
                        } else {
                            issue_tile(Int<0>{}, 0);
                            issue_tile(Int<1>{}, 0);
                        }
                    }
                }
                __builtin_amdgcn_s_barrier();   // the two barriers of the hand-over
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_s_barrier();   // the store waves take the sums of the finished block
                if (!more) return;
                ph = ph_next;
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // rounds 0 and 1 and the tile chunk of the next block
            }
        } else {
            // rounds 0 .. 2 at once; then, at the top of every round, the loads of round + 3 into the slot that the
            // barrier has just freed
            for (int32_t d = 0; d < 3 && d < n_rounds; ++d) issue_round(d);
            // round 0 is readable once it has landed (two younger rounds may be in flight)
            if (n_rounds >= 3) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd + kEven));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __builtin_amdgcn_s_barrier();   // meets the MFMA waves' "table written, round 0 readable"
            for (int32_t g = 0; g < n_rounds; ++g) {
                // round g + 1 has to be readable when the MFMA waves pass this barrier; the loads of round g + 2 (with
                // the tile chunk if that round is even) are younger and may stay in flight
                if (g + 2 < n_rounds) {
                    if (g & 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kOdd));
                    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(kEven));
                } else {
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                }
                __builtin_amdgcn_s_barrier();
                if (g + 3 < n_rounds) issue_round(g + 3);
            }
            __builtin_amdgcn_s_barrier();   // the two barriers of the hand-over
            __builtin_amdgcn_s_barrier();
            return;
        }
    }

    // =================================================================================================
    // MFMA waves
    // =================================================================================================
    // alpha of replica t in lane t (at most 64 replicas), fetched by hand so that the compiler places no wait
    // for it inside the rounds
    float alpha_lanes = 0.f;
    if constexpr (WIN) {
        for (int32_t i = tid; i < P.n_alpha; i += 256) {
            const uint32_t v = __float_as_uint(alpha[i]);
            asm volatile("ds_write_b32 %0, %1" : : "v"(static_cast<uint32_t>(kAlphaOff) + static_cast<uint32_t>(i) * 4u), "v"(v) : "memory");
        }
    } else {
        const int t = P.n_alpha == 1 ? 0 : (lane < P.reps ? lane : P.reps - 1);
        const uint32_t off = static_cast<uint32_t>(t) * 4u;
        asm volatile("global_load_dword %0, %1, %2" : "=v"(alpha_lanes) : "v"(off), "s"(alpha));
    }

    int32_t ph = 0;   // ring phase of the current block

    // sign table: entry e, element i is +1 if bit i of e is set, else -1
    if (tid < 256) {
        u32x4_t t;
        const int e = tid;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            t[v] = (((e >> (2 * v)) & 1) ? 0x3f80u : 0xbf80u) | ((((e >> (2 * v + 1)) & 1) ? 0x3f80u : 0xbf80u) << 16);
        lds_write16<kTableOff>(static_cast<uint32_t>(e) * 16u, t);
    }

    // operand read addresses inside a ring slot: row slot 32*tm + ln, K step ks: chunk 2*ks + lg at chunk slot
    // (2*ks + lg) ^ ((ln >> 1) & 7)
    uint32_t a_rd[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        a_rd[ks] = static_cast<uint32_t>(kRingOff + grp * 16384 + ln * 128 + (((2 * ks + lg) ^ ((ln >> 1) & 7)) << 4));
    // window read: LDS row 64*wn + ln (tn = 0) and + 32 (tn = 1) of the chunk, the K group's 8 bytes of the piece
    const uint32_t w_rd = static_cast<uint32_t>(kTileOff + (64 * wn + ln) * 16 + 8 * grp);
    // byte 2*ks + lg of a window: word ks / 2, bits 16*(ks % 2) + 8*lg on
    uint32_t bsh[2] = {8u * static_cast<uint32_t>(lg), 16u + 8u * static_cast<uint32_t>(lg)};
    asm volatile("" : "+v"(bsh[0]), "+v"(bsh[1]));

    f32x16_t acc[4][2];
    Frag A[2][4];       // [operand set][tm]
    Frag B[2][2];       // [operand set][tn]
    u32x4_t win[2];     // [round parity]: words 0-1 the 64 window bits of column tn = 0, words 2-3 of tn = 1

    auto table_read = [&](u32x4_t &dst, uint32_t word, uint32_t shift) {
        const uint32_t addr = __builtin_amdgcn_ubfe(word, shift, 8) << 4;
        lds_read16<kTableOff>(dst, addr);
    };

    auto settle = [&]() {   // all of operand set 0 has landed
        lds_wait<0>();
        tie(B[0][0].q); tie(B[0][1].q);
        tie(A[0][0].q); tie(A[0][1].q); tie(A[0][2].q); tie(A[0][3].q);
    };

    // ---- one K step: 8 MFMAs ---------------------------------------------------------------------
    // Multiplies with operand set S and requests the operands of the following K step into the other set: six
    // LDS reads, one in each of the first six MFMA slots, in the order in which that step's MFMAs need them
    // (+-1 operand of tn = 0, activation fragment of tm = 0, +-1 operand of tn = 1, fragments of tm = 1, 2, 3).
    // LDS operations complete in order, so "at most N pending" names exactly which operands have arrived;
    // three waits cover the step, and every operand has the time of at least six MFMAs to arrive.  A slot is:
    // wait, request, MFMA, side work.  W1 = 1: the window read of the next round was issued behind the previous
    // step's requests.
    auto kstep = [&](auto s_c, auto w1_c, uint32_t n_addr, uint32_t nw0, uint32_t nw1, auto nks_c, auto &&side) __attribute__((always_inline)) {
        constexpr int S = decltype(s_c)::value, N = S ^ 1, W1 = decltype(w1_c)::value, NKS = decltype(nks_c)::value;
        auto mfma = [&](int tm, int tn) {
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(B[S][tn].v, A[S][tm].v, acc[tm][tn], 0, 0, 0);
        };
        lds_wait<3 + W1>(); tie(B[S][0].q); tie(A[S][0].q); tie(B[S][1].q);
        side(Int<-1>{});   // what else this wait covers
        table_read(B[N][0].q, nw0, bsh[NKS]);
        mfma(0, 0);
        side(Int<0>{});
        __builtin_amdgcn_sched_barrier(0);
        lds_read16<0>(A[N][0].q, n_addr);
        mfma(0, 1);
        side(Int<1>{});
        __builtin_amdgcn_sched_barrier(0);
        lds_wait<4 + W1>(); tie(A[S][1].q);
        table_read(B[N][1].q, nw1, bsh[NKS]);
        mfma(1, 0);
        side(Int<2>{});
        __builtin_amdgcn_sched_barrier(0);
        lds_read16<4096>(A[N][1].q, n_addr);
        mfma(1, 1);
        side(Int<3>{});
        __builtin_amdgcn_sched_barrier(0);
        lds_wait<4 + W1>(); tie(A[S][2].q); tie(A[S][3].q);
        lds_read16<8192>(A[N][2].q, n_addr);
        mfma(2, 0);
        side(Int<4>{});
        __builtin_amdgcn_sched_barrier(0);
        lds_read16<12288>(A[N][3].q, n_addr);
        mfma(2, 1);
        side(Int<5>{});
        __builtin_amdgcn_sched_barrier(0);
        mfma(3, 0);
        side(Int<6>{});
        __builtin_amdgcn_sched_barrier(0);
        mfma(3, 1);
        side(Int<7>{});
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- one round: four K steps, 32 MFMAs -------------------------------------------------------------
    // PAR: parity of the round.  The round opens with the barrier that makes round + 1 readable (its loads were
    // issued two rounds ago) and frees the slot of round - 1 for the loads of round + 3.  On entry the operands
    // of the first K step have been requested into set 0.
    auto round = [&](auto par_c, int32_t g) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par_c)::value;
        __builtin_amdgcn_s_barrier();
        const uint32_t cur = static_cast<uint32_t>(((g + ph) & (kNB - 1)) * kSlotBytes);
        const uint32_t nxt = static_cast<uint32_t>(((g + 1 + ph) & (kNB - 1)) * kSlotBytes);
        // windows of the next round: an even round reads the second piece of its own chunk, an odd round the
        // first piece of the next chunk
        const uint32_t w_addr = w_rd + static_cast<uint32_t>((((g + 1) >> 1) % kTileSlots) * kTileSlotBytes + (PAR == 0 ? 2048 : 0));
        u32x4_t &wc = win[PAR];       // this round's windows
        u32x4_t &wx = win[PAR ^ 1];   // the next round's
        kstep(Int<0>{}, Int<0>{}, a_rd[1] + cur, wc[0], wc[2], Int<1>{}, [&](auto slot_c) __attribute__((always_inline)) {
            constexpr int SLOT = decltype(slot_c)::value;
            if constexpr (SLOT == 6) lds_read2x8(wx, w_addr);
        });
        kstep(Int<1>{}, Int<1>{}, a_rd[2] + cur, wc[1], wc[3], Int<0>{}, [&](auto) __attribute__((always_inline)) {});
        kstep(Int<0>{}, Int<0>{}, a_rd[3] + cur, wc[1], wc[3], Int<1>{}, [&](auto slot_c) __attribute__((always_inline)) {
            constexpr int SLOT = decltype(slot_c)::value;
            if constexpr (SLOT == -1) tie(wx);   // the window read is older than this step's operands
        });
        kstep(Int<1>{}, Int<0>{}, a_rd[0] + nxt, wx[0], wx[2], Int<0>{}, [&](auto) __attribute__((always_inline)) {});
    };

    lds_wait<0>();   // the table
    if constexpr (WIN) __builtin_amdgcn_s_barrier();   // the load and store waves': the words of the first chunks are there
    for (;;) {   // one block per pass (a single pass unless PERSIST)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // ---- first operands -------------------------------------------------------------------------
    __builtin_amdgcn_s_barrier();   // table written, round 0 readable (PERSIST: and every wave is done with the hand-over area)
    lds_read2x8(win[0], w_rd);      // windows of round 0: chunk slot 0, piece 0
    lds_wait<0>();
    tie(win[0]);
    {
        const uint32_t first = a_rd[0] + static_cast<uint32_t>(ph * kSlotBytes);
        table_read(B[0][0].q, win[0][0], bsh[0]);
        lds_read16<0>(A[0][0].q, first);
        table_read(B[0][1].q, win[0][2], bsh[0]);
        lds_read16<4096>(A[0][1].q, first);
        lds_read16<8192>(A[0][2].q, first);
        lds_read16<12288>(A[0][3].q, first);
    }
    settle();

    // One plain loop over pairs of rounds; the operands that its last round requests (of a round that does not
    // exist) land before anything else touches their registers.
    for (int32_t g = 0; g < n_rounds; g += 2) {
        round(Int<0>{}, g);
        round(Int<1>{}, g + 1);
    }
    settle();

    // ---- the K groups add their partial sums ---------------------------------------------------------
    // Accumulator index tm of group g stands for row block (tm + 2g) % 4: each group keeps acc[0..1] and hands
    // acc[2..3] to the other one through its 16 KiB slot (the ring is free: every load has landed, every read
    // of it is done once all waves are here).  The matrix pipe must have written the accumulators back before
    // the assembly below reads them.
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    asm volatile("" : "+v"(alpha_lanes));
    __builtin_amdgcn_s_barrier();
    asm volatile("s_nop 15");
    asm volatile("s_nop 15");
    const uint32_t xchg_mine = xchg_base(ph) + static_cast<uint32_t>(li * 16384);
    {
        const uint32_t dst = xchg_base(ph) + static_cast<uint32_t>((li ^ 2) * 16384) + static_cast<uint32_t>(lane) * 16u;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            u32x4_t s[8];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[t * 4 + q][e] = __float_as_uint(acc[2 + half][t][4 * q + e]);
            const uint32_t d = dst + static_cast<uint32_t>(half * 8192);
            lds_write16<0 * 1024>(d, s[0]);
            lds_write16<1 * 1024>(d, s[1]);
            lds_write16<2 * 1024>(d, s[2]);
            lds_write16<3 * 1024>(d, s[3]);
            lds_write16<4 * 1024>(d, s[4]);
            lds_write16<5 * 1024>(d, s[5]);
            lds_write16<6 * 1024>(d, s[6]);
            lds_write16<7 * 1024>(d, s[7]);
        }
    }
    lds_wait<0>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        u32x4_t got[8];
        const uint32_t src = xchg_mine + static_cast<uint32_t>(half * 8192) + static_cast<uint32_t>(lane) * 16u;
        lds_read16<0 * 1024>(got[0], src);
        lds_read16<1 * 1024>(got[1], src);
        lds_read16<2 * 1024>(got[2], src);
        lds_read16<3 * 1024>(got[3], src);
        lds_read16<4 * 1024>(got[4], src);
        lds_read16<5 * 1024>(got[5], src);
        lds_read16<6 * 1024>(got[6], src);
        lds_read16<7 * 1024>(got[7], src);
        lds_wait<0>();
#pragma unroll
        for (int i = 0; i < 8; ++i) tie(got[i]);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[half][t][4 * q + e] += __uint_as_float(got[t * 4 + q][e]);
    }

    // ---- epilogue: y[m, u + t*U] = alpha[t] * Z[m, u] ---------------------------------------------------
    // The lane holds, for row block tm, row 32*tm + ln and, in registers 4q .. 4q + 3 of tiles 0 and 1, columns
    // 16*q + 8*lg .. + 7 of the wave's 64.  The wave turns 32 rows at a time round through the part of its slot
    // that it has read already, so that eight lanes hold one row's 64 columns: a store instruction then writes
    // eight whole 128-byte lines.  LDS row r is 256 bytes; the 16-byte chunk ch of it (columns 4*ch .. 4*ch + 3)
    // sits at chunk position ch ^ s(r), s(r) = ((r >> 1) & 7) ^ (2 * (r & 1)): the writes (lanes = rows) and the
    // reads (eight lanes per row; a lane reads chunks 2*g8 and 2*g8 + 1, the upper four lanes in the other
    // order) are then free of bank conflicts.
    if constexpr (PERSIST) {
        // the store waves write the replicas: leave both 32-row halves in this wave's part of the hand-over area (all of
        // which the wave has read by now), in the layout described above
        const int s_w = ((ln >> 1) & 7) ^ (2 * (ln & 1));
#pragma unroll
        for (int tm = 0; tm < 2; ++tm)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int tn = 0; tn < 2; ++tn) {
                    const int ch = 4 * q + 2 * lg + tn;
                    u32x4_t v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(acc[tm][tn][4 * q + e]);
                    lds_write16<0>(xchg_mine + static_cast<uint32_t>(tm * 8192 + ln * 256 + ((ch ^ s_w) << 4)), v);
                }
        lds_wait<0>();
        __builtin_amdgcn_s_barrier();   // the store waves take the sums from here
            const uint32_t next = bid + gridDim.x;
        if (next >= n_blocks) break;
        bid = next;
        ph = (ph + n_rounds) & 3;
        continue;
    }
    const bool col_ok = n0 + 64 * wn + 8 * g8 < P.U;
#pragma unroll
    for (int tm = 0; tm < 2; ++tm) {
        float zr[4][8];
        {
            const int s_w = ((ln >> 1) & 7) ^ (2 * (ln & 1));
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int tn = 0; tn < 2; ++tn) {
                    const int ch = 4 * q + 2 * lg + tn;
                    u32x4_t v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(acc[tm][tn][4 * q + e]);
                    lds_write16<0>(xchg_mine + static_cast<uint32_t>(ln * 256 + ((ch ^ s_w) << 4)), v);
                }
            lds_wait<0>();
            __builtin_amdgcn_wave_barrier();
            const int ch_a = 2 * g8 + (g8 >> 2), ch_b = 2 * g8 + 1 - (g8 >> 2);
            u32x4_t za[4], zb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = rr + 8 * i;
                const int s_r = ((r >> 1) & 7) ^ (2 * (r & 1));
                lds_read16<0>(za[i], xchg_mine + static_cast<uint32_t>(r * 256 + ((ch_a ^ s_r) << 4)));
                lds_read16<0>(zb[i], xchg_mine + static_cast<uint32_t>(r * 256 + ((ch_b ^ s_r) << 4)));
            }
            lds_wait<0>();
#pragma unroll
            for (int i = 0; i < 4; ++i) { tie(za[i]); tie(zb[i]); }
            __builtin_amdgcn_wave_barrier();   // the next 32 rows overwrite the staging area
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    zr[i][e] = __uint_as_float(g8 < 4 ? za[i][e] : zb[i][e]);
                    zr[i][4 + e] = __uint_as_float(g8 < 4 ? zb[i][e] : za[i][e]);
                }
        }
        // rows m0 + 64*grp + 32*tm + rr + 8*i, columns n0 + 64*wn + 8*g8 .. + 7
        const int64_t row0 = m0 + 64 * grp + 32 * tm;
        const int64_t rows_left = P.M - row0;   // may be <= 0
        if constexpr (SPLIT) {
            typedef __attribute__((address_space(1))) u32x4_t global_u32x4_t;
            unsigned char *dst = reinterpret_cast<unsigned char *>(P.partial + (int64_t(split) * P.M + row0) * P.U + n0 + 64 * wn);
            const uint32_t lane_off = (static_cast<uint32_t>(rr) * static_cast<uint32_t>(P.U) + static_cast<uint32_t>(8 * g8)) * 4u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (col_ok && rr + 8 * i < rows_left) {
                    const uint32_t off = lane_off + static_cast<uint32_t>(i) * static_cast<uint32_t>(P.U) * 32u;   // eight rows on
                    u32x4_t lo, hi;
#pragma unroll
                    for (int e = 0; e < 4; ++e) { lo[e] = __float_as_uint(zr[i][e]); hi[e] = __float_as_uint(zr[i][4 + e]); }
                    *(global_u32x4_t *)(dst + off) = lo;
                    *(global_u32x4_t *)(dst + off + 16) = hi;
                }
            }
            continue;
        }
        unsigned char *z_rep = reinterpret_cast<unsigned char *>(y) + (row0 * P.out + n0 + 64 * wn) * 2;
        uint32_t alpha_at[8];
        if constexpr (WIN) alpha_index(n0 + 64 * wn + 8 * g8, alpha_at);
        for (int32_t t = 0; t < P.reps; ++t, z_rep += rep_bytes) {
            float al[8];
            bool exists = col_ok;
            if constexpr (WIN) {
                alphas_of(alpha_at, t, al);
                exists = col_ok && n0 + 64 * wn + 8 * g8 + t * P.U < P.out;
            } else {
                const float one = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha_lanes), t));
#pragma unroll
                for (int e = 0; e < 8; ++e) al[e] = one;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] = al[e] * zr[i][e];
                    if (RELU) v[e] = fmaxf(v[e], 0.f);
                }
                const u32x4_t pk = {pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
                typedef __attribute__((address_space(1))) u32x4_t global_u32x4_t;
                unsigned char *dst = z_rep;
                asm volatile("" : "+s"(dst));
                uint32_t off = z_lane + static_cast<uint32_t>(i) * out_bytes8;
                asm volatile("" : "+v"(off));   // scalar base + 32-bit lane offset
                if (exists && rr + 8 * i < rows_left) *(global_u32x4_t *)(dst + off) = pk;
            }
        }
    }
    break;   // one block per workgroup
    }
}

// Second pass of split K: z = partial[0] + partial[1] + ... (ascending, float32), y[m, u + t*U] = alpha[t] * z.
// One thread per eight adjacent distinct columns of a row.
template <bool RELU>
__global__ __launch_bounds__(128) void linear_split_reduce_kernel(const float *__restrict__ partial, uint16_t *__restrict__ y,
                                                                  const float *__restrict__ alpha, BlockParams P) {
    const int64_t groups = P.U / 8;
    const int64_t idx = int64_t(blockIdx.x) * 128 + threadIdx.x;
    if (idx >= P.M * groups) return;
    const int64_t m = idx / groups, g = idx - m * groups;
    const int64_t plane = P.M * int64_t(P.U);
    const float *src = partial + m * P.U + 8 * g;
    float z[8];
    {
        const float4 a = *reinterpret_cast<const float4 *>(src), b = *reinterpret_cast<const float4 *>(src + 4);
        z[0] = a.x; z[1] = a.y; z[2] = a.z; z[3] = a.w; z[4] = b.x; z[5] = b.y; z[6] = b.z; z[7] = b.w;
    }
    for (int32_t s = 1; s < P.splits; ++s) {
        const float4 a = *reinterpret_cast<const float4 *>(src + s * plane), b = *reinterpret_cast<const float4 *>(src + s * plane + 4);
        z[0] += a.x; z[1] += a.y; z[2] += a.z; z[3] += a.w; z[4] += b.x; z[5] += b.y; z[6] += b.z; z[7] += b.w;
    }
    uint16_t *dst = y + m * P.out + 8 * g;
    for (int32_t t = 0; t < P.reps; ++t, dst += P.U) {
        const float al = alpha[P.n_alpha == 1 ? 0 : t];
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = al * z[e];
            if (RELU) v[e] = fmaxf(v[e], 0.f);
        }
        *reinterpret_cast<u32x4_t *>(dst) = u32x4_t{pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
    }
}

int device_cus() {
    int device = 0, cus = 256;
    if (hipGetDevice(&device) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && v > 0) cus = v;
    }
    return cus;
}

void fill_params(const LinearArgs &a, BlockParams &P) {
    P.M = a.M;
    P.in = static_cast<int32_t>(a.in);
    P.out = static_cast<int32_t>(a.out);
    P.U = static_cast<int32_t>(a.p / a.in);
    P.reps = static_cast<int32_t>(a.out / P.U);
    P.n_alpha = a.n_alpha;
    P.tiles_m = static_cast<uint32_t>((a.M + kBM - 1) / kBM);
    P.tiles_n = (P.U + kBN - 1) / kBN;
    P.n_rounds = P.in / 128;
    P.splits = 1;
    P.vrows = P.tiles_m;
    P.partial = nullptr;
}

tbn_status set_lds_limit_once(const void *kernel, int lds) {
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    return e == hipSuccess ? TBN_OK : TBN_ERR_DEVICE;
}

}  // namespace

// Shapes this kernel takes: bfloat16, tile of whole rows, K in whole pairs of rounds (in % 256 == 0), 16-byte
// stores possible, every offset inside a block in 32 bits.
bool linear_block_supported(const LinearArgs &a) {
    if (a.dt != TBN_BF16) return false;
    if (a.in % 256 != 0 || a.p % a.in != 0) return false;
    const int64_t U = a.p / a.in;
    if (U > a.out || a.out % U != 0) return false;   // (holds whenever p % in == 0; U = out / k)
    if (U % 8 != 0 || a.out / U > 64) return false;
    if (a.in > (1 << 20) || a.out > (1 << 22) || a.p >= (int64_t(1) << 31)) return false;
    if (a.M < 1 || a.M > (int64_t(1) << 36)) return false;
    if ((reinterpret_cast<uintptr_t>(a.x) & 15u) || (reinterpret_cast<uintptr_t>(a.y) & 15u)) return false;
    if (reinterpret_cast<uintptr_t>(a.tile) & 15u) return false;
    const int64_t blocks = ((a.M + kBM - 1) / kBM) * ((U + kBN - 1) / kBN);
    return blocks <= 0x7fffffffLL;
}

// Split K: how many workgroups share a block's K loop so that the grid about fills the chip (0: no split).  A part
// is a whole number of round pairs (256 elements of K) and at least one.  The split costs a second launch and a
// round trip of the float32 partial sums, about 12 us more fixed time than one kernel on MI355X, so it is taken
// only where a cost model fitted to measurements at 512 distinct columns predicts a gain of more than 10 %
// (R = in / 128 rounds; one kernel: 8 + 0.26 R (1 + blocks / 256) us on the streaming kernel's grids, 12 + 0.55 R us
// at 128 blocks and more; split: 20 + 0.55 R / S + 8 blocks / 128 us.  Measured, out = 4096, k = 8:
// in = 16384, batch 512 / 1024 / 2048 / 4096: 26 / 26 / 38 / 64 us against 40 / 44 / 47 / 72; in = 8192: equal;
// in = 4096: 22 / 22 / 25 / 31 against 15 / 16 / 17 / 27, not taken).  TBN_FLAG_SPLIT_K skips the model.
int linear_split_plan(const LinearArgs &a) {
    if (!linear_block_supported(a)) return 0;
    const int64_t U = a.p / a.in;
    const int64_t blocks = ((a.M + kBM - 1) / kBM) * ((U + kBN - 1) / kBN);
    const int64_t pairs = a.in / 256;
    const int cus = device_cus();
    int best = 0;
    for (int s = 2; s <= 16; s *= 2)
        if (blocks * s <= cus && pairs % s == 0) best = s;
    if (!best || (a.flags & TBN_FLAG_SPLIT_K)) return best;
    const double R = double(a.in) / 128.0;
    const double one = blocks <= 128 ? 8.0 + 0.26 * R * (1.0 + double(blocks) / 256.0) : 12.0 + 0.55 * R;
    const double split = 20.0 + 0.55 * R / best + 8.0 * double(blocks) / 128.0;
    return split < 0.9 * one ? best : 0;
}

size_t linear_split_workspace_bytes(const LinearArgs &a, int splits) {
    return static_cast<size_t>(splits) * static_cast<size_t>(a.M) * static_cast<size_t>(a.p / a.in) * sizeof(float);
}

tbn_status launch_linear_split(const LinearArgs &a, int splits, void *workspace) {
    BlockParams P;
    fill_params(a, P);
    P.splits = splits;
    P.n_rounds = P.in / 128 / splits;
    P.vrows = P.tiles_m * static_cast<uint32_t>(splits);
    P.partial = static_cast<float *>(workspace);
    const int64_t wgs = int64_t(P.vrows) * P.tiles_n;
    typedef void (*kernel_t)(const uint16_t *, uint16_t *, const uint32_t *, const float *, BlockParams);
    static const kernel_t kernel = &linear_block_bf16_kernel<false, true, false, false>;
    static const tbn_status attr = set_lds_limit_once(reinterpret_cast<const void *>(kernel), kLdsBytes);
    if (attr != TBN_OK) {
        set_error("tbn_linear_forward_ws: cannot reserve %d bytes of LDS for the block kernel", kLdsBytes);
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(wgs)), dim3(512), kLdsBytes, a.stream,
                       static_cast<const uint16_t *>(a.x), static_cast<uint16_t *>(a.y), a.tile, a.alpha, P);
    tbn_status st = check_launch("tbn_linear_forward_ws (split-K matrix-core kernel)");
    if (st != TBN_OK) return st;
    const int64_t threads = a.M * (P.U / 8);
    const dim3 grid(static_cast<unsigned>((threads + 127) / 128));
    if (a.flags & TBN_FLAG_RELU)
        hipLaunchKernelGGL(linear_split_reduce_kernel<true>, grid, dim3(128), 0, a.stream, P.partial, static_cast<uint16_t *>(a.y), a.alpha, P);
    else
        hipLaunchKernelGGL(linear_split_reduce_kernel<false>, grid, dim3(128), 0, a.stream, P.partial, static_cast<uint16_t *>(a.y), a.alpha, P);
    return check_launch("tbn_linear_forward_ws (sum of the split-K partial sums)");
}

// The windowed form: any row length in multiples of 8 and tile starts anywhere, a row holding at most one of them.
static bool linear_window_supported(const LinearArgs &a) {
    if (a.dt != TBN_BF16 || a.in % 8 != 0 || a.in < 8) return false;
    if (a.p < a.in || a.p < 512 || a.p >= (int64_t(1) << 31) - 512) return false;   // positions in 32 bits, at most one tile end in two pieces
    if (a.in > (1 << 20) || a.out > (1 << 22) || a.out % 8 != 0) return false;
    if (unique_rows(a.out, a.in, a.p) % 8 != 0 || a.n_alpha > kMaxWinAlphas) return false;
    if (a.M < 1 || a.M > (int64_t(1) << 36)) return false;
    if ((reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.y)) & 15u) return false;
    if (reinterpret_cast<uintptr_t>(a.tile) & 3u) return false;
    // the repair pass of the columns with two alphas must be able to run (its fallback counts groups of 16 rows in 16 bits)
    if (a.n_alpha > 1 && a.p % a.in != 0 && a.M > int64_t(65535) * 16) return false;
    return ((a.M + kBM - 1) / kBM) * ((unique_rows(a.out, a.in, a.p) + kBN - 1) / kBN) <= 0x7fffffffLL;
}

// Where the windowed form beats the general matrix-core kernel (graph replays of both kernels over 10700 random layers that the latter
// took; microseconds, general / this).
//   * With at most one block per CU nearly always (1090 x 744 -> 1600, k = 12: 23.0 / 15.6; 2048 x 3000 -> 1024 distinct columns
//     36.2 / 29.7 with the repair pass; 3746 x 952 -> 584 15.2 / 13.0), but not on rows of one pair of rounds that is mostly padding.
//   * Every tile start among a block's 128 rows stops a load wave for a chain of reads (put_tile), so not where a block has many:
//     128 in / p of them.  One alpha: from three on (3141 x 3608 -> 80, k = 11, 17.6 of them: 23.9 / 33.0; three to four: level, a quarter of
//     the layers more than 4 % slower), on two pairs of rounds from one on (level, a quarter slower).  An alpha per tile copy costs
//     the general kernel more: from five on, with rows of more than 1024 and at most two replicas (427 layers 5 % slower here; those that
//     stay 17 % faster).
//   * On larger grids the general kernel has two workgroups per CU and smaller losses in the last, incomplete wave of blocks (288
//     blocks: 25 / 60); rows that do not start on lines cost it more: there two models by least squares (R rounds, W = blocks per CU
//     rounded up; 10 and 11 % off on the 2787 drawn layers that the last sentence leaves them), and this form has to be
//     estimated 3 % faster (8192 x 3000 -> 1024 distinct columns: 60.6 / 55.0), 5 % with rows of at most 2048, which must not be a
//     tenth padding either (15 layers of 1300 - 1700: 6 % slower).  Rows of whole lines stay with the general kernel (8192 x 3008 ->
//     1024: 51 / 53; 369 drawn ones: 11 % slower here), and so do five replicas and more, or three where activations and
//     outputs overflow the last-level cache: the models do not see the cost of the non-temporal stores (21113 x 3512 -> 3552, 12
//     replicas: 101 / 162; 17647 x 4000 -> 4880, ten: 153 / 210).
bool linear_window_preferred(const LinearArgs &a) {
    if ((a.flags & ~uint32_t(TBN_FLAG_RELU)) || !linear_window_supported(a)) return false;   // flags that steer to another kernel
    const int64_t U = unique_rows(a.out, a.in, a.p), reps = (a.out + U - 1) / U, cus = device_cus();
    const int64_t blocks = ((a.M + kBM - 1) / kBM) * ((U + kBN - 1) / kBN);
    const auto starts = [&](int64_t n) { return a.p % a.in != 0 && kBN * a.in >= n * a.p; };   // at least n tile starts inside a block's rows
    if (blocks <= cus) {
        if (a.in < 200) return false;
        if (a.n_alpha == 1) return !starts(3) && !(starts(1) && a.in > 256 && a.in <= 512);
        return !(starts(5) && a.in > 1024 && reps <= 2);
    }
    if (a.in % 64 == 0 || starts(3)) return false;
    const bool overflow = a.M * (a.in + a.out) > 85000000;   // 170 MB in bfloat16
    if (reps >= 5 || (reps >= 3 && overflow)) return false;
    const bool short_rows = a.in <= 2048;
    const double R = 2.0 * static_cast<double>((a.in + 255) / 256), W = static_cast<double>((blocks + cus - 1) / cus);
    if (short_rows && R * 128.0 > 1.1 * static_cast<double>(a.in)) return false;
    const double outputs = 1e-6 * static_cast<double>(a.M) * static_cast<double>(a.out);
    const double per_cu = static_cast<double>(blocks) / static_cast<double>(cus), pairs = static_cast<double>((blocks + 2 * cus - 1) / (2 * cus));
    const double general = 5.71 + R * (0.2685 * per_cu + 0.687 * W + 0.1293 * pairs) + 0.231 * outputs;
    const double here = 7.30 + 0.7866 * W * R + 1.7866 * W + 0.2972 * outputs;
    return here < (short_rows ? 0.95 : 0.97) * general;
}

tbn_status launch_linear_window(const LinearArgs &a) {
    BlockParams P;
    const int64_t U = unique_rows(a.out, a.in, a.p);
    P.M = a.M;
    P.in = static_cast<int32_t>(a.in);
    P.out = static_cast<int32_t>(a.out);
    P.U = static_cast<int32_t>(U);
    P.reps = static_cast<int32_t>((a.out + U - 1) / U);
    P.n_alpha = a.n_alpha;
    P.tiles_m = static_cast<uint32_t>((a.M + kBM - 1) / kBM);
    P.tiles_n = (P.U + kBN - 1) / kBN;
    P.n_rounds = 2 * static_cast<int32_t>((a.in + 255) / 256);
    P.splits = 1;
    P.vrows = P.tiles_m;
    P.partial = nullptr;
    P.p = static_cast<int32_t>(a.p);
    P.alpha_step = a.n_alpha > 1 && P.reps > 1 ? static_cast<int32_t>(U * a.in / a.p) : 0;   // (more than one replica: U is the period)
    const int lds = kAlphaOff + 4 * a.n_alpha;
    const bool relu = (a.flags & TBN_FLAG_RELU) != 0;
    int cus = device_cus() & ~7;
    if (cus < 8) cus = 8;
    const int64_t blocks = int64_t(P.tiles_m) * P.tiles_n;
    const bool persist = blocks > cus && P.n_rounds >= 4;
    typedef void (*kernel_t)(const uint16_t *, uint16_t *, const uint32_t *, const float *, BlockParams);
    static const kernel_t kernels[4] = {&linear_block_bf16_kernel<false, false, false, true>, &linear_block_bf16_kernel<true, false, false, true>,
                                        &linear_block_bf16_kernel<false, false, true, true>, &linear_block_bf16_kernel<true, false, true, true>};
    static const tbn_status attr[4] = {set_lds_limit_once(reinterpret_cast<const void *>(kernels[0]), 160 * 1024),
                                       set_lds_limit_once(reinterpret_cast<const void *>(kernels[1]), 160 * 1024),
                                       set_lds_limit_once(reinterpret_cast<const void *>(kernels[2]), 160 * 1024),
                                       set_lds_limit_once(reinterpret_cast<const void *>(kernels[3]), 160 * 1024)};
    const int which = (relu ? 1 : 0) + (persist ? 2 : 0);
    if (attr[which] != TBN_OK) {
        set_error("tbn_linear_forward: cannot reserve %d bytes of LDS for the block kernel", lds);
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL(kernels[which], dim3(static_cast<unsigned>(persist ? cus : blocks)), dim3(512), lds, a.stream,
                       static_cast<const uint16_t *>(a.x), static_cast<uint16_t *>(a.y), a.tile, a.alpha, P);
    const tbn_status st = check_launch("tbn_linear_forward (matrix-core kernel with load waves, windows)");
    if (st != TBN_OK || a.n_alpha == 1 || a.p % a.in == 0) return st;
    return launch_linear_tile_ends(a);   // columns whose weight row holds a tile start: two alphas
}

tbn_status launch_linear_block(const LinearArgs &a) {
    BlockParams P;
    fill_params(a, P);
    const dim3 grid(static_cast<unsigned>(int64_t(P.tiles_m) * P.tiles_n));
    const bool relu = (a.flags & TBN_FLAG_RELU) != 0;
    typedef void (*kernel_t)(const uint16_t *, uint16_t *, const uint32_t *, const float *, BlockParams);
    // more blocks than CUs and at least four rounds: one persistent workgroup per CU
    int cus = device_cus() & ~7;
    if (cus < 8) cus = 8;
    const bool persist = int64_t(P.tiles_m) * P.tiles_n > cus && P.n_rounds >= 4;
    // (its store waves write with non-temporal stores whatever the shape: next to a running K loop, plain stores push
    // the activations that the other column blocks of the same rows still need out of the XCD's L2)
    static const kernel_t kernels[4] = {&linear_block_bf16_kernel<false, false, false, false>, &linear_block_bf16_kernel<true, false, false, false>,
                                        &linear_block_bf16_kernel<false, false, true, false>, &linear_block_bf16_kernel<true, false, true, false>};
    // dynamic LDS above the default limit has to be allowed once per kernel (thread-safe static initialisation)
    static const tbn_status attr[4] = {set_lds_limit_once(reinterpret_cast<const void *>(kernels[0]), kLdsBytes),
                                       set_lds_limit_once(reinterpret_cast<const void *>(kernels[1]), kLdsBytes),
                                       set_lds_limit_once(reinterpret_cast<const void *>(kernels[2]), kLdsBytes),
                                       set_lds_limit_once(reinterpret_cast<const void *>(kernels[3]), kLdsBytes)};
    const int which = (relu ? 1 : 0) + (persist ? 2 : 0);
    if (attr[which] != TBN_OK) {
        set_error("tbn_linear_forward: cannot reserve %d bytes of LDS for the block kernel", kLdsBytes);
        return TBN_ERR_DEVICE;
    }
    hipLaunchKernelGGL(kernels[which], persist ? dim3(static_cast<unsigned>(cus)) : grid, dim3(512), kLdsBytes, a.stream,
                       static_cast<const uint16_t *>(a.x), static_cast<uint16_t *>(a.y), a.tile, a.alpha, P);
    return check_launch("tbn_linear_forward (matrix-core kernel with load waves)");
}

}  // namespace tbn
