// tbn_pack_tile: tile construction (Eq. 1-3) and scalars (Eq. 6, Eq. 7-8) in one pass over
// the real weights.
//
// The flattened weight is viewed as k rows of p entries (Eq. 1).  A thread owns a few tile
// positions i and walks the k rows in ascending order, so its loads of row r are coalesced
// with its neighbours' and each weight is read exactly once.  Column sums s_i (Eq. 2) are kept
// in double precision in row order, which makes the sign (Eq. 3) independent of the launch
// shape and identical to a sequential double-precision sum.  |a| is summed per row in double
// precision: a block reduces its share of row r and writes one partial per (block, r) to the
// workspace; a second small kernel adds the partials in a fixed order and divides (Eq. 6 / 8).
// No floating-point atomics are used, so results are reproducible bit for bit.  A tile of one block
// needs neither workspace nor second kernel (6000 weights, k = 3, three scalars: 5.7 -> 4.0 us as graph replays, 7.5 -> 5.0 in
// calls in a row through the binding).
//
// One kernel for every size, its last block adding the partials, was slower: with a ticket per call 512 blocks wait 15 us
// for each other's operations on one address (30 ns each), with a ticket per 32 blocks the chain of four or five
// device-scope operations takes as long as the second kernel (1,600,000 weights, k = 8: 10.2 -> 11.3 us).
//
// The same kernels build the tile of the column-tiled layout (GPU Inference Kernel section): there the k
// summands of tile position i = o * blk + j are the entries (o, r * blk + j) of an out x in matrix with
// blk = in / k, i.e. summand r of position i sits at (i / blk) * ld + r * blk + i % blk with ld = in.  The flat
// layout of Eq. 1 is the case blk = p (one "row" holds the whole tile).
#include "tbn_common.h"

#include <mutex>
#include <type_traits>

namespace tbn {

constexpr int kPackThreads = 256;
constexpr int kPackWaves = kPackThreads / kWave;
constexpr int kPackQ = 4;  // loads per row per thread, one row at a time; small tiles: one load, kRowsAhead rows at a time
constexpr int kRowsAhead = 4;
constexpr int kMaxRows = 64;   // summands per position whose block sums fit the LDS array; beyond, one partial per wave

template <int VEC> struct PackVec;
template <> struct PackVec<4> { using type = float4; };
template <> struct PackVec<1> { using type = float; };

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ double alpha_denominator(int32_t n_alpha, int64_t p, int32_t k) {
    return n_alpha == 1 ? static_cast<double>(p) * static_cast<double>(k) : static_cast<double>(p);
}

// Q: loads per row per thread; R: rows requested together; BY_BLOCK: a partial per block and row (k <= kMaxRows), else per wave.
// Positions handled by one block: kPackThreads * VEC * Q, a multiple of 64
template <int VEC, bool SEPARATE_A, int Q, int R, bool BY_BLOCK>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(const float *__restrict__ w,
                                                            const float *__restrict__ a, int64_t p, int32_t k,
                                                            int64_t blk, int64_t ld,
                                                            uint32_t *__restrict__ tile_out,
                                                            double *__restrict__ partial, int32_t n_alpha,
                                                            float *__restrict__ alpha_out) {
    __shared__ double row_sum[kPackWaves][BY_BLOCK ? kMaxRows : 1];
    const int64_t n_words = (p + 31) / 32;
    constexpr int64_t kChunk = int64_t(kPackThreads) * VEC;   // positions covered by one load round
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int64_t block_base = int64_t(blockIdx.x) * kChunk * Q;

    double s[Q][VEC];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int v = 0; v < VEC; ++v) s[q][v] = 0.0;

    int64_t pos[Q];   // offset of summand 0 of the thread's positions
    bool live[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = block_base + q * kChunk + int64_t(tid) * VEC;
        live[q] = i < p;  // VEC == 4 is only used when p % 4 == 0: a vector is all in or all out
        pos[q] = (blk == p || !live[q]) ? i : (i / blk) * ld + i % blk;   // blk % 4 == 0 with VEC == 4: no vector spans two rows
    }

    double *my_partial = partial + (int64_t(blockIdx.x) * kPackWaves + wave) * k;

    for (int32_t r0 = 0; r0 < k; r0 += R) {
        float wv[R][Q][VEC];
        float av[R][Q][VEC];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int32_t r = R == 1 || r0 + j < k ? r0 + j : k - 1;   // past the last row: that one again, not added
            const float *wr = w + int64_t(r) * blk;
            const float *ar = SEPARATE_A ? a + int64_t(r) * blk : wr;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (live[q]) {
                    if constexpr (VEC == 4) {
                        const float4 t = *reinterpret_cast<const float4 *>(wr + pos[q]);
                        wv[j][q][0] = t.x; wv[j][q][1] = t.y; wv[j][q][2] = t.z; wv[j][q][3] = t.w;
                        if constexpr (SEPARATE_A) {
                            const float4 u = *reinterpret_cast<const float4 *>(ar + pos[q]);
                            av[j][q][0] = u.x; av[j][q][1] = u.y; av[j][q][2] = u.z; av[j][q][3] = u.w;
                        }
                    } else {
                        wv[j][q][0] = wr[pos[q]];
                        if constexpr (SEPARATE_A) av[j][q][0] = ar[pos[q]];
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) { wv[j][q][v] = 0.f; av[j][q][v] = 0.f; }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (R > 1 && r0 + j >= k) break;
            double l1 = 0.0;
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    s[q][v] += static_cast<double>(wv[j][q][v]);
                    l1 += static_cast<double>(fabsf(SEPARATE_A ? av[j][q][v] : wv[j][q][v]));
                }
            l1 = wave_sum_f64(l1);
            if (lane == 0) {
                if constexpr (BY_BLOCK) row_sum[wave][r0 + j] = l1;
                else my_partial[r0 + j] = l1;
            }
        }
    }

    // Eq. 3 and bit packing, LSB first
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if constexpr (VEC == 4) {
            uint32_t nib = 0;
#pragma unroll
            for (int v = 0; v < 4; ++v) nib |= (s[q][v] > 0.0 ? 1u : 0u) << v;
            uint32_t word = nib << (4 * (lane & 7));
            word |= __shfl_xor(word, 1, kWave);
            word |= __shfl_xor(word, 2, kWave);
            word |= __shfl_xor(word, 4, kWave);
            const int64_t wi = (block_base + q * kChunk + int64_t(tid & ~7) * 4) >> 5;
            if ((lane & 7) == 0 && wi < n_words) tile_out[wi] = word;
        } else {
            const unsigned long long mask = __ballot(s[q][0] > 0.0);
            const int64_t wi = (block_base + q * kChunk + int64_t(wave) * kWave) >> 5;
            if (lane == 0 && wi < n_words) tile_out[wi] = static_cast<uint32_t>(mask);
            if (lane == 1 && wi + 1 < n_words) tile_out[wi + 1] = static_cast<uint32_t>(mask >> 32);
        }
    }

    if constexpr (BY_BLOCK) {
        __syncthreads();
        double sum = 0.0;
        if (tid < k) {
#pragma unroll
            for (int wv = 0; wv < kPackWaves; ++wv) sum += row_sum[wv][tid];
        }
        if (gridDim.x > 1) {
            if (tid < k) partial[int64_t(blockIdx.x) * k + tid] = sum;
        } else if (wave == 0) {   // (k <= 64)
            const double all = n_alpha == 1 ? wave_sum_f64(sum) : sum;
            if (tid < n_alpha) alpha_out[tid] = static_cast<float>(all / alpha_denominator(n_alpha, p, k));
        }
    }
}

// alpha[r] = (sum over the n_part partials of row r) / p, or one alpha = total / n: then all partials, which lie side by side,
// are one row.  One block per output scalar; fixed strided order + fixed tree -> reproducible.  (With one alpha, 256 threads
// going through the rows one after the other took as long as the tile kernel, graph replays: 4096 x 4096, k = 8 18.2 us in all
// instead of 14.9; 64 million weights, k = 16: 87 instead of 51.)
constexpr int kAlphaThreads = 1024;   // 256 for few partials
__global__ __launch_bounds__(kAlphaThreads) void pack_alpha_kernel(const double *__restrict__ partial, int64_t n_part,
                                                                   int32_t k, int32_t n_alpha, int64_t p,
                                                                   float *__restrict__ alpha_out) {
    __shared__ double red[kAlphaThreads / kWave];
    const int tid = threadIdx.x;
    const int64_t stride = n_alpha == 1 ? 1 : k, n = n_alpha == 1 ? n_part * k : n_part;
    const double *src = partial + blockIdx.x;
    double acc = 0.0;
    const int64_t T = blockDim.x;
    int64_t i = tid;
    for (; i + 3 * T < n; i += 4 * T) {   // four independent loads in flight
        double t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = src[(i + j * T) * stride];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += t[j];
    }
    for (; i < n; i += T) acc += src[i * stride];
    acc = wave_sum_f64(acc);
    if ((tid & (kWave - 1)) == 0) red[tid / kWave] = acc;
    __syncthreads();
    if (tid == 0) {
        double total = 0.0;
        for (int wv = 0; wv < static_cast<int>(T / kWave); ++wv) total += red[wv];
        alpha_out[blockIdx.x] = static_cast<float>(total / alpha_denominator(n_alpha, p, k));
    }
}

static int64_t pack_blocks(int64_t p, int vec, int q = kPackQ) {
    const int64_t per_block = int64_t(kPackThreads) * vec * q;
    return (p + per_block - 1) / per_block;
}

size_t pack_workspace_bytes(int64_t n, int32_t k, int32_t /*n_alpha*/) {
    // sized for the scalar-load variant (the larger grid) so the choice of variant, which
    // depends on pointer alignment, never changes the requirement
    const int64_t p = n / k;
    return static_cast<size_t>(pack_blocks(p, 1) * kPackWaves * k) * sizeof(double);
}

tbn_status launch_pack(const float *w, const float *a, int64_t n, int32_t k, int32_t n_alpha,
                       uint32_t *tile_out, float *alpha_out, void *workspace, hipStream_t stream,
                       int64_t blk, int64_t ld) {
    const int64_t p = n / k;
    if (blk <= 0) { blk = p; ld = 0; }   // flat layout
    const bool vec4 = (p % 4 == 0) && (blk % 4 == 0) && (ld % 4 == 0) && ((reinterpret_cast<uintptr_t>(w) & 15u) == 0) &&
                      (!a || (reinterpret_cast<uintptr_t>(a) & 15u) == 0);
    // Up to 192 blocks of four loads per row a thread takes one load of four rows at a time: as many bytes in flight, four times
    // the blocks (graph replays: 49 blocks, k = 8 9.6 -> 7.2 us; 13 blocks, k = 16 14.8 -> 9.8; 98 blocks, k = 8 9.9 -> 7.9; but 245
    // blocks, k = 4 7.3 -> 7.9).  With fewer than four rows some of these loads are idle, and with scalar loads the second kernel has four
    // times the partials of fewer weights to add: there up to 128 blocks below eight rows (141 - 190 blocks, k = 3 / 5: 5.8 -> 6.1, 7.1 -> 7.5; 128 blocks:
    // 5.7 -> 5.5, 6.8 -> 6.5), never with one row, and with one row and vector loads up to 96 (183: 5.3 -> 5.5; 72: 5.0).  One row and scalar
    // loads: with 2 - 128 blocks what a partial per block waits for costs more than it saves (12 - 50 blocks 4.4 -> 4.9; 170: level).
    // With a partial per block (64 rows or fewer) the small form's partials still fit the workspace.
    const int64_t large_blocks = pack_blocks(p, vec4 ? 4 : 1), most = vec4 ? (k == 1 ? 96 : 192) : k >= 8 ? 192 : k >= 2 ? 128 : 0;
    const bool by_block = k <= kMaxRows && !(k == 1 && !vec4 && large_blocks > 1 && large_blocks <= 128);
    const bool small = by_block && large_blocks > 1 && large_blocks <= most;
    const int64_t blocks = pack_blocks(p, vec4 ? 4 : 1, small ? 1 : kPackQ);
    if (blocks > 0x7fffffffLL) {
        set_error("tbn_pack_tile: tile of %lld bits is beyond the supported range", (long long)p);
        return TBN_ERR_UNSUPPORTED;
    }
    double *partial = static_cast<double *>(workspace);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kPackThreads), 0, stream, w, a, p, k, blk, ld, tile_out,
                           partial, n_alpha, alpha_out);
    };
    auto pick = [&](auto vec, auto separate) {
        constexpr int V = decltype(vec)::value;
        constexpr bool A = decltype(separate)::value;
        if (small) launch(&pack_kernel<V, A, 1, kRowsAhead, true>);
        else if (by_block) launch(&pack_kernel<V, A, kPackQ, 1, true>);
        else launch(&pack_kernel<V, A, kPackQ, 1, false>);
    };
    if (vec4) {
        if (a) pick(std::integral_constant<int, 4>{}, std::true_type{});
        else   pick(std::integral_constant<int, 4>{}, std::false_type{});
    } else {
        if (a) pick(std::integral_constant<int, 1>{}, std::true_type{});
        else   pick(std::integral_constant<int, 1>{}, std::false_type{});
    }
    tbn_status st = check_launch("tbn_pack_tile (tile kernel)");
    if (st != TBN_OK || (by_block && blocks == 1)) return st;   // (one block has written the scalars)
    const int64_t n_part = by_block ? blocks : blocks * kPackWaves;
    hipLaunchKernelGGL(pack_alpha_kernel, dim3(static_cast<unsigned>(n_alpha)), dim3((n_alpha == 1 ? n_part * k : n_part) > 1024 ? kAlphaThreads : 256), 0,
                       stream, partial, n_part, k, n_alpha, p, alpha_out);
    return check_launch("tbn_pack_tile (alpha kernel)");
}

// ---- tbn_pack_tile_noalloc: the same two kernels with the partial sums in a file-scope device array ----------
// Every GPU the library runs on holds its own copy of the array at its own address until the process ends.  In
// host code the array's name is only a stand-in for the symbol: the device address is looked up once per device,
// with that device current, and that pointer is what the kernels and every other use get.
static __device__ __align__(256) unsigned char scratch[TBN_PACK_NOALLOC_SCRATCH_BYTES];

static tbn_status pack_scratch_address(void **out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *address[kMaxDevices] = {};
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess || device < 0 || device >= kMaxDevices) {
        set_error("tbn_pack_tile_noalloc: cannot identify the current device: %s",
                  e != hipSuccess ? hipGetErrorString(e) : "device index out of range");
        return TBN_ERR_DEVICE;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!address[device]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            set_error("tbn_pack_tile_noalloc: cannot resolve the scratch array on device %d: %s", device,
                      hipGetErrorString(e));
            return TBN_ERR_DEVICE;
        }
        address[device] = ptr;
    }
    *out = address[device];
    return TBN_OK;
}

tbn_status launch_pack_noalloc(const float *w, const float *a, int64_t n, int32_t k, int32_t n_alpha,
                               uint32_t *tile_out, float *alpha_out, hipStream_t stream) {
    const size_t need = pack_workspace_bytes(n, k, n_alpha);
    if (need > sizeof(scratch)) {
        set_error("tbn_pack_tile_noalloc: these sizes need %zu bytes of scratch memory, the built-in array holds %zu; "
                  "use tbn_pack_tile with a workspace", need, sizeof(scratch));
        return TBN_ERR_UNSUPPORTED;
    }
    void *ptr = nullptr;
    tbn_status st = pack_scratch_address(&ptr);
    if (st != TBN_OK) return st;
    // nothing in the array has to start at zero: every partial sum that the second kernel reads is written by
    // the first one of the same call
    return launch_pack(w, a, n, k, n_alpha, tile_out, alpha_out, ptr, stream);
}

}  // namespace tbn
