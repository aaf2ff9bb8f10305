// Sensitivity reduction of GACT's Alg. 1 (arXiv 2206.11357, Sec. 4.2) and the
// running gradient statistics behind its variance alert, for MI355X (gfx950).
//
// Both are multi-buffer streaming reductions bound by HBM: a block of 512
// threads takes 16 KB of each buffer it only reads with two coalesced 16-byte
// loads per thread, accumulates in binary64 per thread, reduces over the block,
// and leaves one result per block; the results are added in a fixed order
// (gact_sum.h), so that the sum does not depend on scheduling.
// Two pieces per thread: four, with 256 threads for the same 16 KB, keep 59 to 81
// registers and wait longer for the last of them.  Us on 302 M parameters, 312
// buffers, threads x pieces:            256 x 4   512 x 2   512 x 3   512 x 4   1024 x 1
//   sensitivity, fp32                     362       356       357       362       409
//   statistics, fp32                      610       600       628       628       670
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gact_device.h"
#include "gact_sum.h"

namespace gact {

typedef uint32_t u4r __attribute__((ext_vector_type(4)));
typedef uint32_t u2r __attribute__((ext_vector_type(2)));
typedef float    f4r __attribute__((ext_vector_type(4)));

constexpr int kRedWaves = kReduceWaves, kRedThreads = 64 * kRedWaves;
constexpr int kPieces = 2;              // per thread and buffer
// A statistics chunk is two pieces of four elements per thread, or one of twice as many threads (stats_chunk).
constexpr int stats_pieces(bool wide) { return wide ? 1 : kPieces; }
static_assert(stats_threads(false) == kRedThreads && kStatsChunkElems == stats_threads(false) * stats_pieces(false) * 4 &&
              kStatsChunkElems == stats_threads(true) * stats_pieces(true) * 4, "the elements of a statistics chunk");
static_assert(reduce_chunk_elems(GACT_DT_F32) == kRedThreads * kPieces * 4 &&
              reduce_chunk_elems(GACT_DT_BF16) == kRedThreads * kPieces * 8, "two pieces of 16 bytes per thread");

// Sums over the block of N values a thread, valid in thread 0.  One barrier, behind which all
// wavefronts but the first end: with a barrier on either side of each sum and the wavefronts' sums through
// the LDS crossbar, sensitivity of 302 M fp32 elements took 351 us a call, now 343.
template <int WAVES, int N>
__device__ __forceinline__ void block_sums(double (&v)[N]) {
    static_assert((WAVES & (WAVES - 1)) == 0, "the tree below");
    __shared__ double part[N][WAVES];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = add_lanes(v[j]);
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) part[j][wave] = v[j];
    }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double s[WAVES];
#pragma unroll
        for (int i = 0; i < WAVES; ++i) s[i] = part[j][i];
#pragma unroll
        for (int m = WAVES / 2; m > 0; m /= 2)
#pragma unroll
            for (int i = 0; i < m; ++i) s[i] = s[2 * i] + s[2 * i + 1];
        v[j] = s[0];
    }
}

__device__ __forceinline__ int find_buffer(const uint32_t* first_block, int K, uint32_t b) {
    int lo = 0, hi = K;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first_block[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// eight fp32 values of a 16-byte piece of bf16, or four of fp32 (rest unused)
template <int DT>
__device__ __forceinline__ void unpack_piece(const u4r w, float v[8]) {
    // components are copied to scalars first: a bit cast applied directly to a
    // vector component reads component 0
    const uint32_t c0 = w.x, c1 = w.y, c2 = w.z, c3 = w.w;
    if (DT == GACT_DT_F32) {
        v[0] = __builtin_bit_cast(float, c0); v[1] = __builtin_bit_cast(float, c1);
        v[2] = __builtin_bit_cast(float, c2); v[3] = __builtin_bit_cast(float, c3);
    } else {
        v[0] = __builtin_bit_cast(float, c0 << 16); v[1] = __builtin_bit_cast(float, c0 & 0xFFFF0000u);
        v[2] = __builtin_bit_cast(float, c1 << 16); v[3] = __builtin_bit_cast(float, c1 & 0xFFFF0000u);
        v[4] = __builtin_bit_cast(float, c2 << 16); v[5] = __builtin_bit_cast(float, c2 & 0xFFFF0000u);
        v[6] = __builtin_bit_cast(float, c3 << 16); v[7] = __builtin_bit_cast(float, c3 & 0xFFFF0000u);
    }
}

// One 16-byte piece starting at element e of a buffer with n elements; pieces
// that cross the end are read element by element and padded with zeros.
template <int DT, bool FULL = false>
__device__ __forceinline__ u4r load_piece16(const void* base, int64_t e, int64_t n) {
    constexpr int P = DT == GACT_DT_F32 ? 4 : 8;
    u4r w = {0u, 0u, 0u, 0u};
    if (FULL || e + P <= n) {
        if (DT == GACT_DT_F32) w = __builtin_nontemporal_load((const u4r*)((const uint32_t*)base + e));
        else w = __builtin_nontemporal_load((const u4r*)((const uint16_t*)base + e));
    } else if (e < n) {
        uint32_t t[4] = {0u, 0u, 0u, 0u};
        if (DT == GACT_DT_F32) {
            for (int j = 0; j < P; ++j) if (e + j < n) t[j] = ((const uint32_t*)base)[e + j];
        } else {
            for (int j = 0; j < P; ++j)
                if (e + j < n) t[j >> 1] |= (uint32_t)((const uint16_t*)base)[e + j] << (16 * (j & 1));
        }
        w.x = t[0]; w.y = t[1]; w.z = t[2]; w.w = t[3];
    }
    return w;
}

// ------------------------------------------------------------- sensitivity
// FULL: the whole chunk lies inside the buffer, so all loads are unguarded and
// issued back to back.
template <int DT, bool FULL>
__device__ __forceinline__ double diff_sq_chunk(const ReduceArgs& r, int64_t chunk, const Finish& fin, uint64_t& first_word) {
    constexpr int P = DT == GACT_DT_F32 ? 4 : 8;
    const int64_t e0 = chunk * (int64_t)(kRedThreads * kPieces * P) + (int64_t)threadIdx.x * P;
    u4r a[kPieces], b[kPieces];
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int64_t e = e0 + (int64_t)k * kRedThreads * P;
        a[k] = load_piece16<DT, FULL>(r.a, e, r.n);
        b[k] = load_piece16<DT, FULL>(r.b, e, r.n);
    }
    if (threadIdx.x < 64) first_word = result_word(fin);       // behind the others' loads, in nobody's way
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        float x[8], y[8];
        unpack_piece<DT>(a[k], x);
        unpack_piece<DT>(b[k], y);
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const double d = (double)x[j] - (double)y[j];
            acc += d * d;
        }
    }
    return acc;
}

__device__ __forceinline__ void diff_sq_block(const ReduceArgs& r, int64_t chunk, uint32_t place, double* partial,
                                              const Finish& fin) {
    uint64_t first_word = 0;
    const bool full = (chunk + 1) * reduce_chunk_elems(r.dtype) <= r.n;
    double acc;
    if (r.dtype == GACT_DT_F32)
        acc = full ? diff_sq_chunk<GACT_DT_F32, true>(r, chunk, fin, first_word) : diff_sq_chunk<GACT_DT_F32, false>(r, chunk, fin, first_word);
    else
        acc = full ? diff_sq_chunk<GACT_DT_BF16, true>(r, chunk, fin, first_word) : diff_sq_chunk<GACT_DT_BF16, false>(r, chunk, fin, first_word);
    double sum[1] = {acc};
    block_sums<kRedWaves>(sum);
    if (threadIdx.x < 64) put_result<kRedWaves>(partial, place, sum[0], fin, first_word, (int)threadIdx.x);
}

// Table in device memory (uploaded to the caller's workspace): any number of buffers.
__global__ __launch_bounds__(kRedThreads) void diff_sq_kernel(const ReduceArgs* __restrict__ table,
                                                              const uint32_t* __restrict__ first_block,
                                                              int K, double* partial, Finish fin) {
    const uint32_t place = blockIdx.x - fin.ahead;
    if (place >= fin.blocks) {
        finish_block<kRedWaves, true>((uint64_t*)partial, fin, adding_block(fin, blockIdx.x));
        return;
    }
    const uint32_t b = ordered_block(place, runs_end(fin.blocks, kDiffRunShift), kDiffRunShift);
    const int k = find_buffer(first_block, K, b);
    const ReduceArgs r = table[k];
    diff_sq_block(r, (int64_t)(b - first_block[k]), place, partial, fin);
}

// Table by value in the kernel arguments: no upload, which takes the stream 5 us
// ahead of the kernel (96 bf16 pairs of 101 M elements: 67.8 us with, 65.6 us without).
__global__ __launch_bounds__(kRedThreads) void diff_sq_inline_kernel(ReduceTable tab, int K,
                                                                     double* partial, Finish fin) {
    const uint32_t place = blockIdx.x - fin.ahead;
    if (place >= fin.blocks) {
        finish_block<kRedWaves, true>((uint64_t*)partial, fin, adding_block(fin, blockIdx.x));
        return;
    }
    const uint32_t b = ordered_block(place, runs_end(fin.blocks, kDiffRunShift), kDiffRunShift);
    const int k = find_buffer(tab.first_block, K, b);
    diff_sq_block(tab.t[k], (int64_t)(b - tab.first_block[k]), place, partial, fin);
}

// ---------------------------------------------------------------- footprint
template <int DT, bool FULL>
__device__ __forceinline__ double sum_chunk(const ReduceArgs& r, int64_t chunk) {
    constexpr int P = DT == GACT_DT_F32 ? 4 : 8;
    const int64_t e0 = chunk * (int64_t)(kRedThreads * kPieces * P) + (int64_t)threadIdx.x * P;
    u4r a[kPieces];
#pragma unroll
    for (int k = 0; k < kPieces; ++k)
        a[k] = load_piece16<DT, FULL>(r.a, e0 + (int64_t)k * kRedThreads * P, r.n);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        float x[8];
        unpack_piece<DT>(a[k], x);      // elements past n were loaded as 0
#pragma unroll
        for (int j = 0; j < P; ++j) acc += (double)x[j];
    }
    return acc;
}

// one buffer; block b takes chunk b
__global__ __launch_bounds__(kRedThreads) void sum_kernel(ReduceArgs r, double* __restrict__ partial) {
    const int64_t chunk = (int64_t)blockIdx.x;
    const bool full = (chunk + 1) * reduce_chunk_elems(r.dtype) <= r.n;
    double acc;
    if (r.dtype == GACT_DT_F32)
        acc = full ? sum_chunk<GACT_DT_F32, true>(r, chunk) : sum_chunk<GACT_DT_F32, false>(r, chunk);
    else
        acc = full ? sum_chunk<GACT_DT_BF16, true>(r, chunk) : sum_chunk<GACT_DT_BF16, false>(r, chunk);
    double sum[1] = {acc};
    block_sums<kRedWaves>(sum);
    if (threadIdx.x == 0) partial[blockIdx.x] = sum[0];
}

// ------------------------------------------------------- gradient statistics
// Four elements of a bf16 buffer from element e on, as load_piece16 (in the low half).
template <bool FULL>
__device__ __forceinline__ u4r load_bf16x4(const void* base, int64_t e, int64_t n) {
    const uint16_t* p = (const uint16_t*)base + e;
    u4r w = {0u, 0u, 0u, 0u};
    if (FULL || e + 4 <= n) {
        const u2r h = __builtin_nontemporal_load((const u2r*)p);
        w.x = h.x; w.y = h.y;
    } else if (e < n) {
        uint32_t t[2] = {0u, 0u};
        for (int j = 0; j < 4; ++j) if (e + j < n) t[j >> 1] |= (uint32_t)p[j] << (16 * (j & 1));
        w.x = t[0]; w.y = t[1];
    }
    return w;
}

// A piece is four elements for both types of gradient, so that neighbouring lanes read and write
// neighbouring 16 bytes of the mean.  (With 16 bytes of a bf16 gradient per lane, every lane had two
// 16-byte pieces of the mean 32 bytes from the next lane's, loads and stores of half lines: 764 us for
// 302 M parameters, 312 buffers, now 472 us, 6.4 TB/s.)
//
// WIDE: one piece a thread, blocks of 1024, the mean written through the L2 (non-temporal, device scope).  A
// wavefront's stores are then one burst of 1 KB a block, which HBM takes better beside two streams of
// reads, but the block's sum is a larger part of its life.  Us, fp32, hidden width and parameters:
//               1024, 302 M   768, 170 M   1024, 101 M   1024, 50 M   768, 28 M   384, 2.4 M   1000, 360 M
//   512 x 2         581           325          194          98.0         57.2         11.0          693
//   1024 x 1        552           315          188          97.0         57.4         11.6          707
// So it is for launches of kWideStats blocks and more (stage_reduction), and only where every mean starts
// on a line: in the last column most do not, and a line that two wavefronts write leaves in two parts.  bf16
// gradients, half the bytes for as much to add up: 1024 x 1 takes 507 us on 302 M parameters, 512 x 2 472.
template <int DT, bool FULL, bool WIDE>
__device__ __forceinline__ void stats_chunk(const ReduceArgs& r, int64_t chunk, float rt,
                                            double& sg2, double& sm2) {
    constexpr int T = stats_threads(WIDE), P = stats_pieces(WIDE);
    const int64_t e0 = chunk * kStatsChunkElems + (int64_t)threadIdx.x * 4;
    float* mean = (float*)r.b;
    u4r g[P];
    f4r m[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int64_t e = e0 + (int64_t)k * T * 4;
        if (DT == GACT_DT_F32) g[k] = load_piece16<GACT_DT_F32, FULL>(r.a, e, r.n);
        else g[k] = load_bf16x4<FULL>(r.a, e, r.n);
        m[k] = __builtin_bit_cast(f4r, load_piece16<GACT_DT_F32, FULL>(mean, e, r.n));
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int64_t e = e0 + (int64_t)k * T * 4;
        float x[8];
        unpack_piece<DT>(g[k], x);
        const float old[4] = {m[k].x, m[k].y, m[k].z, m[k].w};
        float nw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float gi = x[j];
            const float d = gi - old[j];
            const float s = d * rt;
            nw[j] = old[j] + s;
            if (FULL || e + j < r.n) {
                sg2 += (double)gi * (double)gi;
                sm2 += (double)nw[j] * (double)nw[j];
            }
        }
        const f4r o = {nw[0], nw[1], nw[2], nw[3]};
        if (FULL && WIDE) {
            // The offset is the lanes' own and there is no scalar one: with a scalar offset the compiler
            // leaves out the wait states between such a store and the next write to its data registers.
            constexpr int kBytes = (int)kStatsChunkElems * 4, kThrough = 2 | 16;      // nt, sc1
            const __amdgpu_buffer_rsrc_t span =
                __builtin_amdgcn_make_buffer_rsrc(mean + chunk * kStatsChunkElems, 0, kBytes, 0x00027000);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4r, o), span, (int)threadIdx.x * 16, 0, kThrough);
        } else if (FULL || e + 4 <= r.n) {
            __builtin_nontemporal_store(o, (f4r*)(mean + e));
        } else {
            for (int j = 0; j < 4; ++j) if (e + j < r.n) mean[e + j] = nw[j];
        }
    }
}

// bf16_chunks: how many chunks of a bf16 buffer this launch's blocks take (stats_block_elems)
template <bool WIDE>
__device__ __forceinline__ void grad_stats_block(const ReduceArgs& r, int64_t block, float rt, int bf16_chunks,
                                                 uint32_t blocks, double* __restrict__ partial) {
    const uint32_t b = blockIdx.x;
    double sg2 = 0.0, sm2 = 0.0;
    if (WIDE || r.dtype == GACT_DT_F32) {
        if ((block + 1) * kStatsChunkElems <= r.n) stats_chunk<GACT_DT_F32, true, WIDE>(r, block, rt, sg2, sm2);
        else stats_chunk<GACT_DT_F32, false, WIDE>(r, block, rt, sg2, sm2);
    } else {
        int64_t chunk = block * bf16_chunks;
#pragma unroll 1
        for (const int64_t end = chunk + bf16_chunks; chunk < end; ++chunk) {
            if ((chunk + 1) * kStatsChunkElems <= r.n) stats_chunk<GACT_DT_BF16, true, false>(r, chunk, rt, sg2, sm2);
            else stats_chunk<GACT_DT_BF16, false, false>(r, chunk, rt, sg2, sm2);
        }
    }
    // The block keeps its place until its stores are acknowledged: the fewer are under way, the better the
    // memory takes them beside the reads (us, 302 M parameters: fp32 589 without, 580 with; bf16 478, 468;
    // WIDE 552 without, 571 with).  Not in short launches (kShortStats).
    if (!WIDE && blocks >= kShortStats) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    double sum[2] = {sg2, sm2};
    block_sums<stats_threads(WIDE) / 64>(sum);
    if (threadIdx.x == 0) { partial[b] = sum[0]; partial[blocks + b] = sum[1]; }
}

template <bool WIDE>
__global__ __launch_bounds__(stats_threads(WIDE)) void grad_stats_kernel(const ReduceArgs* __restrict__ table,
                                                                         const uint32_t* __restrict__ first_block,
                                                                         int K, float rt, int bf16_chunks, uint32_t blocks,
                                                                         double* __restrict__ partial) {
    const uint32_t b = ordered_block(blockIdx.x, stats_runs_end(blocks, WIDE), kStatsRunShift);
    const int k = find_buffer(first_block, K, b);
    const ReduceArgs r = table[k];
    grad_stats_block<WIDE>(r, (int64_t)(b - first_block[k]), rt, bf16_chunks, blocks, partial);
}

template <bool WIDE>
__global__ __launch_bounds__(stats_threads(WIDE)) void grad_stats_inline_kernel(ReduceTable tab, int K, float rt,
                                                                                int bf16_chunks, uint32_t blocks,
                                                                                double* __restrict__ partial) {
    const uint32_t b = ordered_block(blockIdx.x, stats_runs_end(blocks, WIDE), kStatsRunShift);
    const int k = find_buffer(tab.first_block, K, b);
    grad_stats_block<WIDE>(tab.t[k], (int64_t)(b - tab.first_block[k]), rt, bf16_chunks, blocks, partial);
}

// ------------------------------------------------------------ final addition
// out[j] = scale * (sum of the `count` results of output j, out_pitch apart), in the order of gact_sum.h,
// where the reducing launch has not added them itself.  Up to kFinRows rows by one block of 1024 threads;
// more by a block for every 16 rows, of which the last adds up what the others leave (before, a kernel
// of its own brought such lists down to 128 results: 73,926 pairs took 12 us, now 6).
// Blocks from `adders` on take a footprint's sample points, 1024 a block: they are
// a few loads, and a kernel of their own took 4.5 us of a footprint's 47 on 51 M
// fp32 elements.
constexpr int kFinThreads = 1024, kFinWaves = kFinThreads / 64;
constexpr uint32_t kFinRows = 4 * kFinWaves;
__global__ __launch_bounds__(kFinThreads) void finish_kernel(double* partial, uint32_t adders, size_t out_pitch,
                                                             Finish fin, ReduceArgs r, int n_samples) {
    __shared__ double lds[kFinRows];
    const uint32_t f = blockIdx.x;
    if (f >= adders) {
        const int j = (int)((f - adders) * kFinThreads + threadIdx.x);
        if (j < n_samples) sample(r.a, r.dtype, r.n, j, n_samples, fin.out);
        return;
    }
    double* p = partial + (size_t)blockIdx.y * out_pitch;
    fin.out += blockIdx.y;
    if (adders > 1) {
        finish_block<kFinWaves, false>((uint64_t*)p, fin, f);
        return;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t rows = rows_of(fin.blocks);
    for (uint32_t row = (uint32_t)wave; row < rows; row += kFinWaves) {
        const double s = plain_row(p, fin.blocks, row, lane);
        if (lane == 0) lds[row] = s;
    }
    __syncthreads();
    if (wave != 0) return;
    const double total = add_lanes(add_own_rows(0.0, lds, 0, rows, lane));
    if (lane == 0) *fin.out = fin.scale * total;
}

// out[0 .. nout) = 0
__global__ void zero_kernel(double* __restrict__ out, int nout) {
    const int j = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (j < nout) out[j] = 0.0;
}

// Enqueues the final addition of `count` terms for each of `nout` outputs, and the sample points of r.
static void launch_finish(double* d_partial, unsigned count, int nout, uint64_t tag, double scale, double* d_out,
                          hipStream_t s, const ReduceArgs& r = ReduceArgs{}, int n_samples = 0,
                          const Late* late = nullptr) {
    const uint32_t adders = rows_of(count) <= kFinRows ? 1u : adders_for<kFinWaves>(count);
    const dim3 grid(adders + (n_samples + kFinThreads - 1) / kFinThreads, nout);
    hipLaunchKernelGGL(finish_kernel, grid, dim3(kFinThreads), 0, s, d_partial, adders, (size_t)count,
                       finish_of(tag, scale, d_out, count, 0, late), r, n_samples);
}

}  // namespace gact

extern "C" int gact_launch_diff_sq(const gact::ReduceTable* inline_table, const gact::ReduceArgs* d_table,
                                   const uint32_t* d_first, int K, unsigned blocks, double* d_partial, int tagged,
                                   uint64_t tag, double scale, double* d_out, void* stream, const gact::Late* late) {
    hipStream_t s = (hipStream_t)stream;
    const uint32_t adders = tagged ? gact::adders_for<gact::kRedWaves>(blocks) : 0;
    const gact::Finish fin = gact::finish_of(tagged ? tag : 0, scale, d_out, blocks, adders, late);
    const dim3 grid(blocks + adders);
    if (inline_table)
        hipLaunchKernelGGL(gact::diff_sq_inline_kernel, grid, dim3(gact::kRedThreads), 0, s, *inline_table,
                           K, d_partial, fin);
    else
        hipLaunchKernelGGL(gact::diff_sq_kernel, grid, dim3(gact::kRedThreads), 0, s, d_table, d_first,
                           K, d_partial, fin);
    if (hipGetLastError() != hipSuccess) return -1;       // no addition of what nothing leaves
    if (!tagged) gact::launch_finish(d_partial, blocks, 1, tag, scale, d_out, s);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <bool WIDE>
static void launch_stats(const gact::ReduceTable* inline_table, const gact::ReduceArgs* d_table, const uint32_t* d_first,
                         int K, float rt, int bf16_chunks, unsigned blocks, double* d_partial, hipStream_t s) {
    const dim3 grid(blocks), block(gact::stats_threads(WIDE));
    if (inline_table)
        hipLaunchKernelGGL(gact::grad_stats_inline_kernel<WIDE>, grid, block, 0, s, *inline_table, K, rt, bf16_chunks,
                           blocks, d_partial);
    else
        hipLaunchKernelGGL(gact::grad_stats_kernel<WIDE>, grid, block, 0, s, d_table, d_first, K, rt, bf16_chunks,
                           blocks, d_partial);
}

extern "C" int gact_launch_grad_stats(const gact::ReduceTable* inline_table, const gact::ReduceArgs* d_table,
                                      const uint32_t* d_first, int K, float rt, int bf16_chunks, int wide, unsigned blocks,
                                      double* d_partial, uint64_t tag, double* d_out, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (wide) launch_stats<true>(inline_table, d_table, d_first, K, rt, bf16_chunks, blocks, d_partial, s);
    else launch_stats<false>(inline_table, d_table, d_first, K, rt, bf16_chunks, blocks, d_partial, s);
    if (hipGetLastError() != hipSuccess) return -1;
    gact::launch_finish(d_partial, blocks, 2, tag, 1.0, d_out, s);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// out[0 .. nout) = 0 through a kernel (no memset node, so callers may capture it)
extern "C" int gact_launch_zero(double* d_out, int nout, void* stream) {
    hipLaunchKernelGGL(gact::zero_kernel, dim3((nout + 255) / 256), dim3(256), 0, (hipStream_t)stream, d_out, nout);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// The footprint from per-block sums that a compress launch left in d_partial.
extern "C" int gact_launch_footprint_finish(const gact::ReduceArgs* r, unsigned count, double* d_partial, uint64_t tag,
                                            int n_samples, double* d_out, void* stream) {
    gact::launch_finish(d_partial, count, 1, tag, 1.0, d_out, (hipStream_t)stream, *r, n_samples);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

extern "C" int gact_launch_footprint(const gact::ReduceArgs* r, unsigned blocks, double* d_partial, uint64_t tag,
                                     int n_samples, double* d_out, void* stream, const gact::Late* late) {
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(gact::sum_kernel, dim3(blocks), dim3(gact::kRedThreads), 0, s, *r, d_partial);
    if (hipGetLastError() != hipSuccess) return -1;
    gact::launch_finish(d_partial, blocks, 1, tag, 1.0, d_out, s, *r, n_samples, late);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
