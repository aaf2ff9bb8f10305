// The final addition of per-block results (binary64) of a reduction launch, for the kernels of
// gact_reduce.hip and gact_kernels.hip.
//
// Order of the additions, the same in every kernel that does them, so that the result does not
// depend on which one a call takes: a row is kRowTerms consecutive results; lane l of the wavefront
// that adds a row takes its terms l, l + 64, ... l + 448 in a tree, then the lanes add up in a
// butterfly.  One wavefront adds the row sums: lane l the rows l, l + 64, ... one after the other,
// then the butterfly again.
//
// Who does it: blocks at the end of the reducing launch itself where the results can be tagged
// (below), else finish_kernel behind it.  A launch of its own starts only when the last block has
// ended, waits for its first loads, and takes the host as long as any other (sensitivity, us a call with
// a second launch and without: 0.4 M fp32 elements 6.8, 4.2; 100 M bf16 64.7, 62.1).
//
// Tagged results.  A block that adds results of the same launch has to know which of them are there.
// A counter would have to start at zero, and the workspace is the caller's and holds anything, so each
// result carries its own proof: two words, the value's bits and the same bits XOR the call's tag, a
// number that no two calls share.  A pair is taken when the XOR of its words is the tag.  Words are
// written and read as single relaxed atomics of device scope (write-through, past the L2s of the
// reader's XCD); no order between them is needed, because a pair of one old and one new word passes
// only if the old word has the value that the new one would have.  What a workspace holds from before
// passes with a probability of 2^-64 per pair.
// The adding blocks have the highest indices of their grid, so that the blocks they wait for have been
// dispatched before them, and those wait for nothing.  The wait is bounded all the same: calls that
// share a workspace and overlap in time, which the interface forbids, overwrite each other's results,
// and the sum is then a NaN and not a kernel that stays.
#ifndef GACT_SUM_H
#define GACT_SUM_H

#include <stdint.h>

#include "gact_device.h"

namespace gact {

constexpr uint32_t kRowTerms = 512;               // eight a lane: their loads are in flight together
constexpr uint32_t kMaxPolls = 1u << 18;          // at about a microsecond each; what is awaited takes some ten

__host__ __device__ constexpr uint32_t rows_of(uint32_t count) { return (count + kRowTerms - 1) / kRowTerms; }

// What a reducing launch needs to add its results itself.  tag 0: they stay as they are, one word each.
struct Finish {
    uint64_t tag;
    double   scale;
    double*  out;                                 // out[0] = scale * sum
    uint32_t blocks;                              // that leave a result; the adding blocks come behind them
};

#ifdef __HIPCC__
__device__ __forceinline__ uint64_t load_word(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_tagged(uint64_t* pair, double v, uint64_t tag) {
    const uint64_t w = __builtin_bit_cast(uint64_t, v);
    __hip_atomic_store(pair, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(pair + 1, w ^ tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// block b's result
__device__ __forceinline__ void put_result(double* partial, uint32_t b, double v, uint64_t tag) {
    if (tag) put_tagged((uint64_t*)partial + 2 * (size_t)b, v, tag);
    else partial[b] = v;
}

// Sum over the wavefront, in all lanes: a butterfly of steps 32, 16, 8, 4, 2, 1.  As register moves (two
// half-wave swaps, then rotations of a row of 16, which are the butterfly's exchanges because after a step
// of s the values repeat every s lanes): through the LDS crossbar the six steps are six round trips, 0.4 us.
template <int CTRL>
__device__ __forceinline__ double row_rotated(double v) {
    const uint64_t w = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)w, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(w >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double add_lanes(double v) {
    typedef uint32_t pair __attribute__((ext_vector_type(2)));
    uint64_t w = __builtin_bit_cast(uint64_t, v);
    pair lo = __builtin_amdgcn_permlane32_swap((uint32_t)w, (uint32_t)w, false, false);
    pair hi = __builtin_amdgcn_permlane32_swap((uint32_t)(w >> 32), (uint32_t)(w >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)hi.x << 32 | lo.x) + __builtin_bit_cast(double, (uint64_t)hi.y << 32 | lo.y);
    w = __builtin_bit_cast(uint64_t, v);
    lo = __builtin_amdgcn_permlane16_swap((uint32_t)w, (uint32_t)w, false, false);
    hi = __builtin_amdgcn_permlane16_swap((uint32_t)(w >> 32), (uint32_t)(w >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)hi.x << 32 | lo.x) + __builtin_bit_cast(double, (uint64_t)hi.y << 32 | lo.y);
    v += row_rotated<0x128>(v);
    v += row_rotated<0x124>(v);
    v += row_rotated<0x122>(v);
    return v + row_rotated<0x121>(v);
}
__device__ __forceinline__ double add_row(const double (&v)[8]) {
    return add_lanes(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])));
}

// Sum of row `row` of `count` tagged results, in all lanes.
__device__ __forceinline__ double tagged_row(const uint64_t* pairs, uint32_t count, uint32_t row, uint64_t tag, int lane) {
    double v[8];
    for (uint32_t polls = 0;; ++polls) {
        bool there = true;
        uint64_t w[8], x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t i = row * kRowTerms + (uint32_t)(k * 64 + lane);
            const uint64_t* p = pairs + 2 * (size_t)(i < count ? i : count - 1);
            w[k] = load_word(p);
            x[k] = load_word(p + 1);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            there = there && (w[k] ^ x[k]) == tag;
            v[k] = row * kRowTerms + (uint32_t)(k * 64 + lane) < count ? __builtin_bit_cast(double, w[k]) : 0.0;
        }
        if (__all(there)) return add_row(v);
        if (polls == kMaxPolls) return __builtin_nan("");
        __builtin_amdgcn_s_sleep(1);
    }
}
__device__ __forceinline__ double plain_row(const double* partial, uint32_t count, uint32_t row, int lane) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t i = row * kRowTerms + (uint32_t)(k * 64 + lane);
        v[k] = partial[i < count ? i : count - 1];
        v[k] = i < count ? v[k] : 0.0;
    }
    return add_row(v);
}

// The rows' sums as lane `lane` of the wavefront that adds them takes them: rows lane, lane + 64, ... in
// [0, end), one after the other onto acc: tagged pairs that other blocks leave in the place of each row's
// first two words.
__device__ __forceinline__ double add_left_rows(double acc, const uint64_t* words, size_t row_words, uint32_t end,
                                                uint64_t tag, int lane) {
    for (uint32_t r = (uint32_t)lane; r < end; r += 64) {
        const uint64_t* p = words + (size_t)r * row_words;
        uint64_t w;
        uint32_t polls = 0;
        while (((w = load_word(p)) ^ load_word(p + 1)) != tag) {
            if (polls++ == kMaxPolls) { w = 0x7FF8000000000000ull; break; }
            __builtin_amdgcn_s_sleep(1);
        }
        acc += __builtin_bit_cast(double, w);
    }
    return acc;
}
// ... rows [first, end) whose sums are in `mine`
__device__ __forceinline__ double add_own_rows(double acc, const double* mine, uint32_t first, uint32_t end, int lane) {
    for (uint32_t r = first + (((uint32_t)lane - first) & 63u); r < end; r += 64) acc += mine[r - first];
    return acc;
}

// Adding block f of adders_for<WAVES>(count): a wavefront adds one row; all blocks but the last leave
// the row's sum behind, the last adds them up.  PAIRS: the results are tagged (else each is one word),
// so that a row has twice as many words.
template <int WAVES>
__host__ __device__ constexpr uint32_t adders_for(uint32_t count) { return (rows_of(count) + WAVES - 1) / WAVES; }

template <int WAVES, bool PAIRS>
__device__ __forceinline__ void finish_block(uint64_t* words, uint32_t count, uint64_t tag, double scale,
                                             double* __restrict__ out, uint32_t f) {
    __shared__ double lds[WAVES];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t rows = rows_of(count), adders = adders_for<WAVES>(count);
    const uint32_t row = f * WAVES + (uint32_t)wave;
    constexpr size_t kRowWords = (PAIRS ? 2 : 1) * (size_t)kRowTerms;
    const bool last = f + 1 == adders;
    // The last block's first wavefront takes what the other blocks leave before it waits for its own
    // row, which is complete later than theirs.
    double acc = 0.0;
    if (last && wave == 0) acc = add_left_rows(acc, words, kRowWords, f * WAVES, ~tag, lane);
    if (row < rows) {
        const double s = PAIRS ? tagged_row(words, count, row, tag, lane) : plain_row((const double*)words, count, row, lane);
        // another tag than the results', one of which was in this place
        if (lane == 0) {
            if (last) lds[wave] = s;
            else put_tagged(words + (size_t)row * kRowWords, s, ~tag);
        }
    }
    if (!last) return;
    __syncthreads();
    if (wave != 0) return;
    const double total = add_lanes(add_own_rows(acc, lds, f * WAVES, rows, lane));
    if (lane == 0) *out = scale * total;
}

// A footprint's sample point: out[1 + j] = element floor(j * n / n_samples) as binary64
__device__ __forceinline__ void sample(const void* x, int dtype, int64_t n, int j, int n_samples, double* __restrict__ out) {
    const int64_t i = (int64_t)(((unsigned __int128)(uint64_t)j * (uint64_t)n) / (uint64_t)n_samples);
    float v;
    if (dtype == GACT_DT_F32) v = ((const float*)x)[i];
    else v = __builtin_bit_cast(float, (uint32_t)((const uint16_t*)x)[i] << 16);
    out[1 + j] = (double)v;
}
#endif  // __HIPCC__

}  // namespace gact

#endif
