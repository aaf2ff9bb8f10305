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
//
// No result depends on how long another stream's kernel takes.  The adding blocks have the highest indices
// of their grid and wait for blocks that wait for nothing, but each XCD starts its share of a grid by itself:
// an adding block of one can run while the blocks that it waits for stand behind another stream's kernel on
// another XCD, for as long as that kernel likes.  So the last adding block leaves a mark in the place of the
// result when its patience ends (given_up), and every block looks for the mark when its loads are out.
//   * A block that finds it leaves its result, waits until the result is in memory, and then adds up
//     everything itself if everything is there (try_finish, in the order that the adding blocks have): the
//     last such block finds all that the others have left.
//   * A block that does not find it was running before the mark was there.  It has some microseconds of work,
//     for which the adding block goes on looking kGrace times, a second and more of its own running time; at
//     the end of that it tries to finish too.
// Every wait is thus bounded, and the result is the sum whichever block ends last.  Only calls that share a
// workspace and overlap in time, which the interface forbids, can leave the mark, a NaN.
// What the look costs, us a call without and with it: sensitivity, bf16, 101 M elements 62.4, 61.6, 302 M 176.5,
// 174.0, fp32, 6 M 11.1, 11.4, 302 M 341.5, 342.1; compressor with a footprint, fp32, 1 M 4.7, 4.9, 51 M 38.5, 38.8,
// 200 M 135.0, 134.4.  As the block's first load, which its other loads then queue behind: 62.8, 176.9, 11.4, 341.6;
// 5.1, 39.0, 134.1.  Behind every result, with a wait until that is in memory, and so without any grace: 62.8, 177.1,
// 11.5, 342.4; 5.1, 39.2, 139.4.
#ifndef GACT_SUM_H
#define GACT_SUM_H

#include <stdint.h>

#include "gact_device.h"

namespace gact {

constexpr uint32_t kRowTerms = 512;               // eight a lane: their loads are in flight together
constexpr uint32_t kPatience = 1u << 14;          // looks, at about a microsecond each; what is awaited takes some ten
constexpr uint32_t kGrace = 1u << 20;

__host__ __device__ constexpr uint32_t rows_of(uint32_t count) { return (count + kRowTerms - 1) / kRowTerms; }
// Adding blocks of WAVES wavefronts, a row each.
template <int WAVES>
__host__ __device__ constexpr uint32_t adders_for(uint32_t count) { return (rows_of(count) + WAVES - 1) / WAVES; }
// Blocks that take a footprint's sample points, one a thread.
template <int WAVES>
__host__ __device__ constexpr uint32_t samplers_for(int n_samples) { return ((uint32_t)n_samples + 64 * WAVES - 1) / (64 * WAVES); }
// Whether a launch of `blocks` such blocks has room for them.
template <int WAVES>
constexpr bool room_for_adders(uint64_t blocks, int n_samples = 0) {
    return launchable(blocks, 64 * WAVES) &&
           launchable(blocks + adders_for<WAVES>((uint32_t)blocks) + samplers_for<WAVES>(n_samples), 64 * WAVES);
}

// What a reducing launch needs to add its results itself.  tag 0: they stay as they are, one word each.
struct Finish {
    uint64_t tag;
    double   scale;
    double*  out;                                 // out[0] = scale * sum
    uint32_t blocks;                              // that leave a result; the adding blocks come behind them
    uint32_t ahead;                               // those of them that stand in front of the grid: none (Late)
    uint32_t patience, grace;                     // kPatience, kGrace
};

inline Finish finish_of(uint64_t tag, double scale, double* out, uint32_t blocks, uint32_t adders, const Late* late) {
    if (late) return Finish{tag, scale, out, blocks, late->ahead ? adders : 0, late->patience, late->grace};
    return Finish{tag, scale, out, blocks, 0, kPatience, kGrace};
}

#ifdef __HIPCC__
// which adding block workgroup b is
__device__ __forceinline__ uint32_t adding_block(const Finish& fin, uint32_t b) { return fin.ahead ? b : b - fin.blocks; }

__device__ __forceinline__ uint64_t load_word(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_word(uint64_t* p, uint64_t w) {
    __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_tagged(uint64_t* pair, double v, uint64_t tag) {
    const uint64_t w = __builtin_bit_cast(uint64_t, v);
    put_word(pair, w);
    put_word(pair + 1, w ^ tag);
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

// Sum of row `row` of `count` tagged results, in all lanes; false if one of them is not there.
__device__ __forceinline__ bool tagged_row(const uint64_t* pairs, uint32_t count, uint32_t row, uint64_t tag, int lane,
                                           double& sum) {
    double v[8];
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
    if (!__all(there)) return false;
    sum = add_row(v);
    return true;
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

// The mark that the last adding block leaves in the place of the result: a NaN of this call's own.
__device__ __forceinline__ uint64_t given_up(uint64_t tag) { return 0x7FF8000000000000ull | tag >> 13; }
// What this wavefront has written is in memory.
__device__ __forceinline__ void await_writes() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// What lies in the place of the result, and whether it is the mark (asked where the answer is needed, so that
// a block does not wait for the load).
__device__ __forceinline__ uint64_t result_word(const Finish& fin) { return load_word((const uint64_t*)fin.out); }
__device__ __forceinline__ bool marked(const Finish& fin, uint64_t word) { return __all(word == given_up(fin.tag)); }

// One more look of an adding wavefront at what is not there.  False: it has looked long enough.
struct Looks {
    uint32_t n = 0;
    __device__ __forceinline__ bool again(const Finish& fin, bool last) {
        if (last && n == fin.patience) {
            put_word((uint64_t*)fin.out, given_up(fin.tag));
            await_writes();
        }
        if (n++ == fin.patience + fin.grace) return false;
        __builtin_amdgcn_s_sleep(1);
        return true;
    }
};

// The rows' sums as lane `lane` of the wavefront that adds them takes them: rows lane, lane + 64, ... in
// [0, end), one after the other onto acc: tagged pairs that other blocks leave in the place of each row's
// first two words.  False: one did not come.
__device__ __forceinline__ bool add_left_rows(double& acc, const uint64_t* words, size_t row_words, uint32_t end,
                                              const Finish& fin, int lane, Looks& looks) {
    for (uint32_t r = (uint32_t)lane; r < end; r += 64) {
        const uint64_t* p = words + (size_t)r * row_words;
        uint64_t w;
        while (((w = load_word(p)) ^ load_word(p + 1)) != ~fin.tag)
            if (!looks.again(fin, true)) return false;
        acc += __builtin_bit_cast(double, w);
    }
    return true;
}
// ... rows [first, end) whose sums are in `mine`
__device__ __forceinline__ double add_own_rows(double acc, const double* mine, uint32_t first, uint32_t end, int lane) {
    for (uint32_t r = first + (((uint32_t)lane - first) & 63u); r < end; r += 64) acc += mine[r - first];
    return acc;
}

// Adding block f of adders_for<WAVES>(count): a wavefront adds one row; all blocks but the last leave
// the row's sum behind, the last adds them up.  PAIRS: the results are tagged (else each is one word, and all
// are there), so that a row has twice as many words.
template <bool PAIRS>
__host__ __device__ constexpr size_t row_words() { return (PAIRS ? 2 : 1) * (size_t)kRowTerms; }

// Sum of row `row`, in all lanes, from what lies in the workspace now.
template <int WAVES, bool PAIRS>
__device__ __forceinline__ bool row_now(const uint64_t* words, const Finish& fin, uint32_t row, int lane, double& sum) {
    if (row < (adders_for<WAVES>(fin.blocks) - 1) * WAVES) {       // a row whose sum is left behind
        const uint64_t* p = words + (size_t)row * row_words<PAIRS>();
        const uint64_t w = load_word(p), x = load_word(p + 1);
        if (__all((w ^ x) == ~fin.tag)) { sum = __builtin_bit_cast(double, w); return true; }
        if (!PAIRS) return false;
    }
    if (PAIRS) return tagged_row(words, fin.blocks, row, fin.tag, lane, sum);
    sum = plain_row((const double*)words, fin.blocks, row, lane);
    return true;
}

// The result, if everything that it needs is there; one wavefront.  `row` is looked at first.
template <int WAVES, bool PAIRS>
__device__ __forceinline__ void try_finish(const uint64_t* words, const Finish& fin, uint32_t row, int lane) {
    double s, acc = 0.0;
    if (!row_now<WAVES, PAIRS>(words, fin, row, lane, s)) return;
    for (uint32_t r = 0; r < rows_of(fin.blocks); ++r) {
        if (!row_now<WAVES, PAIRS>(words, fin, r, lane, s)) return;
        if ((r & 63u) == (uint32_t)lane) acc += s;
    }
    const double total = add_lanes(acc);
    if (lane == 0) put_word((uint64_t*)fin.out, __builtin_bit_cast(uint64_t, fin.scale * total));
}

// Behind what a late block's first wavefront or an adding block's leaves in the workspace, of row `row`.
template <int WAVES, bool PAIRS>
__device__ __forceinline__ void look_for_mark(const uint64_t* words, const Finish& fin, uint32_t row, int lane) {
    await_writes();
    if (marked(fin, result_word(fin))) try_finish<WAVES, PAIRS>(words, fin, row, lane);
}

// Block b's result, by the block's first wavefront.  first_word: result_word behind the block's loads.  WAVES: those of
// an adding block.
template <int WAVES>
__device__ __forceinline__ void put_result(double* partial, uint32_t b, double v, const Finish& fin, uint64_t first_word,
                                           int lane) {
    if (fin.tag == 0) {
        if (lane == 0) partial[b] = v;
        return;
    }
    uint64_t* words = (uint64_t*)partial;
    if (lane == 0) put_tagged(words + 2 * (size_t)b, v, fin.tag);
    if (marked(fin, first_word)) look_for_mark<WAVES, true>(words, fin, b / kRowTerms, lane);
}

template <int WAVES, bool PAIRS>
__device__ __forceinline__ void finish_block(uint64_t* words, const Finish& fin, uint32_t f) {
    __shared__ double lds[WAVES];
    __shared__ bool missing[WAVES];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t rows = rows_of(fin.blocks), adders = adders_for<WAVES>(fin.blocks);
    const uint32_t row = f * WAVES + (uint32_t)wave;
    const bool last = f + 1 == adders;
    // The last block's first wavefront takes what the other blocks leave before it waits for its own
    // row, which is complete later than theirs.
    Looks looks;
    double acc = 0.0, s = 0.0;
    bool there = true;
    if (last && wave == 0) there = __all(add_left_rows(acc, words, row_words<PAIRS>(), f * WAVES, fin, lane, looks));
    if (row < rows && there) {
        if (!PAIRS) s = plain_row((const double*)words, fin.blocks, row, lane);
        else while (there && !tagged_row(words, fin.blocks, row, fin.tag, lane, s)) there = __all(looks.again(fin, last));
    }
    if (!last) {
        if (!there) return;
        // another tag than the results', one of which was in this place
        if (lane == 0) put_tagged(words + (size_t)row * row_words<PAIRS>(), s, ~fin.tag);
        look_for_mark<WAVES, PAIRS>(words, fin, row, lane);
        return;
    }
    if (lane == 0) { lds[wave] = s; missing[wave] = !there; }
    __syncthreads();
    if (wave != 0) return;
    bool all = true;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) all = all && !missing[w];
    if (all) {
        const double total = add_lanes(add_own_rows(acc, lds, f * WAVES, rows, lane));
        if (lane == 0) *fin.out = fin.scale * total;
        return;
    }
    try_finish<WAVES, PAIRS>(words, fin, 0, lane);
}

// A footprint's sample point: out[1 + j] = element floor(j * n / n_samples) as binary64.  (j < 2^15, and n at most
// 2^44, from the number of blocks that a launch may have.)
__device__ __forceinline__ void sample(const void* x, int dtype, int64_t n, int j, int n_samples, double* __restrict__ out) {
    const int64_t i = (int64_t)((uint64_t)j * (uint64_t)n / (uint32_t)n_samples);
    float v;
    if (dtype == GACT_DT_F32) v = ((const float*)x)[i];
    else v = __builtin_bit_cast(float, (uint32_t)((const uint16_t*)x)[i] << 16);
    out[1 + j] = (double)v;
}
#endif  // __HIPCC__

}  // namespace gact

#endif
