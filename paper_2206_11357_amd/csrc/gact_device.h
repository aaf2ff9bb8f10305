// Records passed from the host entry points to the kernels.  Internal to the
// library; the public interface is include/gact.h.
#ifndef GACT_DEVICE_H
#define GACT_DEVICE_H

#include <stddef.h>
#include <stdint.h>

#ifndef __HIPCC__
#define __host__
#define __device__
#endif

#define GACT_DT_F32 0
#define GACT_DT_BF16 1

namespace gact {

// One tensor of a launch (56 bytes).  Pointers are device pointers.
struct TensorArgs {
    void*       io;        // compress: input x (read only); decompress: output y
    void*       packed;    // bit string (compress output, decompress input)
    float*      gmin;      // per-group minimum
    float*      gscale;    // per-group dequantisation step
    int64_t     n;         // elements
    uint32_t    seed_lo, seed_hi;
    // Whole dwords only: a sub-dword field would be fetched with a vector load,
    // which queues behind the kernel's own HBM traffic at the start of every block,
    // whereas dword fields of a uniform record come through the scalar cache.
    uint32_t    blk_base_lo;  // Philox block of element 0 (index_base / 8), low word
    uint32_t    meta;         // bits | dtype << 8 | (index_base / 8 >> 32) << 16
    __host__ __device__ int bits() const { return (int)(meta & 0xFFu); }
    __host__ __device__ int dtype() const { return (int)((meta >> 8) & 0xFFu); }
    __host__ __device__ uint64_t blk_base() const {
        return ((uint64_t)(meta >> 16) << 32) | blk_base_lo;
    }
};

// How a group size maps onto a wavefront: a lane owns 32 consecutive
// elements, a group is `lpg` = G/32 neighbouring lanes, a tile holds as many
// whole groups as fit into 64 lanes.
struct Geometry {
    int32_t lpg;           // lanes per group, 1..32
    int32_t lanes_used;    // (64 / lpg) * lpg
    int32_t pow2;          // lpg is a power of two (DPP reductions, full tiles)
    int32_t groups_per_tile;
    int32_t group_shift;   // element e belongs to group (e >> 4) * group_magic >> 32 >> group_shift
    uint32_t group_magic;  // (group_divisor)
    int32_t lpg_magic;     // floor(65536 / lpg) + 1: lane / lpg = lane * lpg_magic >> 16 for lane < 64
    int32_t lds_wave_dwords;   // compress: LDS dwords per wavefront (lds_dwords_per_wave of the widest dtype launched)
};
// The single-tensor kernels' arguments stay below 112 bytes: from 120 on, the runtime takes the host 0.6 us
// longer per launch (3.1 -> 3.7 us), which is what bounds small calls.
static_assert(sizeof(TensorArgs) + sizeof(Geometry) + 16 <= 112, "arguments of the single-tensor kernels");
// Division of e >> 4 by d = 2 lpg, for e < 2^35, as a product (Granlund, Montgomery 1994, Thm. 4.2):
// with 2^(s+1) >= d, m = floor(2^(32+s) / d) + 1 exceeds 2^(32+s) / d by at most 1, so that
// the product is at most e >> 4 < 2^31 <= 2^(32+s) / d, less than one d-th of 2^(32+s), too large.
// d is at least 2, so that m fits 32 bits; where d is a power of two, m = 2^31 without the 1 is exact.
constexpr int64_t kMagicElems = (int64_t)1 << 35;
inline void group_divisor(Geometry* geo) {
    const uint32_t d = 2u * (uint32_t)geo->lpg;
    int32_t s = 0;
    while ((2u << s) < d) ++s;
    geo->group_shift = s;
    geo->group_magic = (uint32_t)(((uint64_t)1 << (32 + s)) / d + ((d & (d - 1)) != 0 ? 1 : 0));
}
// the geometry in front of a launch table that starts on a 64-byte line, behind three dwords
struct LineGeometry {
    Geometry geo;
    int32_t  pad[5];
};
static_assert(12 + sizeof(LineGeometry) == 64, "the launch table starts on a line");

// How blocks are dealt to the XCDs (work_block, runs_for).
struct Runs {
    uint32_t end;          // blocks in whole windows of eight runs; 0: plain order
    uint32_t shift;        // log2 of the neighbouring blocks one XCD takes in a run
};

#ifdef __HIPCC__
// The block of work that workgroup b takes (work_block in gact_kernels.hip says why).
__device__ __forceinline__ uint32_t ordered_block(uint32_t b, uint32_t run_end, uint32_t s) {
    if (b >= run_end) return b;
    const uint32_t low = (8u << s) - 1u;
    return (b & ~low) | ((b & 7u) << s) | ((b & low) >> 3);
}
#endif

// What a launch does.  A compressing launch is one of three kernels:
//   kCompressBf16  every tensor is bf16: 4 KB of LDS per wavefront, so eight wavefronts per
//                  SIMD are resident if they keep to 64 VGPRs;
//   kCompressAny   fp32 among them: 8 KB of LDS per wavefront, four per SIMD, 128 VGPRs each;
//   kCompressLong  the same in launches of kLongCompress such blocks and more, in blocks of one wavefront:
//                  of these more are resident (a block of four needs 32 KB of the 160 at once) and each
//                  leaves by itself.  Us, blocks of four | of one: 53 fp32 tensors of 0.7 G elements 479 | 469,
//                  4 bits 520 | 507, groups of 1024 490 | 480, one of 0.42 G, 4 bits 307 | 294; 40 of both types,
//                  0.9 G 504 | 505.  Shorter launches gain nothing for sure, or lose (53 fp32 tensors, 2 bits, 89 M
//                  elements 59.0 | 59.1, 0.18 G 119 | 120, 0.27 G 176 | 180), and bf16 gains 1 % on some sets
//                  and loses 2 % on others (400 tensors of 2 G elements 829 | 843).  Nor is it for tiles that leave
//                  1 to 9 lanes without data (long_compress).
// A decompressing launch of fewer than kShortLaunch blocks is a kernel of its own, for
// its units per wavefront and because such a launch has no block order.  (As a branch
// in one kernel it gave back half of what the other units gain: one bf16 tensor of
// 7.5 M elements, 2 bits, 4.4 us; with three units 4.9, this kernel 4.1.)
enum Work { kDecompress, kCompressBf16, kCompressAny, kDecompressShort, kCompressLong };
constexpr bool decompresses(Work w) { return w == kDecompress || w == kDecompressShort; }
constexpr int waves_per_block(Work w) { return w == kCompressLong ? 1 : 4; }
constexpr int kReduceWaves = 8;
constexpr uint64_t kLongCompress = 32768;
// Whether `blocks` of kCompressAny, among them bf16_blocks of bf16 tensors, are launched as kCompressLong (whose grid has
// four times as many).  The time of blocks of four wavefronts over that of blocks of one, lists of 15 and 80 fp32 tensors of
// unequal sizes and widths, 0.3 to 0.7 G elements, by the lanes that hold data in a tile, which are whole groups:
//   lanes        64          63          62         60         58    57    56    55    54    52    51   44-50
//          1.010-1.018  0.991-1.003  0.977  0.969-0.980  0.980 0.988 0.995 1.003 1.009 1.019 1.017  1.020
// (Tiles of the 64 are 8 KB and begin on 8 KB; those that leave 10 lanes and more idle issue so much more per element that
// the resident wavefronts count.)  bf16 beside it, as a share of the elements, 63 lanes: none 0.980-0.991, 0.1 0.980-0.991,
// 0.2 0.994-1.000, 0.3 1.002-1.004, 0.4 1.007-1.011, 0.6 1.018, 0.8 1.021-1.025.
constexpr bool long_compress(uint64_t blocks, uint64_t bf16_blocks, int lanes_used) {
    return blocks >= kLongCompress && blocks <= 0x7FFFFFFFull / 4 &&
           (lanes_used == 64 || lanes_used <= 54 || 4 * bf16_blocks >= blocks);
}

// LDS one compressing wavefront stages its tile in: 64 rows of 32 elements in
// the input's own format.
constexpr int lds_dwords_per_wave(int dtype) { return dtype == GACT_DT_F32 ? 64 * 32 : 64 * 16; }

// Block -> tensor lookup of a multi-tensor launch.  first_block[l] is the first
// block of tensor l (one entry per tensor plus the total).  A search over it
// from scratch is a chain of dependent scalar loads at the start of every
// block (nine for 400 tensors), during which the block issues nothing else, so
// the host also lays a coarse index over the blocks: hint[k] is the tensor that
// holds block k << hint_shift.  Block b then belongs to a tensor in
// [hint[b >> hint_shift], hint[(b >> hint_shift) + 1]], which for all but the
// buckets that contain a tensor boundary is a single tensor.
constexpr int kInlineHints = 128;
// buckets for a table of L tensors in the workspace: a power of two >= 4 L
constexpr int hint_buckets(int L) {
    int h = 64;
    while (h < 4 * L && h < 16384) h *= 2;
    return h;
}

// Bytes of arguments a kernel can have.
constexpr size_t kKernelArguments = 4096;
// A launch table small enough to travel in the kernel arguments.
constexpr int kInlineTensors = 64;
struct InlineTable {
    TensorArgs t[kInlineTensors];
    uint32_t   first_block[kInlineTensors + 1];
    uint32_t   hint[kInlineHints / 4 + 1];   // one byte per bucket, four to a dword (scalar loads fetch dwords)
};
static_assert(12 + sizeof(LineGeometry) + sizeof(InlineTable) <= kKernelArguments, "a list's launch table and what precedes it");
// tensor of bucket k in a byte-packed hint array
__host__ __device__ inline int packed_hint(const uint32_t* hint, uint32_t k) {
    return (int)((hint[k >> 2] >> ((k & 3u) * 8u)) & 0xFFu);
}

// One buffer pair of a reduction launch: sensitivity reads a and b; gradient
// statistics read a (the gradient) and read-modify-write b (the fp32 mean).
struct ReduceArgs {
    const void* a;
    void*       b;
    int64_t     n;
    int32_t     dtype;     // of a (and of b for sensitivity)
    int32_t     pad;
};
// A buffer table small enough to travel in the kernel arguments: 36 bytes a buffer, so that up to 112 would
// fit beside the 56 bytes of the sensitivity kernel's other arguments; eight buffers' room is left.
constexpr int kInlineBuffers = 104;
struct ReduceTable {
    ReduceArgs t[kInlineBuffers];
    uint32_t   first_block[kInlineBuffers + 1];
};
static_assert(sizeof(ReduceTable) + 64 <= kKernelArguments, "a buffer table and what follows it");

// Runs of the reductions' blocks (16 KB of each buffer they only read) that go to one XCD, as a power of two.
// Us a call on MI355X, plain order and runs of 2^s blocks, buffers of an encoder's sizes:
//                                      plain   s=2    s=3    s=4    s=5    s=6    s=7
//   sensitivity, fp32, 302 M elements   350    354    343    344    344    347    351
//   sensitivity, bf16, 302 M            178    179    178    178    181    181    181
//   statistics, fp32, 302 M             601    639    589    609    587    583    595
//   statistics, bf16, 302 M             501    504    483    492    477    478    487
//   statistics, bf16, 85 M              142    141    139    139    138    138    140
// Launches below one window of eight runs keep plain order.
constexpr uint32_t kDiffRunShift = 3, kStatsRunShift = 5;
constexpr uint32_t runs_end(uint32_t blocks, uint32_t s) { return blocks >> (3 + s) << (3 + s); }
// A statistics launch of fewer blocks is in memory at once, or nearly so: plain order, and a block does not wait for its
// stores before it adds up.  Us, plain order and no wait | runs and a wait, an encoder's buffers: fp32, 6.3 M elements 15.9 |
// 16.6, 12.6 M 27.6 | 28.3, 25 M 50.4 | 50.5, 32 M 64.6 | 64.1; bf16, 6.3 M 13.7 | 14.1, 12.6 M 23.9 | 24.3, 25 M 42.5 | 42.6.
constexpr uint32_t kShortStats = 4096;
// (Wide blocks are more than that; asked for it all the same, a block of theirs starts later: 302 M fp32 0.4 %.)
constexpr uint32_t stats_runs_end(uint32_t blocks, bool wide) { return !wide && blocks < kShortStats ? 0 : runs_end(blocks, kStatsRunShift); }

// Elements of one buffer a block covers: 512 threads x 2 pieces, of 16 bytes where the buffers are only
// read, of 4 elements in a statistics step (16 bytes of the fp32 mean, whatever the gradient's type).
// A statistics step in a workspace that holds a pair of results for every reduce_chunk_elems(dtype) and no
// more has its blocks take two such chunks of a bf16 buffer, one after the other (302 M parameters: 528 us;
// 505 us with one chunk a block, which is what gact_reduce_workspace_bytes has room for).
constexpr int64_t reduce_chunk_elems(int dtype) { return dtype == GACT_DT_F32 ? 4096 : 8192; }
constexpr int64_t kStatsChunkElems = 4096;
constexpr int64_t stats_block_elems(int dtype, int bf16_chunks) {
    return dtype == GACT_DT_F32 ? kStatsChunkElems : kStatsChunkElems * bf16_chunks;
}
static_assert(stats_block_elems(GACT_DT_BF16, 2) == reduce_chunk_elems(GACT_DT_BF16) &&
              stats_block_elems(GACT_DT_F32, 2) == reduce_chunk_elems(GACT_DT_F32), "the least workspace");

// Threads of a launch: the runtime takes fewer than 2^32.
constexpr bool launchable(uint64_t blocks, uint32_t threads) { return blocks * threads < 1ull << 32; }

// A statistics launch of this many blocks and more, all of whose buffers are fp32 with a mean that starts
// on a line, is one of wide blocks (stats_chunk), up to what the runtime takes of those (17 G elements); but
// not where a buffer has fewer than kWideBlocks blocks on average: a block first finds its buffer, log2 of their
// number of loads one after the other, then often cut short by the buffer's end, and half as many blocks are
// there to hide that.  Us, narrow | wide blocks, buffers of equal size:
//   M elements, buffers   100         312         600         1000        2000        4000        8000
//        40            79.6 | 80   83.0 | 84   86.2 | 89   89.1 | 92    101 | 110   106 | 120   127 | 161
//        80             159 | 152   159 | 154   166 | 160   170 | 166   175 | 188   181 | 198   191 | 217
//       160             319 | 292   315 | 298   319 | 304   349 | 307   337 | 335   323 | 350   334 | 370
//       300             587 | 544   611 | 547   645 | 561   623 | 562   625 | 586   574 | 612   602 | 655
constexpr uint64_t kWideStats = 8192, kWideBlocks = 24;
constexpr int stats_threads(bool wide) { return wide ? 1024 : 512; }
constexpr bool wide_stats(uint64_t blocks, uint64_t buffers) {
    return blocks >= kWideStats && blocks >= kWideBlocks * buffers && launchable(blocks, stats_threads(true));
}

// Decompress launch shape.  A unit is the 1 KB of output one coalesced
// wavefront store covers (256 fp32 or 512 bf16 elements); a block of four
// wavefronts takes 4 * units consecutive units.  Units per wavefront trade the
// load latency a wavefront hides against the length of its store burst; the
// best value depends on the code width and was chosen by sweep on MI355X, with
// the block order of run_shift_for (us, decompress, every tensor at that width:
// 96 bf16 tensors of 1.4 G elements, 400 bf16 ones of 1.0 G, 53 fp32 ones of 0.7 G,
// 3 fp32 ones of 87 M):
//            units    1                     2                     3                     4
//   b=1      669 524 672  93       532 437 533  76       532 415 471  70       542 424 484  68
//   b=2      691 535 706  97       533 439 536  77       532 415 496  72       537 444 496  71
//   b=4      716 539 702  98       554 431 524  76       638 422 559  73       584 445 571  78
//   b=8      694  -  665   -       665  -  556   -       724  -  664   -       700  -  645   -
// A launch of 53 fp32 tensors of mixed widths around 2 bits, 89 M elements: 65.3 us
// with four units at 2 bits, 66.7 with three.  bf16 at 2 bits takes four as well where
// the launch is shorter than kShortLaunch blocks (us, one tensor; lists of 3 to 100
// tensors cross at the same size, 48 M elements or 7.8k blocks):
//   M elements    4    7.5    12    16    24    32    48    64   100   160
//   three       3.7   4.9   7.0   8.4  11.6  14.7  20.5  26.4  39.5  61.7
//   four        3.5   4.2   6.5   8.5  11.3  14.5  20.7  26.7  40.3  62.2
// The units of 1-, 2-, 4- and 8-bit codes, three bits of a table each at 3 * bits: a
// block computes its length from them without a branch.
constexpr uint32_t dec_unit_table(uint32_t b1, uint32_t b2, uint32_t b4, uint32_t b8) {
    return b1 << 3 | b2 << 6 | b4 << 12 | b8 << 24;
}
constexpr uint32_t kDecUnitsF32 = dec_unit_table(3, 4, 2, 2);
constexpr uint32_t kDecUnitsBf16 = dec_unit_table(3, 3, 2, 2), kDecUnitsBf16Short = dec_unit_table(3, 4, 2, 2);
// blocks, counted with kDecUnitsBf16 (the count with kDecUnitsBf16Short is never larger, so that either
// tells which of the two a launch uses)
constexpr uint64_t kShortLaunch = 8192;
constexpr int dec_units(uint32_t table, int bits) { return (int)(table >> (3 * bits) & 7u); }
// elements of a block; bf16_units: the table of bf16 tensors
constexpr int dec_block_elems(int dtype, int bits, uint32_t bf16_units) {
    return dtype == GACT_DT_F32 ? 4 * 256 * dec_units(kDecUnitsF32, bits) : 4 * 512 * dec_units(bf16_units, bits);
}
// Blocks of n elements.  Without a division by a variable, which for 300 short tensors, counted twice, took the host
// 0.8 us of 12.7.
constexpr int64_t dec_blocks(int64_t n, int dtype, int bits, uint32_t bf16_units) {
    const int64_t rows = dtype == GACT_DT_F32 ? (n + 1023) >> 10 : (n + 2047) >> 11;      // of a block's four wavefronts
    const int units = dec_units(dtype == GACT_DT_F32 ? kDecUnitsF32 : bf16_units, bits);
    return units == 2 ? (rows + 1) >> 1 : units == 4 ? (rows + 3) >> 2 : (rows + 2) / 3;
}
static_assert(dec_units(kDecUnitsF32, 1) == 3 && dec_units(kDecUnitsBf16, 1) == 3, "two, three or four units");

// In what order a decompressing wavefront issues the loads of its units, and how fast.  Back to back they
// are slower than with pauses in between (s_sleep, of 64 cycles): what a wavefront asks for at once arrives
// at once and is stored at once, and HBM takes reads and stores that come in such waves worse than a steady
// mix.  Which order is best depends on the sizes of the loads and was chosen by sweep (us, decompress):
//                                  bf16, 1.0 G in 400 tensors    bf16, 1.4 G in 96        fp32, 0.7 G in 53
//   bits                             1      2      4               1      2      4          1      2      4      8
//   codes, division, group by unit  405    404    414             540    533    555        471    491    532    553
//   the same without the division   400    405    430             536    528    574        487    542    525    550
//   groups, pause, codes by unit    384    384    410             515    542    554        623    496    531    565
//   groups, pause, codes, paused    375    389    415             502    557    563        471    502    514    554
//   codes, pause, groups            444    --     431             544    543    574        467    490    536    551
//   as below                        374    384    409             502    533    552        466    494    504    556
// At 2 and 8 bits of fp32, taken again in turn, division and as below are equal (492, 493; 555, 555); what differs
// are launches of mixed widths: 400 bf16 tensors, about 3 bits, 829, 813 (0.26 G 109.3, 105.6); groups of 224 422, 400;
// 53 fp32 tensors 493, 490; 3 fp32 ones of 87 M 72.4, 69.2, groups of 96 74.7, 69.6; 40 of both types, 0.6 G 361, 336.
// One long tensor of bf16 at 4 bits lost by the order that is best for lists (division, that order, codes first): 34 M
// 15.72, 15.93, 15.86; 80 M 32.2, 32.6, 32.2; 150 M 59.2, 59.3, 58.3; 220 M 84.5, 85.5, 84.3; 290 M 110.9, 112.6, 110.8;
// but 400 of 1.0 G 402, 403, 420, 96 of 1.4 G 558, 557, 579.  Single tensors have a kernel of their own, and this order.
//
// Launches of fewer than kShortLaunch blocks are over before HBM has settled to any mix, and what waits is the
// wavefront: they have orders of their own.  The orders of the long launches lose up to 13 % there, and a product for
// groups that are a power of two (a shift is known three multiplies earlier) up to 4 %, so that these widths choose
// between the two.  Us, one tensor, buffers that are not in the caches, groups of 256 (of 96), the division in the order
// by unit | the orders of long launches, for bf16 the product | as below:
//   M elements            4                      8                    12                     16 (fp32: 15)
//   fp32  b=1   4.99 | 5.20 | 4.82     7.90 | 7.86 | 7.77    11.02 | 10.66 | 10.57   12.93 | 12.81 | 12.83
//         b=2   4.31 | 4.25 | 4.26     7.89 | 7.54 | 7.62    11.28 | 10.89 | 10.91   13.67 | 13.26 | 13.27
//         b=4   4.70 | 5.22 | 4.56     8.26 | 8.60 | 8.00    11.34 | 11.53 | 11.03   13.51 | 13.51 | 13.09
//         b=8   4.29 | 4.50 | 4.29     8.52 | 7.39 | 7.41    11.94 | 10.22 | 10.24   14.35 | 12.38 | 12.40
//   bf16  b=1   3.61 | 3.62 | 3.65     5.04 | 4.48 | 4.38     6.68 |  6.60 |  6.56    8.34 |  8.72 |  8.30
//         b=2   3.65 | 3.60 | 3.68     4.33 | 4.39 | 4.39     6.67 |  5.90 |  5.92    8.64 |  7.17 |  7.19
//         b=4   3.66 | 3.66 | 3.71     4.32 | 4.38 | 4.40     6.77 |  6.89 |  6.88    8.75 |  9.03 |  8.73
//         b=8   3.57 | 3.54 | 3.60     6.32 | 5.01 | 4.96     8.45 |  6.50 |  6.45   10.32 |  8.42 |  8.40
//   (96)  fp32, 8 M, b=1 8.23 | 7.86 | 7.86, b=4 9.09 | 8.61 | 8.60; bf16 b=1 5.61 | 4.56 | 4.96, b=4 5.56 | 4.47 | 4.72
// At 8 bits the last column is the lists' order.  What it gains where the codes were written long ago it loses right behind
// their compressor, 4 % on average; single calls, which come like that, load by unit without a pause.  Us, one tensor
// compressed and decompressed in turn, groups of 256, the division by unit | the lists' order | by unit: bf16, 9.4 M 15.2 |
// 15.5 | 15.3, 13 M 17.6 | 18.5 | 17.7, 16 M 20.0 | 22.0 | 20.1, 19 M 23.3 | 26.1 | 23.4; fp32, 6 M 13.7 | 14.3 | 13.6, 9.4 M
// 19.2 | 20.5 | 19.2, 13 M 25.3 | 26.9 | 25.2, 16 M 28.8 | 31.5 | 28.8.
enum GroupIndex {
    kByProduct,            // a product (group_divisor) for every group size
    kByEither,             // a shift for group sizes that are a power of two, chosen at each piece
    kByBranch              // the same, chosen once around all loads (both of these: codes first, no pauses between units)
};
struct LoadOrder {
    bool by_unit;          // a unit's codes and its minima and steps together, else those of all units in turn
    bool groups_first;     // minima and steps before codes
    int  kinds, units;     // s_sleep between codes and minima, and between units; -1: in this order, without a pause
    GroupIndex group = kByProduct;
};
enum Launch { kLongList, kLongSingle, kShortList, kShortSingle };
constexpr LoadOrder load_order(int dtype, int bits, Launch launch) {
    const bool short_launch = launch == kShortList || launch == kShortSingle;
    if (short_launch && bits == 1) return LoadOrder{false, false, 1, 0, kByEither};
    if (short_launch && bits == 4) return LoadOrder{true, false, 0, 0, kByBranch};
    if (launch == kShortSingle && bits == 8) return LoadOrder{true, false, 0, 0, kByEither};
    if (short_launch && dtype == GACT_DT_BF16) return bits == 2 ? LoadOrder{false, false, 1, 0} : LoadOrder{true, false, 0, 1};
    if (short_launch) return bits == 2 ? LoadOrder{false, false, 4, 0} : LoadOrder{false, false, 1, -1};
    if (dtype == GACT_DT_F32)
        return bits == 1 ? LoadOrder{false, false, 2, 1} : bits == 2 ? LoadOrder{false, false, 4, 0}
             : bits == 4 ? LoadOrder{false, true, 1, 0} : LoadOrder{false, true, 1, 1};
    if (bits == 4 && launch == kLongSingle) return LoadOrder{true, false, 1, 0};
    return bits == 1 ? LoadOrder{false, true, 1, 1} : LoadOrder{true, true, 1, 0};
}

// Length of the runs of neighbouring blocks that go to one XCD, as a power of two
// (us on MI355X, plain order and runs of 2^s blocks):
//                                              plain   s=4    s=5    s=6    s=7    s=8    s=9
//   compress  400 bf16 tensors, 253k blocks     922    901    887    882    871    859    863
//   compress  96 bf16 tensors, 688k blocks     2386   2389   2363   2357   2352   2352   2352
//   compress  53 fp32 tensors, 87k blocks       498    486    481    481    481    483    483
//   compress  400 bf16 tensors, 32k blocks      121    116    115    114    115    117    120
//   compress  3 fp32 tensors, 16k blocks       69.4   68.3   68.2   68.6   69.4   70.0   70.3
//   decompress 96 bf16 tensors, 1.3M blocks    2382   2514   2353   2360   2351   2334   2329
//   decompress 400 bf16 tensors, 419k blocks    830    853    836    839    840    846    846
//   decompress 53 fp32 tensors, 226k blocks     494    493    491    492    494    502    508
//   decompress 400 bf16 tensors, 53k blocks   111.9  108.7  109.3  109.2  107.9  109.7  111.1
//   decompress 3 fp32 tensors, 34k blocks      76.4   73.6   73.4   73.6   74.5   75.4   77.6
//   the same, every buffer on a line           71.8   71.9   71.7   71.9   72.6   73.5   75.7
//   decompress 53 fp32 tensors, 28k blocks     65.2   65.1   65.0   65.5   67.1   67.8   68.8
//   decompress 1 bf16 tensor, 1.8k blocks      4.85    --    5.35
// Compress: runs as long as leave 64 windows, at most 256 blocks.  Decompress: runs of 32 (runs of 4 to 16
// cost up to 10 % on bf16 output at 4 bits, and lengths that are no power of two are worse than 32 throughout),
// for all types and alignments: where no line is shared between blocks they cost nothing, and of the launches
// above one loses (0.7 %).  Launches of few windows keep plain order: the XCDs that get the runs of a last,
// partial window finish late.
constexpr uint32_t kDecompressRunShift = 5;
// Blocks of one wavefront (kCompressLong), 53 fp32 tensors of 0.7 G elements, s = 4 .. 8: 479, 479, 472, 472, 475 us;
// at 4 bits 523, 526, 508, 513, 520.
constexpr uint32_t kCompressLongRunShift = 6;
inline int run_shift_for(Work w, uint64_t blocks) {
    int log2 = 0;
    while ((blocks >> log2) > 1) ++log2;
    if (w == kCompressLong) return (int)kCompressLongRunShift;
    if (!decompresses(w)) return log2 < 13 ? 0 : (log2 - 9 < 8 ? log2 - 9 : 8);
    return log2 < 14 ? 0 : (int)kDecompressRunShift;
}

inline Runs runs_for(Work w, uint64_t blocks) {
    const int s = run_shift_for(w, blocks);
    return Runs{s ? runs_end((uint32_t)blocks, (uint32_t)s) : 0u, (uint32_t)s};
}

// For tests of the in-launch addition (gact_sum.h): how long its adding blocks wait, in looks, and whether they stand
// in front of their grid, so that what they wait for comes late.  Null: as the library's own calls.
struct Late {
    uint32_t patience, grace, ahead;
};

}  // namespace gact

extern "C" int gact_launch_single(gact::Work work, const gact::TensorArgs* t,
                                  const gact::Geometry* geo, unsigned blocks, void* stream);
// `inline_table` is used when it is not null, else the table in device memory
extern "C" int gact_launch_diff_sq(const gact::ReduceTable* inline_table, const gact::ReduceArgs* d_table,
                                   const uint32_t* d_first, int K, unsigned blocks, double* d_partial, int tagged,
                                   uint64_t tag, double scale, double* d_out, void* stream, const gact::Late* late);
extern "C" int gact_launch_compress_sum(const gact::TensorArgs* t, const gact::Geometry* geo,
                                        unsigned blocks, double* d_block_sum, int tagged, uint64_t tag,
                                        int n_samples, double* d_out, void* stream, const gact::Late* late);
extern "C" int gact_launch_footprint_finish(const gact::ReduceArgs* r, unsigned count, double* d_partial, uint64_t tag,
                                            int n_samples, double* d_out, void* stream);
extern "C" int gact_launch_footprint(const gact::ReduceArgs* r, unsigned blocks, double* d_partial, uint64_t tag,
                                     int n_samples, double* d_out, void* stream, const gact::Late* late);
extern "C" int gact_launch_zero(double* d_out, int nout, void* stream);
extern "C" int gact_launch_grad_stats(const gact::ReduceTable* inline_table, const gact::ReduceArgs* d_table,
                                      const uint32_t* d_first, int K, float rt, int bf16_chunks, int wide, unsigned blocks,
                                      double* d_partial, uint64_t tag, double* d_out, void* stream);
extern "C" int gact_launch_copy(void* dst, const void* src, uint64_t nbytes, unsigned workgroups, void* stream);
extern "C" int gact_launch_multi_inline(gact::Work work, const gact::InlineTable* tab, unsigned hint_shift,
                                        const gact::Geometry* geo, unsigned blocks, void* stream);
extern "C" int gact_launch_multi(gact::Work work, const gact::TensorArgs* d_table,
                                 const uint32_t* d_first_block, const uint32_t* d_hint,
                                 unsigned hint_shift, const gact::Geometry* geo, unsigned blocks,
                                 void* stream);

#endif
