// Device-facing side of the C ABI declared in include/gact.h: argument checks,
// launch geometry, the multi-tensor launch table.  The entry points that never
// touch the GPU (sizes, bit allocator, variance alert) are in gact_host.cpp.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <queue>
#include <algorithm>
#include <vector>

#include "gact.h"
#include "gact_device.h"
#include "gact_sum.h"

// Scratch area of gact_compress_footprint_noalloc: device memory that is part
// of the library's code object, one copy per GPU, held until the process ends.
// In host code this name is only a handle for hipGetSymbolAddress; kernels get
// the address that call returns.
static __device__ __align__(256) unsigned char scratch[GACT_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kPerLane = 32;

bool bits_ok(int bits) { return bits == 1 || bits == 2 || bits == 4 || bits == 8; }
bool group_ok(int g) { return g >= 32 && g <= 1024 && g % 32 == 0; }
bool dtype_ok(int dt) { return dt == GACT_F32 || dt == GACT_BF16; }
bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

gact::Geometry make_geometry(int group_size) {
    gact::Geometry geo{};
    geo.lpg = group_size / kPerLane;
    geo.lanes_used = (64 / geo.lpg) * geo.lpg;
    geo.pow2 = (geo.lpg & (geo.lpg - 1)) == 0 ? 1 : 0;
    geo.groups_per_tile = geo.lanes_used / geo.lpg;
    gact::group_divisor(&geo);
    geo.lpg_magic = 65536 / geo.lpg + 1;
    geo.lds_wave_dwords = 0;      // set per launch from the dtypes in it
    return geo;
}

int64_t tiles_for(int64_t n, const gact::Geometry& geo) {
    const int64_t te = (int64_t)geo.lanes_used * kPerLane;
    return (n + te - 1) / te;
}

// Fills `out` and the tensor's tiles; returns GACT_OK or the error for this tensor.
int make_args(bool compress, const void* x, void* packed, float* gmin, float* gscale, void* y,
              int64_t n, uint64_t seed, int64_t index_base, int bits, int dtype,
              const gact::Geometry& geo, gact::TensorArgs* out, uint32_t* out_tiles) {
    if (!bits_ok(bits)) return GACT_E_BITS;
    if (n < 0 || !dtype_ok(dtype)) return GACT_E_ARG;
    // noise is drawn per block of 8 elements: a shard starts on a block boundary
    if (index_base < 0 || (index_base & 7) != 0 || (index_base >> 3) >= (1ll << 48)) return GACT_E_ARG;
    if (n > 0) {
        const void* io = compress ? x : y;
        if (!io || !packed || !gmin || !gscale) return GACT_E_ARG;
        if (!aligned(io, 16) || !aligned(packed, 16) || !aligned(gmin, 4) || !aligned(gscale, 4))
            return GACT_E_ARG;
    }
    const int64_t tiles = tiles_for(n, geo);
    if (tiles > 0xFFFFFFFFll) return GACT_E_ARG;
    *out_tiles = (uint32_t)tiles;
    out->io = compress ? const_cast<void*>(x) : y;
    out->packed = packed;
    out->gmin = gmin;
    out->gscale = gscale;
    out->n = n;
    out->seed_lo = (uint32_t)seed;
    out->seed_hi = (uint32_t)(seed >> 32);
    const uint64_t blk_base = (uint64_t)index_base >> 3;
    out->blk_base_lo = (uint32_t)blk_base;
    out->meta = (uint32_t)bits | ((uint32_t)dtype << 8) | ((uint32_t)(blk_base >> 32) << 16);
    return GACT_OK;
}

// blocks a tensor needs: compress takes a wavefront per tile, decompress
// a fixed span of elements per block.  (The tiles are passed on and not counted anew: the division, once more for
// each of 40,000 tensors where a launch turned out to be long, took the host 100 us beside 355.)
int64_t blocks_for(gact::Work work, const gact::TensorArgs& t, uint32_t tiles) {
    const uint32_t waves = gact::waves_per_block(work);
    if (!decompresses(work)) return ((int64_t)tiles + waves - 1) / waves;
    return gact::dec_blocks(t.n, t.dtype(), t.bits(), work == gact::kDecompressShort ? gact::kDecUnitsBf16Short : gact::kDecUnitsBf16);
}

// The kind of a launch, from the LDS its widest dtype needs; then, its blocks counted as those of that kind,
// the kind it is launched as.
gact::Work work_for(bool compress, const gact::Geometry& geo) {
    if (!compress) return gact::kDecompress;
    return geo.lds_wave_dwords == gact::lds_dwords_per_wave(GACT_BF16) ? gact::kCompressBf16 : gact::kCompressAny;
}
gact::Work work_of_length(gact::Work work, uint64_t blocks, uint64_t bf16_blocks, const gact::Geometry& geo) {
    if (work == gact::kDecompress && blocks < gact::kShortLaunch) return gact::kDecompressShort;
    if (work == gact::kCompressAny && gact::long_compress(blocks, bf16_blocks, geo.lanes_used)) return gact::kCompressLong;
    return work;
}

int run_single(bool compress, const gact::TensorArgs& t, uint32_t tiles, const gact::Geometry& geo, void* stream) {
    if (t.n == 0) return GACT_OK;
    const gact::Work work = work_for(compress, geo);
    int64_t blocks = blocks_for(work, t, tiles);
    if (blocks > 0x7FFFFFFFll) return GACT_E_ARG;
    const gact::Work final_work = work_of_length(work, (uint64_t)blocks, 0, geo);
    if (final_work != work) blocks = blocks_for(final_work, t, tiles);
    return gact_launch_single(final_work, &t, &geo, (unsigned)blocks, stream) == 0
               ? GACT_OK : GACT_E_HIP;
}

// A table upload reads host memory that is gone when a captured graph replays.
// GACT_OK when `stream` is not capturing.
int refuse_if_capturing(void* stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &status) != hipSuccess) return GACT_E_HIP;
    return status == hipStreamCaptureStatusNone ? GACT_OK : GACT_E_CAPTURE;
}

// Whether a launch on `stream` would be recorded into a graph (or that cannot be told).
bool recorded(void* stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();          // not the launch's error
    return true;
}

// Enqueues a copy of a launch table to the workspace; `src` may go when this returns (it is pageable
// memory, of which the runtime takes its own copy first).  The runtime moves up to 16 KB with a small
// kernel, 4.6 us of the stream, and more with the DMA engine, whose hand-over leaves the stream idle for
// 18 to 20 us: tables of up to three such pieces go piece by piece (up to 767 tensors of a block each; fewer
// where the launch has blocks enough to fill the index over them, 545 to 680).  400 tensors, 28 KB: compress
// 115 -> 106 us, decompress 131 -> 109 us (0.25 G bf16 elements).
int upload(void* dst, const unsigned char* src, size_t bytes, void* stream) {
    constexpr size_t kPiece = 16384;
    const size_t piece = bytes <= 3 * kPiece ? kPiece : bytes;
    for (size_t at = 0; at < bytes; at += piece)
        if (hipMemcpyAsync((unsigned char*)dst + at, src + at, std::min(piece, bytes - at), hipMemcpyHostToDevice,
                           (hipStream_t)stream) != hipSuccess)
            return GACT_E_HIP;
    return GACT_OK;
}

size_t table_bytes(int L) { return ((size_t)L * sizeof(gact::TensorArgs) + 15) / 16 * 16; }
size_t first_bytes(int L) { return ((size_t)(L + 1) * sizeof(uint32_t) + 15) / 16 * 16; }

// The coarse block -> tensor index over `first` (live + 1 entries, the last is
// the block total): at most `buckets` buckets of 2^shift blocks; hint[k] is the
// tensor that holds block k << shift, and one more entry closes the last bucket.
template <typename T>
unsigned make_hints(const std::vector<uint32_t>& first, int buckets, std::vector<T>* hint) {
    const uint32_t blocks = first.back();
    const int live = (int)first.size() - 1;
    unsigned shift = 0;
    while ((((uint64_t)blocks - 1) >> shift) + 1 > (uint64_t)buckets) ++shift;
    const uint32_t used = (uint32_t)((((uint64_t)blocks - 1) >> shift) + 1);
    hint->resize((size_t)used + 1);
    int l = 0;
    for (uint32_t k = 0; k < used; ++k) {
        const uint64_t pos = (uint64_t)k << shift;
        while ((uint64_t)first[(size_t)l + 1] <= pos) ++l;
        (*hint)[k] = (T)l;
    }
    (*hint)[used] = (T)(live - 1);
    return shift;
}

int run_multi(bool compress, const gact_tensor_desc* descs, int L, int group_size,
              void* d_workspace, size_t workspace_bytes, void* stream) {
    if (L < 0) return GACT_E_ARG;
    if (!group_ok(group_size)) return GACT_E_GROUP;
    if (L == 0) return GACT_OK;
    if (!descs) return GACT_E_ARG;
    gact::Geometry geo = make_geometry(group_size);

    // one contiguous staging image: table of the non-empty tensors, then the
    // first block of each, then the total
    std::vector<gact::TensorArgs> table;
    std::vector<uint32_t> first, tiles;
    table.reserve(L);
    first.reserve(L + 1);
    if (compress) tiles.reserve(L);
    uint64_t blocks = 0, bf16_blocks = 0;
    for (int l = 0; l < L; ++l) {
        const gact_tensor_desc& d = descs[l];
        if (d.bits == GACT_BITS_UNCOMPRESSED) {          // left uncompressed by the allocator
            if (d.n < 0) return GACT_E_ARG;
            continue;
        }
        gact::TensorArgs t;
        uint32_t its_tiles;
        const int rc = make_args(compress, d.x, d.packed, d.gmin, d.gscale, d.y, d.n, d.seed,
                                 compress ? d.index_base : 0, d.bits, d.dtype, geo, &t, &its_tiles);
        if (rc != GACT_OK) return rc;
        if (d.n == 0) continue;
        first.push_back((uint32_t)blocks);
        table.push_back(t);
        if (compress) tiles.push_back(its_tiles);
        geo.lds_wave_dwords = std::max(geo.lds_wave_dwords, gact::lds_dwords_per_wave(d.dtype));
        const uint64_t its_blocks = (uint64_t)blocks_for(compress ? gact::kCompressAny : gact::kDecompress, t, its_tiles);
        blocks += its_blocks;
        if (d.dtype == GACT_BF16) bf16_blocks += its_blocks;
        if (blocks > 0x7FFFFFFFull) return GACT_E_ARG;
    }
    const int live = (int)table.size();
    if (live == 0) return GACT_OK;
    gact::Work work = work_for(compress, geo);
    if (const gact::Work w = work_of_length(work, blocks, bf16_blocks, geo); w != work) {
        work = w;
        blocks = 0;
        for (int l = 0; l < live; ++l) {
            first[l] = (uint32_t)blocks;
            blocks += (uint64_t)blocks_for(work, table[l], compress ? tiles[l] : 0);
        }
    }
    first.push_back((uint32_t)blocks);

    if (!d_workspace || !aligned(d_workspace, 16) ||
        workspace_bytes < gact_multi_workspace_bytes(L))
        return GACT_E_ARG;

    if (live <= gact::kInlineTensors) {
        // small table: by value in the kernel arguments, nothing to upload
        gact::InlineTable tab;
        std::memset(&tab, 0, sizeof(tab));
        std::memcpy(tab.t, table.data(), (size_t)live * sizeof(gact::TensorArgs));
        std::memcpy(tab.first_block, first.data(), first.size() * sizeof(uint32_t));
        std::vector<uint8_t> hint;
        const unsigned shift = make_hints(first, gact::kInlineHints, &hint);
        for (size_t k = 0; k < hint.size(); ++k) tab.hint[k >> 2] |= (uint32_t)hint[k] << ((k & 3) * 8);
        return gact_launch_multi_inline(work, &tab, shift, &geo, (unsigned)blocks, stream) == 0
                   ? GACT_OK : GACT_E_HIP;
    }

    if (const int rc = refuse_if_capturing(stream)) return rc;
    std::vector<uint32_t> hint;
    const unsigned shift = make_hints(first, gact::hint_buckets(live), &hint);
    const size_t tb = table_bytes(live), fb = first_bytes(live);
    std::vector<unsigned char> image(tb + fb + hint.size() * sizeof(uint32_t));
    std::memcpy(image.data(), table.data(), (size_t)live * sizeof(gact::TensorArgs));
    std::memcpy(image.data() + tb, first.data(), first.size() * sizeof(uint32_t));
    std::memcpy(image.data() + tb + fb, hint.data(), hint.size() * sizeof(uint32_t));
    if (const int rc = upload(d_workspace, image.data(), image.size(), stream)) return rc;
    const unsigned char* base = (const unsigned char*)d_workspace;
    return gact_launch_multi(work, (const gact::TensorArgs*)base, (const uint32_t*)(base + tb),
                             (const uint32_t*)(base + tb + fb), shift, &geo, (unsigned)blocks,
                             stream) == 0 ? GACT_OK : GACT_E_HIP;
}

// ---------------------------------------------------------------- reductions
// The tag of one call's results (gact_sum.h): a number that no other call of this process has, spread over all
// 64 bits (the finaliser of splitmix64), never 0 (untagged) nor all ones (whose complement is).
uint64_t next_tag() {
    static std::atomic<uint64_t> calls{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count()};
    for (;;) {
        uint64_t z = calls.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        if (z != 0 && z != ~0ull) return z;
    }
}

size_t reduce_table_bytes(int K) {
    return ((size_t)K * sizeof(gact::ReduceArgs) + (size_t)(K + 1) * sizeof(uint32_t) + 15) / 16 * 16;
}

// What a reduction launch reads and where it leaves its per-block results.
struct Reduction {
    int K = 0;                                    // buffers that are not empty; 0: nothing to reduce
    unsigned blocks = 0;
    int bf16_chunks = 1;                          // statistics: chunks of a bf16 buffer per block
    gact::ReduceTable inline_table{};             // their table, when it fits the kernel arguments
    bool is_inline = false;
    const gact::ReduceArgs* d_table = nullptr;    // else uploaded to the workspace
    const uint32_t* d_first = nullptr;
    double* d_partial = nullptr;
    bool wide = false;                            // statistics: blocks of 1024 threads
    bool tagged = false;                          // room for two words per result: the launch adds them itself
    const gact::ReduceTable* table() const { return is_inline ? &inline_table : nullptr; }
};

// Builds the buffer table of a reduction launch and uploads it unless it is small.  The per-block
// results lie behind the table's place in the workspace either way.
int stage_reduction(const std::vector<gact::ReduceArgs>& bufs, bool statistics, void* d_workspace,
                    size_t workspace_bytes, void* stream, Reduction* red) {
    const int nout = statistics ? 2 : 1;
    std::vector<gact::ReduceArgs> live;
    std::vector<uint32_t> first;
    for (const gact::ReduceArgs& r : bufs)
        if (r.n != 0) live.push_back(r);
    const int K = (int)live.size();
    const size_t tb = reduce_table_bytes(K);
    uint64_t blocks = 0;
    // false: more blocks than a launch has
    const auto count = [&]() {
        first.clear();
        blocks = 0;
        for (const gact::ReduceArgs& r : live) {
            const int64_t chunk = statistics ? gact::stats_block_elems(r.dtype, red->bf16_chunks)
                                             : gact::reduce_chunk_elems(r.dtype);
            first.push_back((uint32_t)blocks);
            blocks += (uint64_t)((r.n + chunk - 1) / chunk);
            if (blocks > 0x7FFFFFFFull) return false;
        }
        first.push_back((uint32_t)blocks);
        return true;
    };
    const auto need = [&]() { return tb + (size_t)nout * blocks * sizeof(double); };
    bool fits = count();
    if (K == 0) return GACT_OK;
    if (statistics && (!fits || workspace_bytes < need())) {
        red->bf16_chunks = 2;
        fits = count();
    }
    if (!fits || !d_workspace || !aligned(d_workspace, 16) || workspace_bytes < need()) return GACT_E_ARG;
    if (const int rc = refuse_if_capturing(stream)) return rc;      // for both kinds of table
    red->K = K;
    red->blocks = (unsigned)blocks;
    red->d_partial = (double*)((unsigned char*)d_workspace + tb);
    red->wide = statistics && gact::wide_stats(blocks, (uint64_t)K) &&
                std::all_of(live.begin(), live.end(), [](const gact::ReduceArgs& r) { return r.dtype == GACT_F32 && aligned(r.b, 128); });
    red->tagged = !statistics && workspace_bytes >= tb + 2 * blocks * sizeof(double) &&
                  gact::room_for_adders<gact::kReduceWaves>(blocks);
    if (K <= gact::kInlineBuffers) {
        std::memcpy(red->inline_table.t, live.data(), (size_t)K * sizeof(gact::ReduceArgs));
        std::memcpy(red->inline_table.first_block, first.data(), first.size() * sizeof(uint32_t));
        red->is_inline = true;
        return GACT_OK;
    }
    std::vector<unsigned char> image(tb);
    std::memcpy(image.data(), live.data(), (size_t)K * sizeof(gact::ReduceArgs));
    std::memcpy(image.data() + (size_t)K * sizeof(gact::ReduceArgs), first.data(),
                first.size() * sizeof(uint32_t));
    if (const int rc = upload(d_workspace, image.data(), image.size(), stream)) return rc;
    red->d_table = (const gact::ReduceArgs*)d_workspace;
    red->d_first = (const uint32_t*)((const unsigned char*)d_workspace + (size_t)K * sizeof(gact::ReduceArgs));
    return GACT_OK;
}

// Address of `scratch` on the current device, looked up once per device.
int scratch_of_current_device(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static void* address[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GACT_E_HIP;
    std::lock_guard<std::mutex> hold(lock);
    if (!address[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GACT_E_HIP;
        address[dev] = p;
    }
    *out = address[dev];
    return GACT_OK;
}

// gact_compress_footprint on a caller workspace, or (limited = true) on the
// library's own scratch area, where a tensor that needs more is refused.
int compress_footprint(const void* d_x, gact_dtype dtype, int64_t n, int group_size, int bits,
                       uint64_t seed, void* d_packed, float* d_gmin, float* d_gscale, int n_samples,
                       double* d_footprint, void* d_workspace, size_t workspace_bytes, bool limited,
                       void* stream) {
    if (!bits_ok(bits)) return GACT_E_BITS;
    if (!group_ok(group_size)) return GACT_E_GROUP;
    if (n_samples < 0 || n_samples > 32768 || !d_footprint || !aligned(d_footprint, 8)) return GACT_E_ARG;
    gact::Geometry geo = make_geometry(group_size);
    geo.lds_wave_dwords = gact::lds_dwords_per_wave((int)dtype);
    gact::TensorArgs t;
    uint32_t tiles;
    const int rc = make_args(true, d_x, d_packed, d_gmin, d_gscale, nullptr, n, seed, 0, bits,
                             (int)dtype, geo, &t, &tiles);
    if (rc != GACT_OK) return rc;
    if (n == 0)
        return gact_launch_zero(d_footprint, 1 + n_samples, stream) == 0 ? GACT_OK : GACT_E_HIP;
    // The documented size, a sum per tile; one per block of four tiles is used.
    const size_t need = (size_t)tiles * sizeof(double);
    if (!d_workspace || !aligned(d_workspace, 16) || workspace_bytes < need)
        return limited ? GACT_E_SCRATCH : GACT_E_ARG;
    const int64_t blocks = blocks_for(gact::kCompressAny, t, tiles);
    if (blocks > 0x7FFFFFFFll) return GACT_E_ARG;
    // The launch adds its sums itself where the workspace has two words for each (all of the documented size
    // have from two tiles on) and the tag is this call's alone: not in a graph, whose replays share one, nor in
    // the library's scratch area, which calls that overlap in time may overwrite under each other.
    const uint64_t tag = next_tag();
    const bool tagged = !limited && workspace_bytes >= 2 * (size_t)blocks * sizeof(double) &&
                        gact::room_for_adders<gact::waves_per_block(gact::kCompressAny)>((uint64_t)blocks, n_samples) && !recorded(stream);
    if (gact_launch_compress_sum(&t, &geo, (unsigned)blocks, (double*)d_workspace, tagged, tag, n_samples, d_footprint,
                                 stream, nullptr) != 0)
        return GACT_E_HIP;
    if (tagged) return GACT_OK;
    const gact::ReduceArgs r{d_x, nullptr, n, (int32_t)dtype, 0};
    return gact_launch_footprint_finish(&r, (unsigned)blocks, (double*)d_workspace, tag, n_samples,
                                        d_footprint, stream) == 0 ? GACT_OK : GACT_E_HIP;
}

}  // namespace

extern "C" {

int gact_compress(const void* d_x, gact_dtype dtype, int64_t n, int group_size, int bits,
                  uint64_t seed, void* d_packed, float* d_gmin, float* d_gscale, void* stream) {
    if (!bits_ok(bits)) return GACT_E_BITS;
    if (!group_ok(group_size)) return GACT_E_GROUP;
    gact::Geometry geo = make_geometry(group_size);
    geo.lds_wave_dwords = gact::lds_dwords_per_wave((int)dtype);
    gact::TensorArgs t;
    uint32_t tiles;
    const int rc = make_args(true, d_x, d_packed, d_gmin, d_gscale, nullptr, n, seed, 0, bits,
                             (int)dtype, geo, &t, &tiles);
    if (rc != GACT_OK) return rc;
    return run_single(true, t, tiles, geo, stream);
}

int gact_decompress(const void* d_packed, const float* d_gmin, const float* d_gscale, int64_t n,
                    int group_size, int bits, void* d_y, gact_dtype dtype, void* stream) {
    if (!bits_ok(bits)) return GACT_E_BITS;
    if (!group_ok(group_size)) return GACT_E_GROUP;
    const gact::Geometry geo = make_geometry(group_size);
    gact::TensorArgs t;
    uint32_t tiles;
    const int rc = make_args(false, nullptr, const_cast<void*>(d_packed),
                             const_cast<float*>(d_gmin), const_cast<float*>(d_gscale), d_y, n, 0, 0,
                             bits, (int)dtype, geo, &t, &tiles);
    if (rc != GACT_OK) return rc;
    return run_single(false, t, tiles, geo, stream);
}

size_t gact_multi_workspace_bytes(int L) {
    if (L <= 0) return 0;
    return table_bytes(L) + first_bytes(L) + ((size_t)gact::hint_buckets(L) + 1) * sizeof(uint32_t);
}

int gact_compress_multi(const gact_tensor_desc* h_descs, int L, int group_size, void* d_workspace,
                        size_t workspace_bytes, void* stream) {
    return run_multi(true, h_descs, L, group_size, d_workspace, workspace_bytes, stream);
}

int gact_decompress_multi(const gact_tensor_desc* h_descs, int L, int group_size,
                          void* d_workspace, size_t workspace_bytes, void* stream) {
    return run_multi(false, h_descs, L, group_size, d_workspace, workspace_bytes, stream);
}

// -------------------------------------------------- sensitivity, statistics
size_t gact_reduce_workspace_bytes(int K, int64_t total_elems) {
    if (K < 0 || total_elems < 0) return 0;
    // every buffer rounds up to whole 4096-element chunks; two results per block
    const uint64_t blocks = (uint64_t)total_elems / 4096 + (uint64_t)K + 1;
    return reduce_table_bytes(K) + (size_t)(2 * blocks * sizeof(double)) + 16;
}

int gact_sensitivity(const gact_grad_pair* h_pairs, int K, int bits, double* d_out,
                     void* d_workspace, size_t workspace_bytes, void* stream) {
    if (!bits_ok(bits)) return GACT_E_BITS;
    if (K < 0 || !d_out || !aligned(d_out, 8) || (K > 0 && !h_pairs)) return GACT_E_ARG;
    std::vector<gact::ReduceArgs> bufs;
    for (int k = 0; k < K; ++k) {
        const gact_grad_pair& p = h_pairs[k];
        if (p.n < 0 || !dtype_ok(p.dtype)) return GACT_E_ARG;
        if (p.n > 0 && (!p.g0 || !p.g1 || !aligned(p.g0, 16) || !aligned(p.g1, 16))) return GACT_E_ARG;
        bufs.push_back(gact::ReduceArgs{p.g0, const_cast<void*>(p.g1), p.n, p.dtype, 0});
    }
    Reduction red;
    if (const int rc = stage_reduction(bufs, false, d_workspace, workspace_bytes, stream, &red)) return rc;
    if (red.K == 0)     // nothing to reduce: the result is zero
        return gact_launch_zero(d_out, 1, stream) == 0 ? GACT_OK : GACT_E_HIP;
    const double B = (double)((1 << bits) - 1);
    return gact_launch_diff_sq(red.table(), red.d_table, red.d_first, red.K, red.blocks, red.d_partial,
                               red.tagged, next_tag(), 0.5 * B * B, d_out, stream, nullptr) == 0 ? GACT_OK : GACT_E_HIP;
}

int gact_grad_stats_update(const gact_grad_stat* h_stats, int K, int64_t t, double* d_out,
                           void* d_workspace, size_t workspace_bytes, void* stream) {
    if (K < 0 || t < 1 || !d_out || !aligned(d_out, 8) || (K > 0 && !h_stats)) return GACT_E_ARG;
    std::vector<gact::ReduceArgs> bufs;
    for (int k = 0; k < K; ++k) {
        const gact_grad_stat& p = h_stats[k];
        if (p.n < 0 || !dtype_ok(p.dtype)) return GACT_E_ARG;
        if (p.n > 0 && (!p.g || !p.mean || !aligned(p.g, 16) || !aligned(p.mean, 16))) return GACT_E_ARG;
        bufs.push_back(gact::ReduceArgs{p.g, p.mean, p.n, p.dtype, 0});
    }
    Reduction red;
    if (const int rc = stage_reduction(bufs, true, d_workspace, workspace_bytes, stream, &red)) return rc;
    if (red.K == 0) return gact_launch_zero(d_out, 2, stream) == 0 ? GACT_OK : GACT_E_HIP;
    const float rt = (float)(1.0 / (double)t);
    return gact_launch_grad_stats(red.table(), red.d_table, red.d_first, red.K, rt, red.bf16_chunks, red.wide, red.blocks,
                                  red.d_partial, next_tag(), d_out, stream) == 0 ? GACT_OK : GACT_E_HIP;
}

int gact_footprint(const void* d_x, gact_dtype dtype, int64_t n, int n_samples, double* d_out,
                   void* d_workspace, size_t workspace_bytes, void* stream) {
    if (n < 0 || n_samples < 0 || n_samples > 32768 || !dtype_ok((int)dtype) || !d_out ||
        !aligned(d_out, 8))
        return GACT_E_ARG;
    if (n == 0) return gact_launch_zero(d_out, 1 + n_samples, stream) == 0 ? GACT_OK : GACT_E_HIP;
    if (!d_x || !aligned(d_x, 16)) return GACT_E_ARG;
    const int64_t chunk = gact::reduce_chunk_elems((int)dtype);
    const int64_t blocks = (n + chunk - 1) / chunk;
    if (blocks > 0x7FFFFFFFll) return GACT_E_ARG;
    if (!d_workspace || !aligned(d_workspace, 16) ||
        workspace_bytes < (size_t)blocks * sizeof(double))
        return GACT_E_ARG;
    const gact::ReduceArgs r{d_x, nullptr, n, (int32_t)dtype, 0};
    return gact_launch_footprint(&r, (unsigned)blocks, (double*)d_workspace, next_tag(), n_samples, d_out,
                                 stream, nullptr) == 0 ? GACT_OK : GACT_E_HIP;
}

size_t gact_compress_footprint_workspace_bytes(int64_t n, int group_size) {
    if (n <= 0 || !group_ok(group_size)) return 0;
    return (size_t)tiles_for(n, make_geometry(group_size)) * sizeof(double);
}

int gact_compress_footprint(const void* d_x, gact_dtype dtype, int64_t n, int group_size, int bits,
                            uint64_t seed, void* d_packed, float* d_gmin, float* d_gscale,
                            int n_samples, double* d_footprint, void* d_workspace,
                            size_t workspace_bytes, void* stream) {
    return compress_footprint(d_x, dtype, n, group_size, bits, seed, d_packed, d_gmin, d_gscale,
                              n_samples, d_footprint, d_workspace, workspace_bytes, false, stream);
}

// The address a kernel can use for `p`: device memory as it is; host memory only when it is pinned
// and mapped into the device's address space.  nullptr when a kernel must not touch it.
static void* device_visible(const void* p) {
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();                      // an ordinary host pointer: not an error state to keep
        return nullptr;
    }
    return attr.devicePointer;
}

int gact_copy_bounded(void* dst, const void* src, size_t nbytes, int workgroups, void* stream) {
    if (workgroups < 1 || workgroups > 1024 || (nbytes > 0 && (!dst || !src))) return GACT_E_ARG;
    if (nbytes == 0) return GACT_OK;
    if (!aligned(dst, 16) || !aligned(src, 16)) return GACT_E_ARG;
    void* d = device_visible(dst);
    const void* s = device_visible(src);
    if (!d || !s) return GACT_E_ARG;
    return gact_launch_copy(d, s, (uint64_t)nbytes, (unsigned)workgroups, stream) == 0 ? GACT_OK : GACT_E_HIP;
}

int gact_compress_footprint_noalloc(const void* d_x, gact_dtype dtype, int64_t n, int group_size,
                                    int bits, uint64_t seed, void* d_packed, float* d_gmin,
                                    float* d_gscale, int n_samples, double* d_footprint,
                                    void* stream) {
    void* area = nullptr;
    if (const int rc = scratch_of_current_device(&area)) return rc;
    return compress_footprint(d_x, dtype, n, group_size, bits, seed, d_packed, d_gmin, d_gscale,
                              n_samples, d_footprint, area, GACT_NOALLOC_SCRATCH_BYTES, true, stream);
}

}  // extern "C"
