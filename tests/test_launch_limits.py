"""The choices that a launch's size makes, on the host, at the sizes where the runtime takes no more threads (2^32) and
where one form gives way to the next."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2206_11357_amd", "csrc")

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include "gact_device.h"
#include "gact_sum.h"
static int failed = 0;
#define CHECK(X) do { if (!(X)) { std::printf("line %d: %s\n", __LINE__, #X); failed = 1; } } while (0)
template <int WAVES>
void adders() {
    const uint64_t end = (1ull << 32) / (64 * WAVES);              // blocks that the runtime does not take
    uint64_t most = 0;
    for (uint64_t b = end - 20000; b <= end + 20000; ++b) {
        const uint64_t with = b + ((b + 511) / 512 + WAVES - 1) / WAVES;
        CHECK(gact::room_for_adders<WAVES>(b) == (with < end));
        if (gact::room_for_adders<WAVES>(b)) most = b;
        CHECK(gact::room_for_adders<WAVES>(b, 1000) == (with + (1000 + 64 * WAVES - 1) / (64 * WAVES) < end));
    }
    CHECK(most < end && most + most / (512 * WAVES) + 2 >= end);
    for (uint64_t b : {(uint64_t)1, (uint64_t)511, (uint64_t)100000}) CHECK(gact::room_for_adders<WAVES>(b));
    for (uint64_t b : {end, (uint64_t)0x70000000, (uint64_t)0x7FFFFFFF, (uint64_t)1 << 32, ((uint64_t)1 << 32) + 1}) CHECK(!gact::room_for_adders<WAVES>(b));
}
int main() {
    const uint64_t least = gact::kWideStats, end = 1ull << 22;     // 2^32 threads in blocks of 1024
    CHECK(!gact::wide_stats(1, 1) && !gact::wide_stats(least - 1, 1) && gact::wide_stats(least, 1));
    CHECK(gact::wide_stats(end - 1, 1) && !gact::wide_stats(end, 1) && !gact::wide_stats((1ull << 23) - 1, 1) && !gact::wide_stats(0x7FFFFFFFull, 1));
    for (uint64_t b = 1; b < 1ull << 31; b += 4093)
        CHECK(!gact::wide_stats(b, 1) || b * gact::stats_threads(true) < 1ull << 32);
    // many small buffers: a block that is short of its buffer's search
    CHECK(gact::wide_stats(24 * 1000, 1000) && !gact::wide_stats(24 * 1000 - 1, 1000) && !gact::wide_stats(9000, 9000));
    CHECK(!gact::wide_stats(least, least) && gact::wide_stats(least, 312));
    CHECK(gact::launchable((1ull << 23) - 1, gact::stats_threads(false)));
    // a sample point a thread, whatever the number of sums
    CHECK(gact::samplers_for<4>(0) == 0 && gact::samplers_for<4>(1) == 1 && gact::samplers_for<4>(256) == 1);
    CHECK(gact::samplers_for<4>(257) == 2 && gact::samplers_for<4>(32768) == 128);
    adders<gact::kReduceWaves>();
    adders<gact::waves_per_block(gact::kCompressAny)>();
    // long compressing launches: of fp32 alone, or nearly so, not in tiles of 55 to 63 lanes
    for (uint64_t b : {gact::kLongCompress, (uint64_t)1000000, (uint64_t)0x7FFFFFFF / 4})
        for (int lanes = 44; lanes <= 64; ++lanes) {
            CHECK(gact::long_compress(b, 0, lanes) == (lanes < 55 || lanes == 64));
            CHECK(gact::long_compress(b, (b + 3) / 4 - 1, lanes) == (lanes < 55 || lanes == 64));
            CHECK(gact::long_compress(b, (b + 3) / 4, lanes) && gact::long_compress(b, b - 1, lanes));
        }
    for (uint64_t b : {(uint64_t)0, gact::kLongCompress - 1, (uint64_t)0x7FFFFFFF / 4 + 1})
        CHECK(!gact::long_compress(b, b / 2, 64) && !gact::long_compress(b, 0, 64) && !gact::long_compress(b, 0, 52));
    // blocks of a decompressed tensor: as by a division
    for (int dtype : {GACT_DT_F32, GACT_DT_BF16})
        for (int bits : {1, 2, 4, 8})
            for (uint32_t table : {gact::kDecUnitsBf16, gact::kDecUnitsBf16Short}) {
                const int64_t span = gact::dec_block_elems(dtype, bits, table);
                for (int64_t base : {(int64_t)0, 3 * span, 1000003 * span, ((int64_t)1 << 42) / span * span})
                    for (int64_t n = base > 9 ? base - 9 : 1; n < base + 9000; ++n) CHECK(gact::dec_blocks(n, dtype, bits, table) == (n + span - 1) / span);
            }
    // the compressor of long launches takes at most four blocks of 64 threads for each of 256
    CHECK(4 * 64 * gact::waves_per_block(gact::kCompressLong) == 64 * gact::waves_per_block(gact::kCompressAny));
    return failed;
}
"""


def test_launches_keep_to_what_the_runtime_takes(tmp_path):
    src, exe = tmp_path / "limits.cpp", tmp_path / "limits"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout
