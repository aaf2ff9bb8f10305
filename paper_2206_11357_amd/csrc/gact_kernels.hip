// GACT activation compressor / decompressor for MI355X (gfx950, wave64).
//
// What is computed: the per-group stochastic-rounding quantizer of
// arXiv 2206.11357 (App. A.4, applied per group as in Sec. 5) and its inverse;
// the exact arithmetic contract is stated in include/gact.h.
//
// How the work is laid out
//   Compress
//   * One wavefront owns one "tile": 64 lanes x 32 consecutive elements
//     (2048 elements when the group size is a power of two).  A group of G
//     elements is G/32 neighbouring lanes, so group statistics are a handful
//     of DPP steps and every lane does the two IEEE divisions of its group
//     once per 32 elements.
//   * HBM is read with fully coalesced 16-byte loads (lane i of load k reads
//     bytes [k*1024 + 16 i, +16)).  The switch from that layout to "32
//     consecutive elements per lane" goes through a private LDS region per
//     wavefront, in the input's own format (8 KB for fp32, 4 KB for bf16; the
//     16-byte pieces of a row are XOR-swizzled so that 128-bit LDS reads and
//     writes are conflict-free without padding).  The LDS a wavefront holds
//     bounds how many are resident, so the launch sizes it by the widest dtype
//     present.
//   * With 32 elements per lane a lane owns 32*bits packed bits = `bits`
//     dwords, and neighbouring lanes own neighbouring dwords: the packed
//     stream is written coalesced without further staging.
//   * Rounding noise: one Philox4x32-10 block per 8 consecutive elements, so
//     four blocks per lane; the stream depends on (seed, element index) only.
//   Decompress
//   * No layout switch and no LDS: a lane produces one 16-byte piece of output
//     per coalesced store and fetches that piece's codes with one small load.
//   * No MFMA anywhere: the path is a streaming codec, bound by HBM (fp32) or
//     by plain VALU work (bf16 compress), not a contraction.
//
// Three instantiations of the same code (TileKind): full tiles of power-of-two
// group sizes, full tiles of the other group sizes, and the guarded one for the
// end of a tensor.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gact_device.h"
#include "gact_sum.h"

namespace gact {

typedef float    f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

constexpr int kLanes        = 64;
constexpr int kPerLane      = 32;                 // consecutive elements one lane owns
constexpr int kWavesPerBlk  = 4;
constexpr int kBlockThreads = kLanes * kWavesPerBlk;

// 32-bit words of the packed buffer: ceil(n*bits/8) bytes rounded up to 16
__device__ __forceinline__ int64_t packed_words(const TensorArgs& t) {
    return (int64_t)((((uint64_t)t.n * (uint64_t)t.bits() + 127u) >> 7) << 2);
}

// ---------------------------------------------------------------- lane moves
__device__ __forceinline__ float swizzle_xor16(float v) {
    // bit-mask mode: and 0x1f, or 0, xor 0x10 (lane ^ 16 inside each half wave)
    return __builtin_bit_cast(
        float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), (16 << 10) | 0x1F));
}
__device__ __forceinline__ float lane_read(float v, int src_lane) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_ds_bpermute(src_lane << 2, __builtin_bit_cast(int, v)));
}

// min / max of finite values (v_min_f32 / v_min3_f32).  The sign of a zero
// result is not defined by these; the stored minimum is canonicalised later.
__device__ __forceinline__ float fmin2(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float fmax2(float a, float b) { return __builtin_fmaxf(a, b); }

// v = min / max(v, v of the DPP-selected lane) in one instruction.  Written as
// assembly because the compiler otherwise moves the DPP operand into its own
// register and re-canonicalises both inputs (4 instructions per step).
// A DPP operand must not be read in the two issue slots after a vector
// instruction has written it, and the compiler's hazard pass does not look
// inside an assembly statement, so each statement brings its own wait states.
#define GACT_DPP_MINMAX(NAME, OP, CTRL)                                                  \
    __device__ __forceinline__ float NAME(float v) {                                     \
        float r;                                                                          \
        asm("s_nop 1\n\t" OP " %0, %1, %1 " CTRL " row_mask:0xf bank_mask:0xf"          \
            : "=v"(r) : "v"(v));                                                          \
        return r;                                                                         \
    }
GACT_DPP_MINMAX(min_xor1, "v_min_f32_dpp", "quad_perm:[1,0,3,2]")
GACT_DPP_MINMAX(max_xor1, "v_max_f32_dpp", "quad_perm:[1,0,3,2]")
GACT_DPP_MINMAX(min_xor2, "v_min_f32_dpp", "quad_perm:[2,3,0,1]")
GACT_DPP_MINMAX(max_xor2, "v_max_f32_dpp", "quad_perm:[2,3,0,1]")
GACT_DPP_MINMAX(min_half_mirror, "v_min_f32_dpp", "row_half_mirror")
GACT_DPP_MINMAX(max_half_mirror, "v_max_f32_dpp", "row_half_mirror")
GACT_DPP_MINMAX(min_mirror, "v_min_f32_dpp", "row_mirror")
GACT_DPP_MINMAX(max_mirror, "v_max_f32_dpp", "row_mirror")
#undef GACT_DPP_MINMAX

// All lanes of a group (lpg neighbouring lanes, lpg a power of two <= 32,
// groups aligned to lpg) end up with the group's min and max.  After the two
// quad steps all lanes of a quad agree, so the 8- and 16-lane mirrors pair
// each lane with one from the other half.
__device__ __forceinline__ void group_minmax_pow2(float& mn, float& mx, int lpg) {
    if (lpg > 1)  { mn = min_xor1(mn);        mx = max_xor1(mx); }
    if (lpg > 2)  { mn = min_xor2(mn);        mx = max_xor2(mx); }
    if (lpg > 4)  { mn = min_half_mirror(mn); mx = max_half_mirror(mx); }
    if (lpg > 8)  { mn = min_mirror(mn);      mx = max_mirror(mx); }
    if (lpg > 16) { mn = fmin2(mn, swizzle_xor16(mn)); mx = fmax2(mx, swizzle_xor16(mx)); }
}

// Any lpg in [1, 32], groups at multiples of lpg.  A lane that holds the minimum
// of `w` lanes of its group, counted from itself and around the group's end, takes
// the one of the lane min(w, lpg - w) further on: ceil(log2 lpg) steps, windows that
// overlap do no harm.  Lanes past the last whole group read wrapped lanes, unused.
__device__ __forceinline__ void group_minmax_any(float& mn, float& mx, const Geometry& geo, int lane) {
    const int lpg = geo.lpg;
    const int first = (int)(((uint32_t)lane * (uint32_t)geo.lpg_magic) >> 16) * lpg;
    const int pos = lane - first;
    for (int w = 1; w < lpg;) {
        const int step = w < lpg - w ? w : lpg - w;
        const int next = pos + step;
        const int src = first + (next >= lpg ? next - lpg : next);
        const float a = lane_read(mn, src), b = lane_read(mx, src);
        mn = fmin2(mn, a);
        mx = fmax2(mx, b);
        w += step;
    }
}

// ------------------------------------------------------------------- Philox
// Philox4x32-10 (Salmon et al., SC'11) on counter (c0, c1, 0, 0), key (k0, k1).
constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// three-input xor in one v_bitop3_b32 (truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// rounds FIRST .. 9 (round r uses the key bumped r times)
template <int FIRST>
__device__ __forceinline__ void philox_rounds(uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3,
                                              uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = FIRST; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0 + (uint32_t)r * kPhiloxW0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1 + (uint32_t)r * kPhiloxW1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
}

// Rounds 0..2 of a block whose counter is (c0, c1u, 0, 0) with the high word c1u
// and the key uniform over the wavefront -- the case for every block of a tile
// unless the low counter word wraps inside the tile.  Counter words 2 and 3
// being zero, part of these rounds is the same for every lane and is computed
// once per wavefront, on the scalar unit (PhiloxUniform):
//   round 0: M1 * 0 = 0, so word 0 becomes c1u ^ k0 (uniform) and word 1 is 0;
//   round 1: M0 * (uniform word 0) is a scalar product; its low half is the
//            new, uniform, word 3;
//   round 2: the uniform word 3 and the key fold into one scalar operand.
// Four 32 x 32 -> 64 multiplies per block instead of six.
struct PhiloxUniform {
    uint32_t f2, g2;
    __device__ __forceinline__ PhiloxUniform(uint32_t c1u, uint32_t k0, uint32_t k1) {
        const uint32_t a0 = c1u ^ k0;                                      // round 0, word 0
        const uint64_t P0 = (uint64_t)kPhiloxM0 * a0;                       // round 1 product
        f2 = (uint32_t)(P0 >> 32) ^ (k1 + kPhiloxW1);                       // round 1: word 2 = f2 ^ old word 3
        g2 = (uint32_t)P0 ^ (k1 + 2u * kPhiloxW1);                          // round 2: word 2 = hi(M0 word 0) ^ g2
    }
};
__device__ __forceinline__ void philox_head_uniform(uint32_t c0, const PhiloxUniform& u, uint32_t k0,
                                                    uint32_t k1, uint32_t st[4]) {
    const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;                           // round 0
    const uint32_t a2 = (uint32_t)(p0 >> 32) ^ k1;
    const uint32_t a3 = (uint32_t)p0;
    const uint64_t p1 = (uint64_t)kPhiloxM1 * a2;                           // round 1
    const uint32_t b0 = (uint32_t)(p1 >> 32) ^ (k0 + kPhiloxW0);
    const uint32_t b1 = (uint32_t)p1;
    const uint32_t b2 = a3 ^ u.f2;
    const uint64_t q0 = (uint64_t)kPhiloxM0 * b0;                           // round 2
    const uint64_t q1 = (uint64_t)kPhiloxM1 * b2;
    st[0] = xor3((uint32_t)(q1 >> 32), b1, k0 + 2u * kPhiloxW0);
    st[1] = (uint32_t)q1;
    st[2] = (uint32_t)(q0 >> 32) ^ u.g2;
    st[3] = (uint32_t)q0;
}

// The same three rounds for any per-lane 64-bit block number.
__device__ __forceinline__ void philox_head_any(uint64_t blk, uint32_t k0, uint32_t k1, uint32_t st[4]) {
    uint32_t c0 = (uint32_t)blk, c1 = (uint32_t)(blk >> 32), c2 = 0u, c3 = 0u;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0 + (uint32_t)r * kPhiloxW0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1 + (uint32_t)r * kPhiloxW1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    st[0] = c0; st[1] = c1; st[2] = c2; st[3] = c3;
}

// Three-input min / max of finite values.  As assembly because the compiler
// puts a canonicalising v_max_f32 x, x in front of values it cannot prove to be
// free of signalling NaNs (everything that was widened from bf16 with bit
// operations); non-finite input is outside the contract.
__device__ __forceinline__ float fmin3(float a, float b, float c) {
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float fmax3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// x[j] <- x[j] + b[j % 4] for eight values, rounded toward minus infinity.  The
// wavefront's binary32 rounding mode (MODE bits 1:0) is switched to round-down
// for exactly these eight additions and back to nearest-even; the block is one
// volatile statement, so no other floating-point instruction can be scheduled
// into it and everything outside keeps the nearest-even contract.
__device__ __forceinline__ void add8_round_down(float (&x)[8], float b0, float b1, float b2, float b3) {
    asm volatile(
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 2\n\t"
        "v_add_f32 %0, %8, %0\n\t"
        "v_add_f32 %1, %9, %1\n\t"
        "v_add_f32 %2, %10, %2\n\t"
        "v_add_f32 %3, %11, %3\n\t"
        "v_add_f32 %4, %8, %4\n\t"
        "v_add_f32 %5, %9, %5\n\t"
        "v_add_f32 %6, %10, %6\n\t"
        "v_add_f32 %7, %11, %7\n\t"
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
        : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7])
        : "s"(b0), "s"(b1), "s"(b2), "s"(b3));
}

// Instructions the compiler does not select on its own.
// floor(x) as int32 in one instruction.
__device__ __forceinline__ int32_t cvt_floor_i32(float x) {
    int32_t r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
// M * (low / high 16 bits of w) + c
template <int M>
__device__ __forceinline__ uint32_t mad_lo16(uint32_t w, uint32_t c) {
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, %3, %2" : "=v"(r) : "v"(w), "v"(c), "n"(M));
    return r;
}
template <int M>
__device__ __forceinline__ uint32_t mad_hi16(uint32_t w, uint32_t c) {
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, %3, %2 op_sel:[1,0,0,0]" : "=v"(r) : "v"(w), "v"(c), "n"(M));
    return r;
}
// bits of a where m is set, of b elsewhere
__device__ __forceinline__ uint32_t select_bits(uint32_t m, uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
}

// ------------------------------------------------------- tile <-> HBM moves
// The raw 16-byte loads of one tile: fp32 8 per lane, bf16 4 per lane.
template <int DT>
struct RawTile {
    u4 r[DT == GACT_DT_F32 ? 8 : 4];
};

// What a wavefront's tile is:
//   kFull     2048 elements, group size a power of two
//   kFullAny  lanes_used * 32 elements (44 to 63 lanes hold data), any group size;
//             not the tensor's last tile
//   kEdge     anything else: the end of a tensor, or a tile in which the low word of
//             the Philox block number wraps
// Before kFullAny, all tiles of a group size that is no power of two were guarded
// ones, whose branches per element and scan over the group's lanes made the launch
// bound by instruction issue: 130 M fp32 elements, G = 96, 2 bits 90.6 -> 71.1 us
// (4.7 -> 6.0 TB/s), 1.0 G bf16 elements, G = 224, 3 bits 779 -> 511 us.
enum TileKind { kFull, kFullAny, kEdge };

// element i of x as a 32-bit word (bf16 in the low half)
template <int DT>
__device__ __forceinline__ uint32_t load_element(const void* __restrict__ x, int64_t i) {
    return DT == GACT_DT_F32 ? ((const uint32_t*)x)[i] : (uint32_t)((const uint16_t*)x)[i];
}

// Coalesced global loads.  `ne` = number of valid elements of the tile.  The pieces
// that hold none of them repeat the last whole one, which no HBM traffic follows, so
// that all loads go out without a branch between them; kEdge puts the piece that `ne`
// cuts together from single elements (never read past `ne`), the same for all lanes.
template <int DT, TileKind KIND>
__device__ __forceinline__ void load_tile(const void* __restrict__ x, int64_t e0, int ne, int lane,
                                          RawTile<DT>& raw) {
    constexpr int P = DT == GACT_DT_F32 ? 4 : 8, kLoads = DT == GACT_DT_F32 ? 8 : 4;
    const uint8_t* p = (const uint8_t*)x + e0 * (16 / P);
    const int whole = KIND == kEdge ? ne & ~(P - 1) : ne;      // elements in whole pieces
    if (KIND != kEdge || whole > 0) {
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            int e = (k * 64 + lane) * P;
            if (KIND != kFull) e = e < whole - P ? e : whole - P;
            raw.r[k] = __builtin_nontemporal_load((const u4*)(p + e * (16 / P)));
        }
    } else {
#pragma unroll
        for (int k = 0; k < kLoads; ++k) raw.r[k] = u4{0u, 0u, 0u, 0u};
    }
    if (KIND == kEdge && whole != ne) {
        uint32_t h[P];
#pragma unroll
        for (int j = 0; j < P; ++j) h[j] = load_element<DT>(x, e0 + (whole + j < ne ? whole + j : ne - 1));
        u4 t;
        if (DT == GACT_DT_F32) t = u4{h[0], h[1], h[2], h[3]};
        else t = u4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4 % P] | (h[5 % P] << 16), h[6 % P] | (h[7 % P] << 16)};
#pragma unroll
        for (int k = 0; k < kLoads; ++k)
            if ((k * 64 + lane) * P == whole) raw.r[k] = t;
    }
}

// Raw tile -> LDS rows (row r = elements 32 r .. 32 r + 31) in the input's own
// format: 8 (fp32) or 4 (bf16) pieces of 16 bytes per row.  Staging bf16
// unwidened halves the LDS a wavefront holds, which is what bounds the number
// of resident wavefronts.  Rows are not padded; piece p of row r sits at slot
// p ^ s(r), with s(r) = (r >> 1) & 7 for fp32 and (r >> 2) & 3 for bf16.  A
// 128-bit LDS access is served 16 lanes at a time over 64 banks:
//   * writes: 16 neighbouring lanes hold 16 consecutive pieces, i.e. all slots
//     of 2 (4) neighbouring rows that share s(r) -> 16 distinct bank quads;
//   * reads: 16 neighbouring lanes read the same piece index of 16 consecutive
//     rows; the row's own offset covers 2 (4) bank quads and s(r) runs through
//     the 8 (4) values that complete them.
template <int DT>
__device__ __forceinline__ void stage_tile(const RawTile<DT>& raw, uint32_t* __restrict__ lds,
                                           int lane) {
    if (DT == GACT_DT_F32) {
        // load k, lane L: row 8 k + L / 8, piece L % 8, s = (4 k + L / 16) & 7
        uint32_t* base = lds + (lane >> 3) * 32;
        const int slot0 = ((lane & 7) ^ (lane >> 4)) * 4;          // even k
        const int slot1 = slot0 ^ 16;                              // odd k
#pragma unroll
        for (int k = 0; k < 8; ++k)
            *(u4*)(base + k * 256 + ((k & 1) ? slot1 : slot0)) = raw.r[k];
    } else {
        // load k, lane L: row 16 k + L / 4, piece L % 4, s = (L / 16) & 3
        uint32_t* base = lds + (lane >> 2) * 16 + (((lane & 3) ^ (lane >> 4)) * 4);
#pragma unroll
        for (int k = 0; k < 4; ++k) *(u4*)(base + k * 256) = raw.r[k];
    }
}

// The lane's own row as fp32; bf16 is widened here, exactly.
template <int DT>
__device__ __forceinline__ void read_row(const uint32_t* __restrict__ lds, int row, float v[kPerLane]) {
    if (DT == GACT_DT_F32) {
        const uint32_t first = (uint32_t)row * 32u + (((uint32_t)row >> 1) & 7u) * 4u;   // piece 0
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const f4 q = *(const f4*)(lds + (first ^ (uint32_t)(4 * k)));
            v[4 * k + 0] = q.x; v[4 * k + 1] = q.y; v[4 * k + 2] = q.z; v[4 * k + 3] = q.w;
        }
    } else {
        const uint32_t first = (uint32_t)row * 16u + (((uint32_t)row >> 2) & 3u) * 4u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u4 w = *(const u4*)(lds + (first ^ (uint32_t)(4 * k)));
            const uint32_t h[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[8 * k + 2 * j + 0] = __builtin_bit_cast(float, h[j] << 16);
                v[8 * k + 2 * j + 1] = __builtin_bit_cast(float, h[j] & 0xFFFF0000u);
            }
        }
    }
}

// two fp32 -> two bf16 (low half = a), round to nearest even: v_cvt_pk_bf16_f32
typedef float  f2v  __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair_rne(float a, float b) {
    const f2v v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2v));
}

__device__ __forceinline__ void wave_lds_sync() {
    // LDS operations of one wavefront execute in order; this only stops the
    // compiler from moving LDS accesses across the layout switch.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// range / (2^BITS - 1), correctly rounded, for range >= 2^-100: a product with the rounded reciprocal
// and one fused correction (P. Markstein, IBM J. Res. Dev. 34 (1990) 111: four instructions with the
// fix-up instead of the eleven of a general division).  Every significand was compared with the division
// on the host for the divisors 3, 15 and 255; the result does not depend on the exponent as long as the
// remainder (down to 2^-149) and the quotient are exact.  The fix-up gives an infinite range, whose
// correction is inf - inf, its infinite quotient.
template <int BITS>
__device__ __forceinline__ float div_levels(float range) {
    constexpr float Bf = (float)((1u << BITS) - 1u), r = 1.0f / Bf;
    if (BITS == 1) return range;
    const float q = range * r;
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-q, Bf, range), r, q), Bf, range);
}

// Eight 4-bit fields, each in bits 17..20 of its word, to one word: field k in bits 4k..4k+3.
// Byte 2 of a word holds its field; three byte permutes gather four of them.
__device__ __forceinline__ uint32_t gather_nibbles(const uint32_t (&n)[8]) {
    uint32_t d[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        d[h] = __builtin_amdgcn_perm(n[2 + h], n[0 + h], 0x0C0C0602u);
        d[h] = __builtin_amdgcn_perm(n[4 + h], d[h], 0x0C060100u);
        d[h] = __builtin_amdgcn_perm(n[6 + h], d[h], 0x06020100u);
    }
    return select_bits(0x0F0F0F0Fu, d[0] >> 1, d[1] << 3);
}

// every BITS-wide field f of w replaced by -f modulo 2^BITS
template <int BITS>
__device__ __forceinline__ uint32_t negate_fields(uint32_t w) {
    if (BITS == 1) return w;
    constexpr uint32_t one = BITS == 2 ? 0x55555555u : 0x11111111u, top = one << (BITS - 1);
    return ((~w & ~top) + one) ^ (~w & top);
}

// ----------------------------------------------------------------- compress
// What a tile leaves beside its codes (SUM): the sum of its elements; and the word at `look`, if any, as it was when the
// tile's loads were out (gact_sum.h), for the load to be in nobody's way.
struct TileOut {
    const uint64_t* look = nullptr;
    double   sum = 0.0;
    uint64_t word = 0;
};

// One wavefront compresses tile `tile` of tensor `t`.
//   geo.lpg        lanes per group (G/32)
//   geo.lanes_used lanes that hold data in a full tile (64 for power-of-two G)
//   SUM            also return the binary64 sum of the tile's elements in out_sum (the
//                  footprint of Sec. 5.2 from the same read)
template <int DT, int BITS, TileKind KIND, bool SUM>
__device__ __forceinline__ void compress_tile(const TensorArgs& t, const Geometry& geo,
                                              int64_t tile, uint32_t* __restrict__ lds, int lane,
                                              TileOut& out_sum) {
    constexpr uint32_t B = (1u << BITS) - 1u;
    const int tile_elems = geo.lanes_used * kPerLane;
    const int64_t e0 = tile * (int64_t)tile_elems;       // `tile` is uniform over the wavefront
    int ne = tile_elems;
    if (KIND == kEdge) {
        const int64_t left = t.n - e0;
        ne = left < (int64_t)tile_elems ? (int)left : tile_elems;
    }

    RawTile<DT> raw;
    load_tile<DT, KIND>(t.io, e0, ne, lane, raw);
    if (SUM && out_sum.look) out_sum.word = load_word(out_sum.look);

    uint32_t last_word = 0u;                         // the tile's last valid element
    if (KIND == kEdge) last_word = load_element<DT>(t.io, e0 + ne - 1);

    // Noise of the lane's 32 elements, while the loads are in flight: block numbers
    // tile_blk + 4 lane + (0..3).
    const uint64_t tile_blk = t.blk_base() + ((uint64_t)e0 >> 3);
    // The key passes through an empty statement: otherwise the twenty round keys are computed once,
    // ahead of the switch over the instantiations, and spill to vector registers from there.
    uint32_t k0 = t.seed_lo, k1 = t.seed_hi;
    asm volatile("" : "+s"(k0), "+s"(k1));
    // All four blocks for fp32; two (one) for bf16, whose 64 registers hold no more without spilling.
    constexpr int kEarly = DT == GACT_DT_F32 ? 4 : KIND == kEdge ? 1 : 2;
    uint32_t noise[4][4];
    const PhiloxUniform pu((uint32_t)(tile_blk >> 32), k0, k1);
    const uint32_t lane_c0 = (uint32_t)tile_blk + 4u * (uint32_t)lane;
    const auto draw = [&](int c, uint32_t (&r)[4]) {
        if (KIND == kEdge) philox_head_any(tile_blk + (uint64_t)(4 * lane + c), k0, k1, r);
        else philox_head_uniform(lane_c0 + (uint32_t)c, pu, k0, k1, r);
        philox_rounds<3>(r[0], r[1], r[2], r[3], k0, k1);
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 4 - kEarly; c < 4; ++c) draw(c, noise[c]);
    __builtin_amdgcn_sched_barrier(0);

    // layout switch: coalesced rows in, 32 consecutive elements per lane out
    float v[kPerLane];
    stage_tile<DT>(raw, lds, lane);
    wave_lds_sync();
    read_row<DT>(lds, lane, v);

    const int my0 = lane * kPerLane;                 // first element of this lane in the tile
    const int left = ne - my0;                       // its valid elements, if fewer than 32
    if (SUM) {
        // lane: its 32 elements in index order; wavefront: xor butterfly 32, 16, ... 1
        int left_here = left;                        // opaque: the 32 masks are not kept, they would spill
        if (KIND == kEdge) asm volatile("" : "+v"(left_here));
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j)
            if (KIND == kFull || j < left_here) acc += (double)v[j];
        out_sum.sum = add_lanes(acc);
    }

    // Places past the end take the last valid element: it belongs to the last group, whose minimum and
    // maximum a copy does not change.  (Groups with no valid element at all are not stored.)
    if (KIND == kEdge) {
        const float last = __builtin_bit_cast(float, DT == GACT_DT_F32 ? last_word : last_word << 16);
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) v[j] = j < left ? v[j] : last;
    }

    // group statistics
    float mn = fmin3(v[0], v[1], v[2]), mx = fmax3(v[0], v[1], v[2]);
#pragma unroll
    for (int j = 3; j + 1 < kPerLane; j += 2) { mn = fmin3(mn, v[j], v[j + 1]); mx = fmax3(mx, v[j], v[j + 1]); }
    mn = fmin3(mn, v[kPerLane - 1], v[kPerLane - 1]); mx = fmax3(mx, v[kPerLane - 1], v[kPerLane - 1]);
    if (KIND == kFull || (KIND == kEdge && geo.pow2)) group_minmax_pow2(mn, mx, geo.lpg);
    else group_minmax_any(mn, mx, geo, lane);
    mn = mn + 0.0f;                                  // store -0 as +0
    const float range = mx - mn;
    const float Bf = (float)B;
    float inv = 0.0f, step = 0.0f;
    if (range >= 0x1p-100f) { inv = Bf / range; step = div_levels<BITS>(range); }

    // Minimum and step of every group of the tile.  All lanes of a group hold the
    // same pair.  Stored from the first lane of each group, the values would leave
    // from lanes lpg apart, and a store whose active lanes are scattered over the
    // wavefront goes to memory as one small request per lane (with 4 lanes per
    // group those requests cost 7 % of the compressor's time).  So the pairs are
    // first gathered into the low lanes (two ds_bpermute on the LDS crossbar: lane
    // i takes minimum and step of group i from lane i * lpg) and leave as two
    // contiguous runs.  The gathers are issued here and their results stored
    // after the codes, so that nothing waits for the LDS round trip.
    const int64_t g0 = tile * (int64_t)geo.groups_per_tile;        // first group of the tile
    float group_mn = mn, group_step = step;
    if (geo.lpg > 1) {
        const int src = lane * geo.lpg;                            // lanes past the last group read a wrapped lane, unused
        group_mn = lane_read(mn, src);
        group_step = lane_read(step, src);
    }

    // stochastic rounding + packing: 8 elements per Philox block.
    //
    // The rule "q = floor(t) + [ (r+1/2)/2^16 < t - floor(t) ]" is evaluated in
    // integers.  With T = 2^17 t (an exact rescaling of the binary32 product),
    // C = ceil(T) and c = C mod 2^17:  round up  <=>  2 frac 2^16 > 2r + 1
    // <=>  c >= 2r + 2  <=>  2r + 1 - C < -(floor(t) 2^17), hence
    //     -q = (2r + 1 - C) >> 17   (arithmetic shift).
    // Codes of up to 4 bits: the same with everything scaled by 2^s, s = 0 .. 3:
    //     -q = ((2r + 1) 2^s - C) >> (17 + s),   C = ceil(2^s T).
    // 2^s - C = floor(-2^s T) + 2^s comes out of one addition rounded toward
    // minus infinity: 2^s T < 2^22, so the sum -2^s T + (1.5 * 2^23 + 2^s) lies
    // in [2^23, 2^24), where binary32 has a spacing of 1, and the bit pattern of
    // its round-down value is 0x4B400000 + 2^s + floor(-2^s T).  The 16-bit
    // multiply-add that selects the noise half word adds 2^(s+1) r, and because
    // 0x4B400000 is a multiple of 2^22, bits 17+s .. 17+s+BITS-1 of the result
    // hold -q modulo 2^BITS.  s = position in the nibble: the 1, 2 or 4 elements
    // of a nibble land beside each other in bits 17..20 without a shift and are
    // merged by bit selects; byte permutes put eight nibbles into a word.  (The
    // shift and shift-add per element that this replaced issued at 2.5 and 4.1
    // cycles a wavefront; now 1.4 instructions for a 4-bit element, 1.2 for a
    // 2-bit one, 1 for a 1-bit one, where there were 2.)
    // 8-bit codes (T up to 2^25) convert with floor, s = 0, and accumulate the
    // negated codes last element first, one shift-add each.
    constexpr bool kMagic = BITS <= 4;
    uint32_t out[BITS];
    uint32_t nib[8];                                  // of the word under construction
    constexpr int kPerNib = BITS <= 4 ? 4 / BITS : 1; // elements per nibble
    const float ninv = -(inv * 0x1p17f);
    const float ninv_s[4] = {ninv, ninv * (kPerNib == 2 ? 4.0f : 2.0f), kPerNib == 4 ? ninv * 4.0f : ninv,
                             ninv * (kPerNib == 4 ? 8.0f : 4.0f)};
#pragma unroll
    for (int c = 3; c >= 0; --c) {
        uint32_t r[4];
        if (c < 4 - kEarly) draw(c, r);
        else { r[0] = noise[c][0]; r[1] = noise[c][1]; r[2] = noise[c][2]; r[3] = noise[c][3]; }
        float tn[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)                                        // -2^s T
            tn[j] = (v[c * 8 + j] - mn) * ninv_s[kPerNib == 4 ? j & 3 : kPerNib == 2 ? j & 1 : 0];
        if (kMagic) {
            constexpr float m = 12582912.0f;                               // 1.5 * 2^23
            if (kPerNib == 1) add8_round_down(tn, m + 1.0f, m + 1.0f, m + 1.0f, m + 1.0f);
            if (kPerNib == 2) add8_round_down(tn, m + 1.0f, m + 4.0f, m + 1.0f, m + 4.0f);
            if (kPerNib == 4) add8_round_down(tn, m + 1.0f, m + 2.0f, m + 4.0f, m + 8.0f);
            uint32_t y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t n1 = __builtin_bit_cast(uint32_t, tn[j]), w = r[j >> 1];
                if (kPerNib == 1) y[j] = (j & 1) ? mad_hi16<2>(w, n1) : mad_lo16<2>(w, n1);
                if (kPerNib == 2) y[j] = (j & 1) ? mad_hi16<8>(w, n1) : mad_lo16<2>(w, n1);
                if (kPerNib == 4) y[j] = (j & 1) ? ((j & 2) ? mad_hi16<16>(w, n1) : mad_hi16<4>(w, n1))
                                                 : ((j & 2) ? mad_lo16<8>(w, n1) : mad_lo16<2>(w, n1));
            }
            // nibbles of this chunk: 8 / kPerNib of them, at the chunk's place in the word
            constexpr int kNibs = 8 / kPerNib;
            const int n0 = (c * kNibs) & 7;
#pragma unroll
            for (int i = 0; i < kNibs; ++i) {
                uint32_t a = y[i * kPerNib];
                if (kPerNib == 2) a = select_bits(3u << 19, y[i * 2 + 1], a);
                if (kPerNib == 4) {
                    a = select_bits(1u << 18, y[i * 4 + 1], a);
                    a = select_bits(1u << 20, y[i * 4 + 3], select_bits(1u << 19, y[i * 4 + 2], a));
                }
                nib[n0 + i] = a;
            }
            if (n0 == 0) out[c * kNibs / 8] = negate_fields<BITS>(gather_nibbles(nib));
        } else {
#pragma unroll
            for (int j = 7; j >= 0; --j) {
                const uint32_t n1 = (uint32_t)(cvt_floor_i32(tn[j]) + 1);      // 1 - C
                const uint32_t y = (j & 1) ? mad_hi16<2>(r[j >> 1], n1) : mad_lo16<2>(r[j >> 1], n1);
                int32_t nq = (int32_t)y >> 17;                                 // -q
                // t <= B (1 + 2^-23): an overshoot's fraction is below the smallest noise value
                // 2^-17 unless B = 255, so only 8-bit codes can round past the top level
                nq = nq > -(int32_t)B ? nq : -(int32_t)B;
                const int w = (c * 8 + j) >> 2;
                out[w] = ((j & 3) == 3 ? 0u : out[w] << 8) + (uint32_t)nq;
                if ((j & 3) == 0) out[w] = 0u - out[w];
            }
        }
    }

    if (lane < geo.groups_per_tile && (KIND != kEdge || lane * geo.lpg * kPerLane < ne)) {
        float* gm = t.gmin + g0;                                   // uniform bases, lane offsets
        float* gs = t.gscale + g0;
        gm[lane] = group_mn;
        gs[lane] = group_step;
    }

    // lane i owns dwords [i*BITS, (i+1)*BITS) of the tile's packed words
    const int64_t word0 = (e0 >> 5) * BITS + (int64_t)lane * BITS;
    uint32_t* pk = (uint32_t*)t.packed + word0;
    if (KIND == kFullAny && lane >= geo.lanes_used) return;
    if (KIND != kEdge) {
        if (BITS == 1) {
            __builtin_nontemporal_store(out[0], pk);
        } else if (BITS == 2) {
            u2 o = {out[0], out[1]};
            __builtin_nontemporal_store(o, (u2*)pk);
        } else {
#pragma unroll
            for (int w = 0; w < BITS; w += 4) {
                u4 o = {out[w], out[w + 1], out[w + 2], out[w + 3]};
                __builtin_nontemporal_store(o, (u4*)(pk + w));
            }
        }
    } else {
        // the packed buffer ends at a multiple of 16 bytes; places past the end and pad words are zero
        const int64_t words_total = packed_words(t);
        int bits_left = ne - lane * kPerLane;                      // not carried through the rounding loop
        asm volatile("" : "+v"(bits_left));
        bits_left *= BITS;
#pragma unroll
        for (int w = 0; w < BITS; ++w) {
            const int valid = bits_left - 32 * w;                     // bits of this word that hold codes
            const uint32_t mask = valid >= 32 ? 0xFFFFFFFFu : valid <= 0 ? 0u : (1u << valid) - 1u;
            if (lane < geo.lanes_used && word0 + w < words_total) pk[w] = out[w] & mask;
        }
        // when a tile is narrower than 128*8/BITS elements' worth of padding
        // (group sizes that are not a power of two), up to three pad words lie
        // past the last tile's lanes: the last tile zeroes them
        if ((tile + 1) * (int64_t)tile_elems >= t.n && lane < 4) {          // the last tile
            const int64_t w = (e0 >> 5) * BITS + (int64_t)geo.lanes_used * BITS + lane;
            if (w < words_total) ((uint32_t*)t.packed)[w] = 0u;
        }
    }
}

// --------------------------------------------------------------- decompress
// The decompressor needs no layout switch: a lane handles one 16-byte piece of
// output (4 fp32 or 8 bf16 consecutive elements) per "unit", a unit being the
// 1 KB that one coalesced wavefront store covers.  The piece's codes are
// 4*BITS or 8*BITS consecutive bits of the packed string (a nibble, byte, half
// word, word or two words), fetched with one small load; neighbouring lanes
// fetch neighbouring bits, so those loads coalesce too.  The group's min and
// step are two more loads that all lanes of a group share.  Wavefront w of a
// block takes units w, w+4, w+8, ... so that the four wavefronts write one
// contiguous 4 KB at each step.  Stores are the bottleneck here; the number of
// units per wavefront (dec_unit_table) trades load latency hidden per
// wavefront against the length of its store burst and was chosen by sweep.
template <int DT>
struct DecGeom {
    static constexpr int kPiece = DT == GACT_DT_F32 ? 4 : 8;      // elements per lane and unit
    static constexpr int kUnit = 64 * kPiece;                     // elements per unit
};

// codes of one piece, first element in the low bits
template <int DT, int BITS>
struct PieceBits {
    static constexpr int kBits = DecGeom<DT>::kPiece * BITS;      // 4 .. 64
    uint32_t lo, hi;
};

template <int DT, int BITS, bool EDGE>
__device__ __forceinline__ void load_piece(const TensorArgs& t, int64_t e, PieceBits<DT, BITS>& pb) {
    constexpr int nb = PieceBits<DT, BITS>::kBits;
    const uint8_t* base = (const uint8_t*)t.packed;
    const int64_t bit = e * BITS;
    const int64_t byte = bit >> 3;
    pb.lo = 0u; pb.hi = 0u;
    if (EDGE) {
        // byte by byte, never past the end of the (16-byte rounded) buffer
        const int64_t total = packed_words(t) * 4;
#pragma unroll
        for (int k = 0; k < (nb + 7) / 8; ++k) {
            const uint32_t v = (byte + k < total) ? (uint32_t)base[byte + k] : 0u;
            if (k < 4) pb.lo |= v << (8 * k); else pb.hi |= v << (8 * (k - 4));
        }
        if (nb == 4) pb.lo = (pb.lo >> (int)(bit & 7)) & 0xFu;
        return;
    }
    if (nb == 4) {
        pb.lo = ((uint32_t)__builtin_nontemporal_load(base + byte) >> (int)(bit & 7)) & 0xFu;
    } else if (nb == 8) {
        pb.lo = __builtin_nontemporal_load(base + byte);
    } else if (nb == 16) {
        pb.lo = __builtin_nontemporal_load((const uint16_t*)(base + byte));
    } else if (nb == 32) {
        pb.lo = __builtin_nontemporal_load((const uint32_t*)(base + byte));
    } else {
        const u2 w = __builtin_nontemporal_load((const u2*)(base + byte));
        pb.lo = w.x; pb.hi = w.y;
    }
}

// Keeps the compiler from moving loads across (N != 0), and the wavefront from issuing for about 64 N cycles (N > 0).
template <int N>
__device__ __forceinline__ void pause() {
    if constexpr (N != 0) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (N > 0) __builtin_amdgcn_s_sleep(N);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int DT, int BITS, bool EDGE, int UNITS, Launch LAUNCH>
__device__ __forceinline__ void decompress_units(const TensorArgs& t, const Geometry& geo,
                                                 int64_t block_in_tensor, int64_t first_group, int wave, int lane) {
    constexpr uint32_t B = (1u << BITS) - 1u;
    constexpr int P = DecGeom<DT>::kPiece;
    constexpr int U = DecGeom<DT>::kUnit;
    PieceBits<DT, BITS> pb[UNITS];
    float mn[UNITS], step[UNITS];
    int64_t e[UNITS];
    constexpr LoadOrder kOrder = load_order(DT, BITS, LAUNCH);
    const int64_t first_e = first_group * (geo.lpg * kPerLane);
    const auto begin = [&](int k) {
        const int64_t unit = block_in_tensor * (kWavesPerBlk * UNITS) + k * kWavesPerBlk + wave;
        e[k] = unit * U + lane * P;
        mn[k] = 0.0f; step[k] = 0.0f; pb[k].lo = 0u; pb[k].hi = 0u;
    };
    const auto load_codes = [&](int k) {
        if (!EDGE || e[k] < t.n) load_piece<DT, BITS, EDGE>(t, e[k], pb[k]);
    };
    const auto by_product = [&](int64_t at) {
        return first_group + (int64_t)(__umulhi((uint32_t)((at - first_e) >> 4), geo.group_magic) >> geo.group_shift);
    };
    if constexpr (kOrder.group == kByProduct) {
        const auto load_group = [&](int k) {
            if (EDGE && e[k] >= t.n) return;
            const int64_t g = by_product(e[k]);
            mn[k] = t.gmin[g];
            step[k] = t.gscale[g];
        };
#pragma unroll
        for (int k = 0; k < UNITS; ++k) begin(k);
        if constexpr (kOrder.by_unit) {
#pragma unroll
            for (int k = 0; k < UNITS; ++k) {
                if (k) pause<kOrder.units>();
                if (kOrder.groups_first) load_group(k); else load_codes(k);
                pause<kOrder.kinds>();
                if (kOrder.groups_first) load_codes(k); else load_group(k);
            }
        } else {
#pragma unroll
            for (int k = 0; k < UNITS; ++k) {
                if (k) pause<kOrder.units>();
                if (kOrder.groups_first) load_group(k); else load_codes(k);
            }
            pause<kOrder.kinds>();
#pragma unroll
            for (int k = 0; k < UNITS; ++k) {
                if (k) pause<kOrder.units>();
                if (kOrder.groups_first) load_codes(k); else load_group(k);
            }
        }
    } else {
        // codes first; group_of: the group of an element
        const auto load = [&](auto group_of) {
            const auto load_group = [&](int k) {
                if (EDGE && e[k] >= t.n) return;
                const int64_t g = group_of(e[k]);
                mn[k] = t.gmin[g];
                step[k] = t.gscale[g];
            };
#pragma unroll
            for (int k = 0; k < UNITS; ++k) {
                begin(k);
                load_codes(k);
                if constexpr (kOrder.by_unit) load_group(k);
            }
            if constexpr (!kOrder.by_unit) {
                pause<kOrder.kinds>();
#pragma unroll
                for (int k = 0; k < UNITS; ++k) load_group(k);
            }
        };
        const auto by_shift = [&](int64_t at) { return at >> (geo.group_shift + 5); };
        if constexpr (kOrder.group == kByEither) load([&](int64_t at) { return geo.pow2 ? by_shift(at) : by_product(at); });
        else if (geo.pow2) load(by_shift);
        else load(by_product);
    }
#pragma unroll
    for (int k = 0; k < UNITS; ++k) {
        if (EDGE && e[k] >= t.n) continue;
        float o[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int bit = j * BITS;
            const uint32_t q = ((bit < 32 ? pb[k].lo >> bit : pb[k].hi >> (bit - 32))) & B;
            const float prod = (float)q * step[k];
            o[j] = prod + mn[k];
        }
        if (DT == GACT_DT_F32) {
            float* p = (float*)t.io + e[k];
            if (!EDGE || e[k] + P <= t.n) {
                const f4 v = {o[0], o[1], o[2], o[3]};
                if (!EDGE) __builtin_nontemporal_store(v, (f4*)p); else *(f4*)p = v;
            } else {
#pragma unroll
                for (int j = 0; j < P; ++j) if (e[k] + j < t.n) p[j] = o[j];
            }
        } else {
            uint16_t* p = (uint16_t*)t.io + e[k];
            const u4 v = {bf16_pair_rne(o[0], o[1]), bf16_pair_rne(o[2 % P], o[3 % P]),
                          bf16_pair_rne(o[4 % P], o[5 % P]), bf16_pair_rne(o[6 % P], o[7 % P])};
            if (!EDGE || e[k] + P <= t.n) {
                if (!EDGE) __builtin_nontemporal_store(v, (u4*)p); else *(u4*)p = v;
            } else {
                const uint32_t hh[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int j = 0; j < P; ++j)
                    if (e[k] + j < t.n) p[j] = (uint16_t)(hh[j >> 1] >> (16 * (j & 1)));
            }
        }
    }
}

// ------------------------------------------------------------------ kernels
// uniform dispatch over (dtype, bits)
#define GACT_DISPATCH(t, WITH_F32, CALL)                                             \
    switch ((t).dtype() * 16 + (t).bits()) {                                             \
        case GACT_DT_F32 * 16 + 1:  if constexpr (WITH_F32) { CALL(GACT_DT_F32, 1) } break;  \
        case GACT_DT_F32 * 16 + 2:  if constexpr (WITH_F32) { CALL(GACT_DT_F32, 2) } break;  \
        case GACT_DT_F32 * 16 + 4:  if constexpr (WITH_F32) { CALL(GACT_DT_F32, 4) } break;  \
        case GACT_DT_F32 * 16 + 8:  if constexpr (WITH_F32) { CALL(GACT_DT_F32, 8) } break;  \
        case GACT_DT_BF16 * 16 + 1: { CALL(GACT_DT_BF16, 1) } break;                 \
        case GACT_DT_BF16 * 16 + 2: { CALL(GACT_DT_BF16, 2) } break;                 \
        case GACT_DT_BF16 * 16 + 4: { CALL(GACT_DT_BF16, 4) } break;                 \
        case GACT_DT_BF16 * 16 + 8: { CALL(GACT_DT_BF16, 8) } break;                 \
        default: break;                                                              \
    }

// The block of work this workgroup takes.  Workgroups go to the eight XCDs in
// turn, each XCD with an L2 of its own, so that in plain order neighbouring
// blocks never share one: a line of packed codes, minima or steps that two
// blocks write parts of leaves two caches as two partial writes, and one that two
// blocks read is fetched twice.  (That is every line at a block's edge where the
// caller's buffers are not aligned to 128 bytes, as in one buffer per kind cut at
// multiples of 16, and the lines of minima and steps wherever a block has less than
// a line of them: 64 bytes for 4,096 elements in groups of 256.)  Within a window of 8 * 2^s workgroups, XCD x therefore takes
// the 2^s neighbouring blocks x * 2^s ...; what does not fill a window keeps
// plain order.  s and run_end, the first block past the last whole window (Runs;
// 0: plain order), come from the launcher as the kernel's first two arguments, which
// the build has preloaded into scalar registers, as is the shift of the table lookup:
// from memory they put another scalar load in front of every block's lookup and first
// loads.  A block loads nothing before this chain of scalar instructions is through, so
// a decompressing kernel has s as a constant: with s in a register, the lookup's shift in
// memory and the block length found by branches (dec_unit_table), decompressing 53
// fp32 tensors of 89 M elements took 65.6 us, now 64.9 (65.0 before there was an order).
__device__ __forceinline__ uint32_t work_block(uint32_t run_end, uint32_t s) {
    return ordered_block(blockIdx.x, run_end, s);
}

template <bool WITH_F32, bool SUM, int WAVES>
__device__ __forceinline__ void compress_block(const TensorArgs& t, const Geometry& geo,
                                               int64_t block_in_tensor, TileOut& out_sum) {
    // sized by the launcher: geo.lds_wave_dwords per wavefront
    extern __shared__ __attribute__((aligned(16))) uint32_t lds_all[];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    uint32_t* lds = lds_all + wave * geo.lds_wave_dwords;
    const int64_t tile = block_in_tensor * WAVES + __builtin_amdgcn_readfirstlane(wave);
    if (tile * (int64_t)(geo.lanes_used * kPerLane) >= t.n) return;
    // A tile is "full" when all its elements exist.  With other group sizes the last tile is never
    // treated as one: it also zeroes the pad words that lie past its lanes.
    const int64_t end = (tile + 1) * (int64_t)(geo.lanes_used * kPerLane);
#define GACT_C_FULL(DT, BITS) compress_tile<DT, BITS, kFull, SUM>(t, geo, tile, lds, lane, out_sum);
#define GACT_C_ANY(DT, BITS)  compress_tile<DT, BITS, kFullAny, SUM>(t, geo, tile, lds, lane, out_sum);
#define GACT_C_EDGE(DT, BITS) compress_tile<DT, BITS, kEdge, SUM>(t, geo, tile, lds, lane, out_sum);
    // A tile in which the low word of the Philox block number wraps is not either (PhiloxUniform).
    const uint32_t blk = (uint32_t)(t.blk_base() + ((uint64_t)tile * (uint32_t)(geo.lanes_used * kPerLane) >> 3));
    if ((geo.pow2 ? end <= t.n : end < t.n) && blk <= 0xFFFFFEFFu) {
        if (geo.pow2) { GACT_DISPATCH(t, WITH_F32, GACT_C_FULL) } else { GACT_DISPATCH(t, WITH_F32, GACT_C_ANY) }
    } else {
        GACT_DISPATCH(t, WITH_F32, GACT_C_EDGE)
    }
#undef GACT_C_FULL
#undef GACT_C_ANY
#undef GACT_C_EDGE
}

// full: every element of the block's span exists.
// A wavefront ends where its stores are out and not behind the dispatch: otherwise it takes four more jumps,
// each to a line of instructions of its own, which a launch between a model's kernels fetches anew (bf16,
// 4 bits, between the kernels of a training step: 16.8 M elements 11.7 -> 11.3 us, 50 M 24.7 -> 24.1).
template <uint32_t BF16_UNITS, Launch LAUNCH>
__device__ __forceinline__ void decompress_block(const TensorArgs& t, const Geometry& geo,
                                                 int64_t block_in_tensor, bool full) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    // A piece's group comes out of a product (group_divisor), in a tensor that is too long for it counted from
    // the block's first group.  (A division in 64 bits was 110 instructions a unit, with a branch around them for
    // group sizes that are a power of two; in their place the loads are paced as load_order says.)
    int64_t first_group = 0;
    if (t.n > kMagicElems)
        first_group = (int64_t)((uint64_t)block_in_tensor * (uint32_t)dec_block_elems(t.dtype(), t.bits(), BF16_UNITS) / (uint32_t)(geo.lpg * kPerLane));
#define GACT_D_FULL(DT, BITS) \
    decompress_units<DT, BITS, false, dec_units(DT == GACT_DT_F32 ? kDecUnitsF32 : BF16_UNITS, BITS), LAUNCH>(t, geo, block_in_tensor, first_group, wave, lane); \
    __builtin_amdgcn_endpgm();
#define GACT_D_EDGE(DT, BITS) \
    decompress_units<DT, BITS, true, dec_units(DT == GACT_DT_F32 ? kDecUnitsF32 : BF16_UNITS, BITS), LAUNCH>(t, geo, block_in_tensor, first_group, wave, lane); \
    __builtin_amdgcn_endpgm();
    if (full) { GACT_DISPATCH(t, true, GACT_D_FULL) } else { GACT_DISPATCH(t, true, GACT_D_EDGE) }
#undef GACT_D_FULL
#undef GACT_D_EDGE
}

// The kernel of each kind of launch (Work in gact_device.h).
constexpr int waves_per_simd(Work w) { return w == kCompressAny || w == kCompressLong ? 4 : 8; }
constexpr uint32_t bf16_units(Work w) { return w == kDecompressShort ? kDecUnitsBf16Short : kDecUnitsBf16; }

template <Work W>
__device__ __forceinline__ uint32_t work_block_of(uint32_t run_end, uint32_t run_shift) {
    if constexpr (W == kDecompressShort) return blockIdx.x;
    else return work_block(run_end, W == kDecompress ? kDecompressRunShift : W == kCompressLong ? kCompressLongRunShift : run_shift);
}

template <Work W>
__device__ __forceinline__ void run_block(const TensorArgs& t, const Geometry& geo,
                                          int64_t block_in_tensor) {
    if constexpr (decompresses(W)) {
        const int64_t end = (block_in_tensor + 1) * dec_block_elems(t.dtype(), t.bits(), bf16_units(W));
        decompress_block<bf16_units(W), W == kDecompressShort ? kShortList : kLongList>(t, geo, block_in_tensor, end <= t.n);
    } else {
        TileOut unused;
        compress_block<W != kCompressBf16, false, waves_per_block(W)>(t, geo, block_in_tensor, unused);
    }
}

#define GACT_KERNEL(W) \
    __global__ __launch_bounds__(kLanes * waves_per_block(W)) __attribute__((amdgpu_waves_per_eu(waves_per_simd(W), waves_per_simd(W)))) void

// The second argument is the shift of a run where the tensor is compressed.  Where it is decompressed, it is
// the number of blocks in front of the one that the tensor's end cuts, so that a block of a short launch waits
// for no multiplication by a block length that depends on the tensor's record (one bf16 tensor of 14 M
// elements, 4 bits: 7.7 us without, 7.0 with).  An argument of its own puts the record across a 64-byte line,
// which costs a compressing launch of 7 M elements 0.6 %.
template <Work W>
GACT_KERNEL(W) single_kernel(uint32_t run_end, uint32_t shift_or_full, TensorArgs t, Geometry geo) {
    const uint32_t b = work_block_of<W>(run_end, shift_or_full);
    if constexpr (decompresses(W)) decompress_block<bf16_units(W), W == kDecompressShort ? kShortSingle : kLongSingle>(t, geo, (int64_t)b, b < shift_or_full);
    else run_block<W>(t, geo, (int64_t)b);
}

// One tensor, compressed, with the sum of every block's elements as a by-product.  (One sum per block
// and not per tile: the addition that follows reads a quarter of the terms, and the barrier costs
// nothing, because a block's LDS is not given back before its last wavefront ends.)  Behind fin.blocks
// blocks come, if the sums are tagged, those that take the sample points and those that add the sums.
// The former are blocks of their own because there may be more sample points than the adding blocks, one for 16.8 M
// elements, have threads.  Us a call with 8, 1,024 and 32,768 points, points taken by the adding blocks (with a division
// in 128 bits) and as now: 1 M elements 6.0, 11.7, 340 and 6.0, 6.1, 6.0; 17 M 14.9, 24.7, 425 and 15.0, 15.3, 15.4; 51 M
// 37.8, 38.9, 143 and 37.9, 38.1, 38.1.  (With a launch behind for both: 1 M 9.3, 10.2, 11.3; 51 M 40.8, 44.1, 44.8.)
// The arguments pass the 112 bytes that cost the host 0.6 us (gact_device.h); the launch saved was 3.7 us.
// Blocks of four wavefronts at any length, because a block leaves one sum (537 M fp32 elements: 362 us, the compressor
// alone, in blocks of one, 350).
__global__ __launch_bounds__(kBlockThreads) void compress_sum_kernel(uint32_t run_end, uint32_t run_shift, TensorArgs t,
                                                                     Geometry geo, double* block_sum,
                                                                     Finish fin, int n_samples) {
    __shared__ double part[kWavesPerBlk];
    const uint32_t place = blockIdx.x - fin.ahead;
    if (place >= fin.blocks) {
        const uint32_t past = place - fin.blocks, samplers = samplers_for<kWavesPerBlk>(n_samples);
        if (past < samplers) {
            const int j = (int)(past * kBlockThreads + threadIdx.x);
            if (j < n_samples) sample(t.io, t.dtype(), t.n, j, n_samples, fin.out);
            return;
        }
        finish_block<kWavesPerBlk, true>((uint64_t*)block_sum, fin, fin.ahead ? blockIdx.x : past - samplers);
        return;
    }
    const uint32_t b = ordered_block(place, run_end, run_shift);
    TileOut tile;                                     // its sum stays 0 for a wavefront past the end
    if (threadIdx.x < 64) tile.look = (const uint64_t*)fin.out;
    compress_block<true, true, kWavesPerBlk>(t, geo, (int64_t)b, tile);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = tile.sum;
    __syncthreads();
    if (threadIdx.x < 64) put_result<kWavesPerBlk>(block_sum, b, (part[0] + part[1]) + (part[2] + part[3]), fin, tile.word, (int)threadIdx.x);
}

// Multi-tensor: block b belongs to the tensor l with first_block[l] <= b <
// first_block[l+1]; hint[] narrows the search to the tensors that overlap the
// block's bucket (see gact_device.h), usually one.
template <bool PACKED>
__device__ __forceinline__ int find_tensor(const uint32_t* first_block, const uint32_t* hint, uint32_t shift,
                                           uint32_t b) {
    const uint32_t k = b >> shift;
    int lo = PACKED ? packed_hint(hint, k) : (int)hint[k];
    int hi = (PACKED ? packed_hint(hint, k + 1) : (int)hint[k + 1]) + 1;
    // invariant: first_block[lo] <= b < first_block[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first_block[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// Table in device memory (the caller's workspace): any number of tensors.
template <Work W>
GACT_KERNEL(W) multi_kernel(
    uint32_t run_end, uint32_t run_shift, const TensorArgs* __restrict__ table, const uint32_t* __restrict__ first_block,
    const uint32_t* __restrict__ hint, uint32_t hint_shift, Geometry geo) {
    const uint32_t b = work_block_of<W>(run_end, run_shift);
    const int l = find_tensor<false>(first_block, hint, hint_shift, b);
    const TensorArgs t = table[l];
    run_block<W>(t, geo, (int64_t)(b - first_block[l]));
}

// Table passed by value in the kernel arguments: up to kInlineTensors tensors,
// no upload and no host synchronisation before the launch.
template <Work W>
GACT_KERNEL(W) multi_inline_kernel(
    uint32_t run_end, uint32_t run_shift, uint32_t hint_shift, LineGeometry line, InlineTable tab) {
    const Geometry& geo = line.geo;
    const uint32_t b = work_block_of<W>(run_end, run_shift);
    const int l = find_tensor<true>(tab.first_block, tab.hint, hint_shift, b);
    run_block<W>(tab.t[l], geo, (int64_t)(b - tab.first_block[l]));
}

}  // namespace gact

// ------------------------------------------------------------ host launchers
// KERNEL<work>, launched on `blocks` blocks with the LDS its work needs
#define GACT_LAUNCH(KERNEL, ...)                                                                            \
    do {                                                                                                    \
        const gact::Runs runs = gact::runs_for(work, blocks);                                               \
        const dim3 grid(blocks), block(gact::kLanes * gact::waves_per_block(work));                         \
        const unsigned lds = decompresses(work) ? 0u : 4u * gact::waves_per_block(work) * (unsigned)geo->lds_wave_dwords; \
        hipStream_t s = (hipStream_t)stream;                                                                \
        switch (work) {                                                                                     \
            case gact::kDecompress:   hipLaunchKernelGGL(KERNEL<gact::kDecompress>, grid, block, lds, s, __VA_ARGS__); break;   \
            case gact::kDecompressShort: hipLaunchKernelGGL(KERNEL<gact::kDecompressShort>, grid, block, lds, s, __VA_ARGS__); break; \
            case gact::kCompressBf16: hipLaunchKernelGGL(KERNEL<gact::kCompressBf16>, grid, block, lds, s, __VA_ARGS__); break; \
            case gact::kCompressAny:  hipLaunchKernelGGL(KERNEL<gact::kCompressAny>, grid, block, lds, s, __VA_ARGS__); break;  \
            case gact::kCompressLong: hipLaunchKernelGGL(KERNEL<gact::kCompressLong>, grid, block, lds, s, __VA_ARGS__); break; \
        }                                                                                                   \
        return hipGetLastError() == hipSuccess ? 0 : -1;                                                    \
    } while (0)

extern "C" int gact_launch_single(gact::Work work, const gact::TensorArgs* t, const gact::Geometry* geo,
                                  unsigned blocks, void* stream) {
    const uint32_t full_blocks = decompresses(work) ? (uint32_t)(t->n / gact::dec_block_elems(t->dtype(), t->bits(), gact::bf16_units(work))) : 0u;
    GACT_LAUNCH(gact::single_kernel, runs.end, decompresses(work) ? full_blocks : runs.shift, *t, *geo);
}

extern "C" int gact_launch_compress_sum(const gact::TensorArgs* t, const gact::Geometry* geo, unsigned blocks,
                                        double* d_block_sum, int tagged, uint64_t tag, int n_samples, double* d_out,
                                        void* stream, const gact::Late* late) {
    const unsigned lds = 4u * gact::kWavesPerBlk * (unsigned)geo->lds_wave_dwords;
    const gact::Runs runs = gact::runs_for(gact::kCompressAny, blocks);
    const uint32_t adders = tagged ? gact::adders_for<gact::kWavesPerBlk>(blocks) : 0;
    const gact::Finish fin = gact::finish_of(tagged ? tag : 0, 1.0, d_out, blocks, adders, late);
    const dim3 grid(blocks + adders + (tagged ? gact::samplers_for<gact::kWavesPerBlk>(n_samples) : 0));
    hipLaunchKernelGGL(gact::compress_sum_kernel, grid, dim3(gact::kBlockThreads), lds,
                       (hipStream_t)stream, runs.end, runs.shift, *t, *geo, d_block_sum, fin, n_samples);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

extern "C" int gact_launch_multi_inline(gact::Work work, const gact::InlineTable* tab, unsigned hint_shift,
                                        const gact::Geometry* geo, unsigned blocks, void* stream) {
    const gact::LineGeometry line{*geo, {}};
    GACT_LAUNCH(gact::multi_inline_kernel, runs.end, runs.shift, hint_shift, line, *tab);
}

extern "C" int gact_launch_multi(gact::Work work, const gact::TensorArgs* d_table,
                                 const uint32_t* d_first_block, const uint32_t* d_hint,
                                 unsigned hint_shift, const gact::Geometry* geo, unsigned blocks,
                                 void* stream) {
    GACT_LAUNCH(gact::multi_kernel, runs.end, runs.shift, d_table, d_first_block, d_hint, hint_shift, *geo);
}
