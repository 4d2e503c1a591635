// cpes_device.hpp -- device functions of the CoPES hot path for gfx950:
// the Philox4x32-10 counter-based generator, the Box-Muller transform that
// turns its words into the Gaussian noise of Eq. (8), and bf16 storage.
//
// Seed replay (Sec. 3.3, Supp. A.8): the noise of every member is a pure
// function of (seed, position), so perturb, restore and update regenerate it in
// registers and nothing of size d is ever stored.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cpes_bm_tables.hpp"

namespace cpes {

// ----------------------------------------------------------------- Philox --
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
// 32x32->64 multiplies and xors, the key advancing by Weyl constants between
// rounds.  The key words come from kernel arguments, so the key schedule runs
// on the scalar unit; each three-way xor is one v_bitop3_b32 (truth table
// 0x96) on gfx950.

constexpr uint32_t kPhiloxMulA = 0xD2511F53u;
constexpr uint32_t kPhiloxMulB = 0xCD9E8D57u;
constexpr uint32_t kWeylA = 0x9E3779B9u;
constexpr uint32_t kWeylB = 0xBB67AE85u;

struct Words4 {
    uint32_t x, y, z, w;
};

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The rounds from `first` on, keys as at round 0.
template <int FIRST>
__device__ __forceinline__ Words4 philox_rounds(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                                uint32_t k1)
{
    k0 += FIRST * kWeylA;
    k1 += FIRST * kWeylB;
#pragma unroll
    for (int r = FIRST; r < 10; ++r) {
        const uint64_t pa = (uint64_t)kPhiloxMulA * c0;
        const uint64_t pb = (uint64_t)kPhiloxMulB * c2;
        const uint32_t n0 = xor3((uint32_t)(pb >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(pa >> 32), c3, k1);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += kWeylA;
        k1 += kWeylB;
    }
    return Words4{c0, c1, c2, c3};
}

__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1)
{
    return philox_rounds<0>(c0, c1, c2, c3, k0, k1);
}

// Block q of stream (key, domain): counter (lo32 q, hi32 q, domain, 0).  Q is
// uint32_t where every block of a launch is known to be below 2^32 (noise
// indices below 2^34).  With three counter words the same in all lanes, half
// of the first two rounds then belongs to the scalar unit: they are written
// out with plain xors, which the compiler can take there (xor3 is opaque).
// That and the constants held in Bm save 7 and 10 VALU instructions per 8
// normals in the loops of the update and of the in-place perturbation, which
// have 226 and 256 with them.
template <typename Q>
__device__ __forceinline__ Words4 stream_block(uint32_t k0, uint32_t k1, uint32_t domain, Q q)
{
    if constexpr (sizeof(Q) == 8) {
        return philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), domain, 0u, k0, k1);
    } else {
        const uint64_t pa = (uint64_t)kPhiloxMulA * q, pb = (uint64_t)kPhiloxMulB * domain;
        const uint32_t c0 = (uint32_t)(pb >> 32) ^ k0, c2 = (uint32_t)(pa >> 32) ^ k1;
        const uint64_t qa = (uint64_t)kPhiloxMulA * c0, qb = (uint64_t)kPhiloxMulB * c2;
        return philox_rounds<2>((uint32_t)(qb >> 32) ^ ((uint32_t)pb ^ (k0 + kWeylA)), (uint32_t)qb,
                                (uint32_t)pa ^ ((uint32_t)(qa >> 32) ^ (k1 + kWeylB)), (uint32_t)qa, k0, k1);
    }
}

// ------------------------------------------------------------ Box-Muller --
// A pair of words (a, b) gives two normals rho cos(theta), rho sin(theta) with
// rho = sqrt(-2 ln U(a)), theta = 2 pi U(b), U(x) = ((x >> 8) + 1) 2^-24.
// Both factors are evaluated in fp64 (full rate on CDNA4) to ~2^-46 relative
// error and their product is rounded once to fp32, so the result is the
// correctly rounded normal unless the exact value lies within ~2^-46
// relative of a midpoint between two fp32 numbers (and it is always within
// one fp32 ulp of it).  The update, which only needs weighted sums of normals,
// adds the fp64 products themselves.
//
// Two small tables do most of the work (cpes_bm_tables.hpp, generated by
// gen_bm_tables.py): 256 log entries and 512 points of the unit circle,
// 12 KiB staged into LDS once per workgroup by stage_bm_tables<BLOCK>().

static_assert(sizeof(LogEntry) == 16 && sizeof(AngleEntry) == 16, "16-byte table entries");
static_assert(sizeof(BmTables) == 16 * (kLogTableSize + kAngleTableSize), "tables are packed 16-byte entries");

// The tables in LDS, the circle's points at half their size (bm_radius2 gives
// twice the radius), and two polynomial constants in vector registers: an
// instruction reads one constant from the scalar registers, so an fma of two
// constants needs the other one in a vector register, where the compiler would
// move it again in every round of a loop.
struct Bm {
    const BmTables* t;
    double ang_a3, ang_b2;
};

// Entry i of the tables as it is kept in LDS (halving is exact).
__device__ __forceinline__ uint4 staged_entry(int i, uint4 v)
{
    if (i < kLogTableSize) return v;
    AngleEntry t = __builtin_bit_cast(AngleEntry, v);
    t.c *= 0.5;
    t.s *= 0.5;
    return __builtin_bit_cast(uint4, t);
}

// Copy both tables into LDS; every thread of the workgroup must call it (it
// ends with a barrier).  With a BLOCK-thread workgroup each thread issues all
// of its 16-byte loads before the first LDS store, so the workgroup waits for
// one memory round trip instead of one per entry it copies.
template <int BLOCK>
__device__ __forceinline__ Bm stage_bm_tables()
{
    constexpr int kWords = (int)(sizeof(BmTables) / sizeof(uint4));
    constexpr int kPer = (kWords + BLOCK - 1) / BLOCK;
    __shared__ BmTables tb;
    const uint4* src = reinterpret_cast<const uint4*>(&kBmTables);
    uint4* dst = reinterpret_cast<uint4*>(&tb);
    if (blockDim.x == BLOCK) {
        uint4 v[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r)
            if ((r + 1) * BLOCK <= kWords || threadIdx.x + r * BLOCK < kWords) v[r] = src[threadIdx.x + r * BLOCK];
#pragma unroll
        for (int r = 0; r < kPer; ++r)
            if ((r + 1) * BLOCK <= kWords || threadIdx.x + r * BLOCK < kWords)
                dst[threadIdx.x + r * BLOCK] = staged_entry(threadIdx.x + r * BLOCK, v[r]);
    } else {
        for (int i = threadIdx.x; i < kWords; i += blockDim.x) dst[i] = staged_entry(i, src[i]);
    }
    __syncthreads();
    Bm bm = {&tb, kAngA3, kAngB2};
    asm volatile("" : "+v"(bm.ang_a3), "+v"(bm.ang_b2));
    return bm;
}

template <typename E>
__device__ __forceinline__ E lds_entry(const E* table, uint32_t byte_off)
{
    return *reinterpret_cast<const E*>(reinterpret_cast<const char*>(table) + byte_off);
}

// L = -2 ln U for U = m 2^-24, m in [1, 2^24], table-driven (Tang's method):
// mn = m << lz is m normalised to [2^31, 2^32); entry i = bits 30..23 of mn
// holds inv_i ~ 2^-31 / c_i and B_i = -2 ln c_i for a point c_i of that
// 1/256-wide mantissa interval.  Then
//   r = mn inv_i - 1  (one fma, |r| <= 2^-8),
//   L = (lz - 7) 2 ln 2 + B_i - 2 ln(1 + r),
// with -2 ln(1 + r) = r q(r), q of degree 4 (Taylor).  Relative error at
// most 2^-46.5 over all 2^24 inputs.  B_0 carries 2^-400 in place of 0, so
// U = 1 gives L = 2^-400 (a zero normal after rounding) and L is never 0.
__device__ __forceinline__ double bm_log_term(uint32_t a, const Bm& tb)
{
    uint32_t m7;                                           // m 2^7 = (a >> 8) 2^7 + 2^7 <= 2^31
    asm("v_lshl_add_u32 %0, %1, 7, %2" : "=v"(m7) : "v"(a >> 8), "s"(128u));
    const uint32_t e = (uint32_t)__builtin_clz(m7);        // lz - 7, in [0, 24]
    const uint32_t mn = m7 << e;
    const uint32_t byte_off = (mn >> (27 - kLogTableBits)) & ((kLogTableSize - 1) << 4);   // entry * 16
    const LogEntry t = lds_entry(tb.t->log, byte_off);
    const double r = __builtin_fma((double)mn, t.inv, -1.0);
    const double base = __builtin_fma((double)e, kTwoLn2, t.b);
    double q = -0x1.999999999999ap-2;                      // -2/5
    q = __builtin_fma(q, r, 0.5);
    q = __builtin_fma(q, r, -0x1.5555555555555p-1);        // -2/3
    q = __builtin_fma(q, r, 1.0);
    q = __builtin_fma(q, r, -2.0);
    return __builtin_fma(r, q, base);
}

// 2 rho = 2 sqrt(L) for L > 0: hardware reciprocal square root y (2^-24) and
// one Newton step, (L y) (3 - L y^2), to 2^-47; `scale` multiplies it on the
// way.  Leaving the factor two to the circle's table saves an instruction a
// pair against sqrt(L) itself.
__device__ __forceinline__ double bm_radius2(uint32_t a, const Bm& tb)
{
    const double L = bm_log_term(a, tb);
    const double y = __builtin_amdgcn_rsq(L);
    const double g = L * y;
    return g * __builtin_fma(-g, y, 3.0);
}
__device__ __forceinline__ double bm_radius2(uint32_t a, const Bm& tb, double scale)
{
    const double L = bm_log_term(a, tb);
    const double y = __builtin_amdgcn_rsq(L);
    const double g = L * y;
    return (g * scale) * __builtin_fma(-g, y, 3.0);
}

// (cos, sin)(theta) / 2 for theta = 2 pi m 2^-24, m = (b >> 8) + 1 in [1, 2^24],
// as a rotation from the nearest of 512 table angles: i = round(m / 2^15)
// mod 512, offset x = m - 2^15 round(m / 2^15) in [-2^14, 2^14), delta =
// x 2 pi 2^-24.  sin delta (degree 5) and cos delta (degree 4) are Taylor
// polynomials in x, below 2^-53 from the functions for |delta| <= 2^-7.35.
// Every zero of cos or sin lies on a table angle, so near one the rotation
// reduces to +-sin delta and keeps its relative accuracy; the table's signed
// zeros make the quarter-turn angles come out as in an exact quadrant
// reduction.  Relative error below 2^-50 over all 2^24 inputs.
__device__ __forceinline__ void bm_half_angle(uint32_t b, const Bm& tb, double& cos_t, double& sin_t)
{
    // Adding 0x100 to b cannot carry out of its low byte, so bits 8..31 of
    // b + 0x100 are m mod 2^24 (m = 2^24 wraps to 0, the same angle); x is
    // their low 15 bits read as a signed field.  Adding 2^22 more rounds m to
    // the nearest multiple of 2^15, whose top 9 bits index the table.
    const uint32_t s8 = b + 0x100u;
    const double x = (double)((int32_t)(s8 << 9) >> 17);
    const uint32_t byte_off = ((b + 0x400100u) >> (31 - kAngleTableBits - 3)) & ((kAngleTableSize - 1) << 4);
    const AngleEntry t = lds_entry(tb.t->angle, byte_off);
    const double x2 = x * x;                               // exact
    const double sd = x * __builtin_fma(x2, __builtin_fma(x2, kAngA5, tb.ang_a3), kAngA1);
    const double cd = __builtin_fma(x2, __builtin_fma(x2, kAngB4, tb.ang_b2), 1.0);
    cos_t = __builtin_fma(t.c, cd, -(t.s * sd));
    sin_t = __builtin_fma(t.s, cd, t.c * sd);
}

// Two normals of the pair (a, b): z_even = fp32(rho cos theta), z_odd =
// fp32(rho sin theta).
__device__ __forceinline__ void bm_pair(uint32_t a, uint32_t b, const Bm& tb, float& z_even, float& z_odd)
{
    const double rho = bm_radius2(a, tb);
    double c, s;
    bm_half_angle(b, tb, c, s);
    z_even = (float)(rho * c);
    z_odd = (float)(rho * s);
}

// The pair scaled and added to fp64 sums, without the rounding to fp32 between.
__device__ __forceinline__ void bm_pair_add(uint32_t a, uint32_t b, const Bm& tb, double scale, double& even,
                                            double& odd)
{
    const double rho = bm_radius2(a, tb, scale);
    double c, s;
    bm_half_angle(b, tb, c, s);
    even = __builtin_fma(rho, c, even);
    odd = __builtin_fma(rho, s, odd);
}

// Four normals of block q: positions 4q .. 4q+3 (domain 0 is the noise).
template <typename Q>
__device__ __forceinline__ void normals4(uint32_t k0, uint32_t k1, Q q, const Bm& tb, float z[4],
                                         uint32_t domain = 0u)
{
    const Words4 x = stream_block(k0, k1, domain, q);
    bm_pair(x.x, x.y, tb, z[0], z[1]);
    bm_pair(x.z, x.w, tb, z[2], z[3]);
}

// Eight normals of blocks q and q+1: positions 4q .. 4q+7.
template <typename Q>
__device__ __forceinline__ void normals8(uint32_t k0, uint32_t k1, Q q, const Bm& tb, float z[8],
                                         uint32_t domain = 0u)
{
    const Words4 x = stream_block(k0, k1, domain, q);
    const Words4 y = stream_block(k0, k1, domain, (Q)(q + 1u));
    bm_pair(x.x, x.y, tb, z[0], z[1]);
    bm_pair(x.z, x.w, tb, z[2], z[3]);
    bm_pair(y.x, y.y, tb, z[4], z[5]);
    bm_pair(y.z, y.w, tb, z[6], z[7]);
}

// acc[e] += scale times the normal of position 4q + e, N = 4 or 8 of them.
template <int N, typename Q>
__device__ __forceinline__ void add_normals(uint32_t k0, uint32_t k1, Q q, const Bm& tb, double scale, double acc[N])
{
#pragma unroll
    for (int h = 0; h < N / 4; ++h) {
        const Words4 x = stream_block(k0, k1, 0u, (Q)(q + h));
        bm_pair_add(x.x, x.y, tb, scale, acc[4 * h + 0], acc[4 * h + 1]);
        bm_pair_add(x.z, x.w, tb, scale, acc[4 * h + 2], acc[4 * h + 3]);
    }
}

// ------------------------------------------------------------------ bf16 --

__device__ __forceinline__ float bf16_to_f32(uint16_t h)
{
    return __uint_as_float((uint32_t)h << 16);
}

// Round to nearest even; NaN stays a quiet NaN (gfx950 converts in hardware).
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    const __bf16 h = (__bf16)f;
    return __builtin_bit_cast(uint16_t, h);
}

}  // namespace cpes
