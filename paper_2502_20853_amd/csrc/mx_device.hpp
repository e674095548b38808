// Device-side building blocks of the MXFP4 quantizers (gfx950).
//
// Everything here works on FP32 bit patterns so that each decision (shared
// exponent, bracket, rounding direction) is an exact integer operation on a value
// that is a power-of-two multiple of the input.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mx_launch.hpp"

namespace mxd {

// ---- shared exponent (Sec. 3.2) -------------------------------------------
// amax_bits: FP32 bits of M = max |x| over the group (sign cleared).
// Returns the scale byte s + 127.
//   truncation-free: s = ceil(log2(M/6)).  With M = m * 2^e, 1 <= m < 2 and
//     6 = 1.5 * 2^2 this is e - 2 when m <= 1.5 and e - 1 otherwise.
//   Eq. 2:           s = floor(log2 M) - 2 = e - 2.
// The biased exponent field is e + 127, so byte = field - 2 (+1).  Clamping s
// to >= -127 is byte >= 0; subnormal M has field 0 and lands on that clamp.
// M = 0 uses epsilon = 1e-8, for which both rules give s = -29.
__device__ __forceinline__ uint32_t scale_byte(uint32_t amax_bits, bool floor_mode)
{
    // adding 0x3FFFFF carries into the exponent field exactly when the mantissa exceeds 0x400000
    uint32_t field = (amax_bits + (floor_mode ? 0u : 0x3FFFFFu)) >> 23;
    uint32_t b;
    asm("v_sub_u32_e64 %0, %1, 2 clamp" : "=v"(b) : "v"(field));     // max(field - 2, 0) in one instruction
    return amax_bits == 0u ? 98u : b;
}

// 2^-s as FP32 for scale byte b = s + 127 (s in [-127, 126]: always normal).
__device__ __forceinline__ float inv_scale(uint32_t byte)
{
    return __uint_as_float((254u - byte) << 23);
}

// ---- E2M1 rounding (Sec. 3.2) ----------------------------------------------
// The integer form, which round_S uses (round_D of E2M1 goes through conversion instructions further down, E3M0 uses the
// integer form for both).  It never forms y = x / S itself but v = x * 2^(-s-126) (one ldexp), which
// puts |y| in [0, 6] onto FP32 bit patterns whose layout IS the E2M1 grid: |y| < 1 lands
// in FP32's subnormal range (uniform spacing, like E2M1's subnormals 0 and 0.5), [1,2)
// in the first normal binade, and so on, so that
//     bits(v) >> 22           = code of the largest E2M1 magnitude m1 <= |y|,
//     bits(v) & 0x3FFFFF      = p * 2^22,   p = (|y| - m1) / (m2 - m1).
// Rounding is then one integer add that carries into bit 22.  The scaling is exact except
// when the result is subnormal and x has bits below 2^-149; the FP32 rounding mode is set
// so that the inexact case still decides correctly (v_ldexp_f32 rounds a subnormal result
// by the mode, like a multiplication does):
//   round_D, ties to the larger value: y > 0 goes up iff p >= 1/2, which floor(p * 2^22)
//     decides; y < 0 goes up in magnitude iff p > 1/2, which ceil(p * 2^22) decides.  Both
//     are what round-toward-minus-infinity does to the signed value.
//   round_S: up iff r16 < 65536 * p  <=>  p * 2^22 > 64 * r16, which ceil decides:
//     round-toward-plus-infinity on |x|.
__device__ __forceinline__ void f32_round_toward_plus_inf()  { __builtin_amdgcn_s_setreg(0x801, 1); }   // MODE[1:0]
__device__ __forceinline__ void f32_round_toward_minus_inf() { __builtin_amdgcn_s_setreg(0x801, 2); }
__device__ __forceinline__ void f32_round_to_nearest_even()  { __builtin_amdgcn_s_setreg(0x801, 0); }

constexpr uint32_t GRID_MAX_BITS = 0x01C00000u;      // 6 * 2^-126

// Exponent to hand to ldexp for scale byte b = s + 127:  -s - 126 = 1 - b.
__device__ __forceinline__ int grid_exponent(uint32_t byte) { return 1 - (int)byte; }

// |value| of an E2M1 code times 2^s, from the same bit layout: (code & 7) << 22 is
// m * 2^-126 as an FP32 pattern.  Exact in any rounding mode.
__device__ __forceinline__ float dequant_mag(uint32_t code, uint32_t byte)
{
    return __builtin_ldexpf(__uint_as_float((code & 7u) << 22), (int)byte - 1);
}

// Q-EMA (Algorithm 1): bracket from y = w/S, choice by z = w_ema/S.
// y_is_exact_zero: w itself is +-0 (then y = 0 is an E2M1 value and is kept); a nonzero w whose
// y underflowed to 0 in FP32 still has the bracket [0, 0.5].
__device__ __forceinline__ uint32_t round_ema(float y, float z, bool floor_mode, bool w_is_zero)
{
    uint32_t yb = __float_as_uint(y);
    uint32_t ab = yb & 0x7FFFFFFFu;
    if (floor_mode) ab = ab > 0x40C00000u ? 0x40C00000u : ab;
    uint32_t E = ab >> 23;
    E = E < 127u ? 127u : E;
    float f = __uint_as_float((255u - E) << 23);
    float k = __uint_as_float(ab) * f;
    float fl = floorf(k);
    float fr = k - fl;
    uint32_t neg = yb >> 31;
    // z mirrored so that the bracket is [fl, fl+1] on a positive axis
    float zk = __uint_as_float(__float_as_uint(z) ^ (neg << 31)) * f;
    float mid = fl + 0.5f;
    bool up = neg ? (zk > mid) : (zk >= mid);   // |z-q1| < |z-q2| picks q1, else q2
    up = up && (fr != 0.0f || (ab == 0u && !w_is_zero));   // w/S already an E2M1 value: keep it
    return (2u * (E - 127u) + (uint32_t)fl + (up ? 1u : 0u)) | ((yb >> 28) & 8u);
}

// signed value of an E2M1 code times 2^s (byte = s + 127), exact in FP32 (may be subnormal)
__device__ __forceinline__ float dequant(uint32_t code, uint32_t byte)
{
    return __uint_as_float(__float_as_uint(dequant_mag(code, byte)) | ((code & 8u) << 28));
}

// ---- Philox4x32-10 (Salmon et al., SC'11) ----------------------------------
struct U4 { uint32_t w[4]; };

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                            uint32_t k0, uint32_t k1)
{
    const uint32_t MUL_A = 0xD2511F53u, MUL_B = 0xCD9E8D57u;
    const uint32_t WEYL_A = 0x9E3779B9u, WEYL_B = 0xBB67AE85u;
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        uint64_t pa = (uint64_t)MUL_A * c0;
        uint64_t pb = (uint64_t)MUL_B * c2;
        uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c1, k0, 0x96);   // three-way xor
        uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), c3, k1, 0x96);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += WEYL_A;
        k1 += WEYL_B;
    }
    U4 r;
    r.w[0] = c0; r.w[1] = c1; r.w[2] = c2; r.w[3] = c3;
    return r;
}

// The eight 16-bit fields for the 8-element block `blk` (= element index >> 3).
__device__ __forceinline__ U4 sr_block(uint64_t blk, uint32_t tensor_id, uint32_t k0, uint32_t k1)
{
    return philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), tensor_id, 0u, k0, k1);
}

// The same where every lane of the launch has the block number's upper word in common (`hi`, uniform like the tensor id
// and the key): of the first two rounds' four products one is then the same for all lanes in each round, and of their
// values only three depend on the lane and none of these on the tensor id, so the scalar unit does the rest and two
// streams over the same elements share them.  38 vector instructions with the addition that makes `lo`, 34 for a second
// stream, against 43 each.
struct SrCounter32 { uint32_t w3, lo, hi; };

__device__ __forceinline__ SrCounter32 sr_counter(uint32_t lo, uint32_t k1)
{
    const uint32_t MUL_A = 0xD2511F53u, MUL_B = 0xCD9E8D57u;
    const uint64_t pa = (uint64_t)MUL_A * lo;                               // round 1 from (lo, hi, tensor_id, 0)
    const uint64_t pb = (uint64_t)MUL_B * ((uint32_t)(pa >> 32) ^ k1);      // round 2
    return {(uint32_t)pa, (uint32_t)pb, (uint32_t)(pb >> 32)};
}

__device__ __forceinline__ U4 sr_block_uniform_hi(const SrCounter32& c, uint32_t hi, uint32_t tensor_id, uint32_t k0, uint32_t k1)
{
    const uint32_t MUL_A = 0xD2511F53u, MUL_B = 0xCD9E8D57u;
    const uint32_t WEYL_A = 0x9E3779B9u, WEYL_B = 0xBB67AE85u;
    // round 1: words 0 and 1 are uniform after it
    const uint32_t u0 = __umulhi(MUL_B, tensor_id) ^ hi ^ k0, u1 = MUL_B * tensor_id;
    // round 2: word 3 is uniform after it
    const uint32_t s0 = u1 ^ (k0 + WEYL_A), s2 = __umulhi(MUL_A, u0) ^ (k1 + WEYL_B), u3 = MUL_A * u0;
    uint32_t c0 = c.hi ^ s0, c1 = c.lo, c2 = c.w3 ^ s2, c3;
    k0 += 2u * WEYL_A; k1 += 2u * WEYL_B;
    // round 3
    {
        const uint64_t pa = (uint64_t)MUL_A * c0, pb = (uint64_t)MUL_B * c2;
        const uint32_t s3 = u3 ^ k1;
        c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c1, k0, 0x96);
        c2 = (uint32_t)(pa >> 32) ^ s3;
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        k0 += WEYL_A; k1 += WEYL_B;
    }
#pragma unroll
    for (int i = 3; i < 10; ++i) {
        const uint64_t pa = (uint64_t)MUL_A * c0, pb = (uint64_t)MUL_B * c2;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), c3, k1, 0x96);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += WEYL_A; k1 += WEYL_B;
    }
    U4 r;
    r.w[0] = c0; r.w[1] = c1; r.w[2] = c2; r.w[3] = c3;
    return r;
}

// The eight terms 64 * r16 - (2^22 - 1) of an 8-element block, which sr_grid() subtracts: mag - term carries into bit 22
// iff p * 2^22 > 64 * r16.  (Subtracting takes r16 as it stands; adding ((65535 - r16) << 6) | 63 instead costs an
// inversion of each random word, 4 of the 105 instructions a block takes.)
struct U8 { uint32_t w[8]; };

// (16-bit field of w) * 64 - (2^22 - 1) in one instruction; HIGH selects the upper field.
template <bool HIGH>
__device__ __forceinline__ uint32_t sr_term(uint32_t w)
{
    uint32_t r;
    if (HIGH) asm("v_mad_u32_u16 %0, %1, 64, %2 op_sel:[1,0,0,0]" : "=v"(r) : "v"(w), "s"(0xFFC00001u));
    else      asm("v_mad_u32_u16 %0, %1, 64, %2" : "=v"(r) : "v"(w), "s"(0xFFC00001u));
    return r;
}

__device__ __forceinline__ U8 sr_terms_of(const U4& r)
{
    U8 a;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a.w[2 * i] = sr_term<false>(r.w[i]);
        a.w[2 * i + 1] = sr_term<true>(r.w[i]);
    }
    return a;
}

// Where block numbers of the launch differ in their upper word (the WIDE kernels): the block number itself.
struct SrCounter64 { uint64_t blk; };
__device__ __forceinline__ SrCounter64 sr_counter(uint64_t blk, uint32_t) { return {blk}; }

__device__ __forceinline__ U8 sr_terms(const SrCounter32& c, uint32_t hi, uint32_t tensor_id, uint32_t k0, uint32_t k1)
{
    return sr_terms_of(sr_block_uniform_hi(c, hi, tensor_id, k0, k1));
}
__device__ __forceinline__ U8 sr_terms(const SrCounter64& c, uint32_t, uint32_t tensor_id, uint32_t k0, uint32_t k1)
{
    return sr_terms_of(sr_block(c.blk, tensor_id, k0, k1));
}

// ---- E3M0 elements (the other 4-bit format of the paper's format ablation, Table 7) -------------
// Code = sign << 3 | exponent field E (3 bits, no mantissa bit); magnitude 0 for E = 0 and 2^(E-3)
// otherwise: 0, 0.25, 0.5, 1, 2, 4, 8, 16 (bias 3, no Inf/NaN codes), Q_p = 16, E_max = 4.
// The same construction as for E2M1 works one bit higher: v = x * 2^(-s-124) puts |y| in [0, 16] onto
// FP32 patterns whose exponent field IS the code of the lower neighbour (|y| < 0.25 lands in the
// subnormals, the bracket [0, 0.25]) and whose 23 mantissa bits are p * 2^23.
//   truncation-free scale: s = ceil(log2(M / 16)) = e - 4 for M = 2^e exactly, e - 3 otherwise;
//   Eq. 2's scale:         s = floor(log2 M) - 4.
// epsilon = 1e-8 = 1.34 * 2^-27 for an all-zero group gives s = -30 resp. -31.
__device__ __forceinline__ uint32_t scale_byte_e3m0(uint32_t amax_bits, bool floor_mode)
{
    uint32_t field = (amax_bits + (floor_mode ? 0u : 0x7FFFFFu)) >> 23;   // carries iff the mantissa is not zero
    uint32_t b;
    asm("v_sub_u32_e64 %0, %1, 4 clamp" : "=v"(b) : "v"(field));
    return amax_bits == 0u ? (floor_mode ? 96u : 97u) : b;
}

constexpr uint32_t GRID_MAX_BITS_E3M0 = 7u << 23;     // 16 * 2^-124

__device__ __forceinline__ int grid_exponent_e3m0(uint32_t byte) { return 3 - (int)byte; }

// round_D; rounding mode toward minus infinity: on the signed value it floors the magnitude of y > 0 and ceils that of y < 0.
template <bool FLOOR>
__device__ __forceinline__ uint32_t rtn_code_e3m0(float x, int e)
{
    uint32_t vb = __float_as_uint(__builtin_ldexpf(x, e));
    uint32_t mag = vb & 0x7FFFFFFFu;
    if (FLOOR) mag = mag > GRID_MAX_BITS_E3M0 ? GRID_MAX_BITS_E3M0 : mag;
    uint32_t t = mag + 0x400000u + (uint32_t)((int32_t)vb >> 31);
    return (t >> 23) | ((vb >> 28) & 8u);
}

// round_S; rounding mode toward plus infinity; rinv = ((65535 - r16) << 7) | 127.
template <bool FLOOR>
__device__ __forceinline__ uint32_t sr_code_e3m0(float x, int e, uint32_t rinv)
{
    uint32_t mag = __float_as_uint(__builtin_ldexpf(__builtin_fabsf(x), e));
    if (FLOOR) mag = mag > GRID_MAX_BITS_E3M0 ? GRID_MAX_BITS_E3M0 : mag;
    return ((mag + rinv) >> 23) | ((__float_as_uint(x) >> 28) & 8u);
}

__device__ __forceinline__ U8 sr_addends_e3m0(uint64_t blk, uint32_t tensor_id, uint32_t k0, uint32_t k1)
{
    U4 r = sr_block(blk, tensor_id, k0, k1);
    U8 a;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a.w[2 * i] = ((65535u - (r.w[i] & 0xFFFFu)) << 7) | 127u;
        a.w[2 * i + 1] = ((65535u - (r.w[i] >> 16)) << 7) | 127u;
    }
    return a;
}

// signed value of an E3M0 code times 2^s: (E << 23) is 2^(E-127) as an FP32 pattern (0 for E = 0)
__device__ __forceinline__ float dequant_e3m0(uint32_t code, uint32_t byte)
{
    float mag = __builtin_ldexpf(__uint_as_float((code & 7u) << 23), (int)byte - 3);
    return __uint_as_float(__float_as_uint(mag) | ((code & 8u) << 28));
}

// ---- FP4 conversion instructions of gfx950 -----------------------------------
// What the quantizers use of them.  tests/test_gpu_codec.py holds the quantizers that stand on them against a plain C form:
// every bf16 value under every scale that a group with it can have, FP32 thresholds with three neighbours on either side at
// every scale, and all 16 codes at every pair of row and column scales.  The FP32 rounding mode does not enter (round_S
// kernels convert with the mode toward plus infinity).
//   v_cvt_scalef32_pk_fp4_bf16   two bf16 values / 2^s, round to nearest even, saturated at 6  -> one byte
//   v_cvt_scalef32_pk_fp4_f32    the same from FP32; also a packer of values that are already on the grid
//   v_cvt_scalef32_pk_{f32,bf16}_fp4   two codes x 2^s -> two values, exact
// 2^s is given as the FP32 pattern byte << 23 (byte 0 means 2^-127).  Cost, in cycles of a SIMD per wave instruction
// with four waves on it: 9, 9 and 4.5 for two elements; a three-operand integer instruction takes 5, a two-operand
// one 3.  Taking a code apart from the grid sum and packing it took about 15 per element, so both the deterministic
// rounding of bf16 sources (12.5 against 33 with double quantization) and the packing go through them.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_hw __attribute__((ext_vector_type(2)));
typedef float f32x2_hw __attribute__((ext_vector_type(2)));

template <typename D, typename S>
__device__ __forceinline__ D bits_as(S s)
{
    static_assert(sizeof(D) == sizeof(S), "same size");
    return __builtin_bit_cast(D, s);
}

__device__ __forceinline__ float scale_operand(uint32_t byte) { return __uint_as_float(byte << 23); }

__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b)
{
    return bits_as<uint32_t>(__builtin_elementwise_max(bits_as<u16x2>(a), bits_as<u16x2>(b)));
}

// round_D sends a tie to the larger value, the conversion to the even code.  A threshold of E2M1 has at most 3
// significant bits, so of two neighbouring bf16 values at most the one with an even last bit is a threshold: moving
// every even pattern one unit toward +infinity (positive: last bit set; negative: magnitude less one) takes ties to
// the right side and moves nothing across a threshold.  +0 becomes the smallest positive value (code 0); -0 stays
// at the saturation bound of the signed addition and becomes the smallest negative value (code 8).
__device__ __forceinline__ uint32_t ties_to_larger(uint32_t w)
{
    const s16x2 v = bits_as<s16x2>(w);
    return bits_as<uint32_t>(__builtin_elementwise_add_sat(v, v >> (short)15)) | 0x00010001u;
}

// byte SEL of `old` <- codes of the two bf16 values in w (low half first), scale as scale_operand().  A conversion keeps
// the other bytes of its destination.  Where they are all written later, or not used, `old` is the source itself, whose
// register then serves as the destination: a cleared one costs a move.
template <int SEL>
__device__ __forceinline__ uint32_t cvt_fp4_bf16(uint32_t old, uint32_t w, float scale)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(old, bits_as<bf16x2_hw>(w), scale, SEL);
}

// byte SEL of `old` <- codes of two values on the grid layout, sign << 31 | code << 22
template <int SEL>
__device__ __forceinline__ uint32_t pack_grid(uint32_t old, uint32_t g0, uint32_t g1)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(old, __uint_as_float(g0), __uint_as_float(g1), __uint_as_float(1u << 23), SEL);
}

template <int SEL>
__device__ __forceinline__ f32x2_hw cvt_f32_fp4(uint32_t codes, float scale)
{
    return __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, scale, SEL);
}

template <int SEL>
__device__ __forceinline__ uint32_t cvt_bf16_fp4(uint32_t codes, float scale)
{
    return bits_as<uint32_t>(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, SEL));
}

// round_S onto the grid layout, sign << 31 | code << 22.  Rounding mode toward plus infinity.
template <bool FLOOR>
__device__ __forceinline__ uint32_t sr_grid_sum(float x, int e, uint32_t term)
{
    uint32_t mag = __float_as_uint(__builtin_ldexpf(__builtin_fabsf(x), e));
    if (FLOOR) mag = mag > GRID_MAX_BITS ? GRID_MAX_BITS : mag;
    return mag - term;
}

template <bool FLOOR>
__device__ __forceinline__ uint32_t sr_grid(float x, int e, uint32_t term)
{
    return __builtin_amdgcn_bitop3_b32(0x80000000u, sr_grid_sum<FLOOR>(x, e, term) & 0x7FC00000u, __float_as_uint(x), 0xEC);   // b | (a & c)
}

// The same in one instruction less, except that the 22 low bits are those of x.  A dequantized x has none but with scale
// byte 0, whose 0.5 and 1.5 times 2^-127 are FP32 subnormals with bit 21 set: there the caller clears them (& ON_GRID).
template <bool FLOOR>
__device__ __forceinline__ uint32_t sr_grid_dequantized(float x, int e, uint32_t term)
{
    return __builtin_amdgcn_bitop3_b32(0x7FC00000u, sr_grid_sum<FLOOR>(x, e, term), __float_as_uint(x), 0xCA);               // a ? b : c
}

constexpr uint32_t ON_GRID = 0xFFC00000u;

// round_D of FP32 values.  The conversion sends ties to the even code; as for bf16 (ties_to_larger), a threshold's FP32
// pattern is even, so moving even patterns one unit toward +infinity decides ties and moves nothing else across a
// threshold.  -0 stays a negative zero through the saturating addition.  3.5 instructions per element instead of the 5
// of the integer form (scale to the grid, add half a unit, cut).
__device__ __forceinline__ float ties_to_larger_f32(float x)
{
    const int32_t v = (int32_t)__float_as_uint(x);
    return __uint_as_float((uint32_t)__builtin_elementwise_add_sat(v, v >> 31) | 1u);
}

// byte SEL of `old` <- codes of round_D(x0 / 2^s), round_D(x1 / 2^s), scale as scale_operand()
template <int SEL>
__device__ __forceinline__ uint32_t cvt_rtn_f32(uint32_t old, float x0, float x1, float scale)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(old, ties_to_larger_f32(x0), ties_to_larger_f32(x1), scale, SEL);
}

// The same into a fresh register; the other bytes are anything.
template <int SEL>
__device__ __forceinline__ uint32_t cvt_rtn_f32(float x0, float x1, float scale)
{
    const float t = ties_to_larger_f32(x0);
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(__float_as_uint(t), t, ties_to_larger_f32(x1), scale, SEL);
}

__device__ __forceinline__ uint32_t rtn_codes8_f32(const float (&x)[8], uint32_t byte)
{
    const float s = scale_operand(byte);
    uint32_t p = cvt_rtn_f32<0>(x[0], x[1], s);
    p = cvt_rtn_f32<1>(p, x[2], x[3], s);
    p = cvt_rtn_f32<2>(p, x[4], x[5], s);
    return cvt_rtn_f32<3>(p, x[6], x[7], s);
}

// Scale bytes of two group maxima at once, given as bf16 patterns of |x| in the halves of m (see scale_byte: a bf16
// mantissa exceeds 1.5 iff adding 0x3F carries).
template <bool FLOOR>
__device__ __forceinline__ uint32_t scale_bytes_bf16(uint32_t m)
{
    const u16x2 v = bits_as<u16x2>(m);
    const u16x2 field = (FLOOR ? v : (u16x2)(v + (unsigned short)0x3F)) >> (unsigned short)7;
    const u16x2 nonzero = __builtin_elementwise_min(v, (u16x2)(unsigned short)1);
    const u16x2 b = __builtin_elementwise_sub_sat(field, (u16x2)(unsigned short)2);
    return bits_as<uint32_t>((u16x2)(b + (u16x2)(nonzero * (unsigned short)(0u - 98u) + (unsigned short)98)));
}

// |x| maxima of two rows over the 4 lanes of a row group, row 0 in the low half and row 1 in the high half.  m0, m1: a
// lane's maxima of each row as bf16 patterns, two partial ones per register.
__device__ __forceinline__ uint32_t quad_amax_bf16_rows(uint32_t m0, uint32_t m1)
{
    uint32_t m = pk_max(__builtin_amdgcn_perm(m1, m0, 0x05040100u), __builtin_amdgcn_perm(m1, m0, 0x07060302u));
    m = pk_max(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xB1, 0xF, 0xF, true));      // lane ^ 1
    return pk_max(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4E, 0xF, 0xF, true));   // lane ^ 2
}

// Maxima over the 8 lanes that share lane % 8 (the row groups of a wave tile), of four values at once.  A lane-swap
// instruction of two different values leaves half of each beside its partner, so each step halves the number of
// registers instead of repeating the reduction per value (8 instructions for four values; one by one it is 32).
// Returned: rows of 16 lanes 0..3 hold the maxima of m[0], m[2], m[1], m[3].
template <typename MAX>
__device__ __forceinline__ uint32_t reduce_row_groups4(const uint32_t (&m)[4], MAX&& mx)
{
    const auto a = __builtin_amdgcn_permlane32_swap(m[0], m[1], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(m[2], m[3], false, false);
    const uint32_t u0 = mx(a[0], a[1]), u1 = mx(b[0], b[1]);
    const auto c = __builtin_amdgcn_permlane16_swap(u0, u1, false, false);
    const uint32_t v = mx(c[0], c[1]);
    return mx(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true));      // row_ror:8 = lane ^ 8
}

// The way back: every lane gets the four values that reduce_row_groups4 left in the four rows of 16 lanes.
__device__ __forceinline__ void spread_row_groups4(uint32_t v, uint32_t (&q)[4])
{
    const auto w = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const auto a = __builtin_amdgcn_permlane32_swap(w[0], w[0], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(w[1], w[1], false, false);
    q[0] = a[0]; q[1] = a[1]; q[2] = b[0]; q[3] = b[1];
}

// ---- cross-lane max over aligned groups of 4 lanes (one 32-element group) ---
__device__ __forceinline__ uint32_t quad_max(uint32_t v)
{
    uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);  // lane ^ 1
    v = v > o ? v : o;
    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);           // lane ^ 2
    return v > o ? v : o;
}

// ---- source loads: 8 consecutive elements as FP32; a source is read once, so the loads
//      carry the nontemporal hint --------------------------
struct F8 { float v[8]; };

__device__ __forceinline__ F8 load8(const float* p)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4* q = reinterpret_cast<const f4*>(p);
    const f4 a = __builtin_nontemporal_load(q), b = __builtin_nontemporal_load(q + 1);
    F8 r;
    r.v[0] = a.x; r.v[1] = a.y; r.v[2] = a.z; r.v[3] = a.w;
    r.v[4] = b.x; r.v[5] = b.y; r.v[6] = b.z; r.v[7] = b.w;
    return r;
}

__device__ __forceinline__ F8 load8(const uint16_t* p)   // bf16 bit patterns
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const u4 a = __builtin_nontemporal_load(reinterpret_cast<const u4*>(p));
    F8 r;
    r.v[0] = __uint_as_float(a.x << 16); r.v[1] = __uint_as_float(a.x & 0xFFFF0000u);
    r.v[2] = __uint_as_float(a.y << 16); r.v[3] = __uint_as_float(a.y & 0xFFFF0000u);
    r.v[4] = __uint_as_float(a.z << 16); r.v[5] = __uint_as_float(a.z & 0xFFFF0000u);
    r.v[6] = __uint_as_float(a.w << 16); r.v[7] = __uint_as_float(a.w & 0xFFFF0000u);
    return r;
}

// The same in two steps, for loads issued ahead of their use: 4 registers hold 8 bf16 values.
typedef uint32_t bf16x8_raw __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8_raw load8_raw(const uint16_t* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const bf16x8_raw*>(p));
}
__device__ __forceinline__ F8 zero8()
{
    F8 r;
#pragma unroll
    for (int t = 0; t < 8; ++t) r.v[t] = 0.0f;
    return r;
}

// max(|a|, |b|, m) on FP32 bit patterns in one instruction: for finite values the order of the
// magnitudes is the order of their bit patterns, and the source modifiers take the absolute values
// (the separate AND and the two-operand maximum cost more issue cycles than this one instruction).
__device__ __forceinline__ uint32_t absmax3_bits(float a, float b, uint32_t m)
{
    float r;
    asm("v_max3_f32 %0, |%1|, |%2|, %3" : "=v"(r) : "v"(a), "v"(b), "v"(__uint_as_float(m)));
    return __float_as_uint(r);
}

__device__ __forceinline__ uint32_t amax_bits8(const F8& x)
{
    uint32_t m = 0;
#pragma unroll
    for (int t = 0; t < 8; t += 2) m = absmax3_bits(x.v[t], x.v[t + 1], m);
    return m;
}

// Eight source elements of one row, as loaded: bf16 values stay packed in pairs.
template <typename SrcT> using Raw8 = std::conditional_t<std::is_same_v<SrcT, float>, F8, bf16x8_raw>;

__device__ __forceinline__ F8 load_raw8(const float* p) { return load8(p); }
__device__ __forceinline__ bf16x8_raw load_raw8(const uint16_t* p) { return load8_raw(p); }

// The same for a source that other workgroups read too.
__device__ __forceinline__ F8 load_raw8_shared(const float* p)
{
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    return F8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ __forceinline__ bf16x8_raw load_raw8_shared(const uint16_t* p) { return *reinterpret_cast<const bf16x8_raw*>(p); }

__device__ __forceinline__ float element_of(const F8& r, int t) { return r.v[t]; }
__device__ __forceinline__ float element_of(const bf16x8_raw& r, int t)
{
    return __uint_as_float((t & 1) ? r[t >> 1] & 0xFFFF0000u : r[t >> 1] << 16);
}

__device__ __forceinline__ uint32_t abs_max_bf16(const bf16x8_raw& x)                 // two partial maxima
{
    const uint32_t k = 0x7FFF7FFFu;
    return pk_max(pk_max(x[0] & k, x[1] & k), pk_max(x[2] & k, x[3] & k));
}

// Scale byte of a row group from the lane's own eight elements.
template <bool FLOOR>
__device__ __forceinline__ uint32_t row_scale_byte(const F8& x) { return scale_byte(quad_max(amax_bits8(x)), FLOOR); }
template <bool FLOOR>
__device__ __forceinline__ uint32_t row_scale_byte(const bf16x8_raw& x)
{
    const uint32_t m = abs_max_bf16(x);
    return scale_bytes_bf16<FLOOR>(quad_amax_bf16_rows(m, m)) & 0xFFFFu;
}

// round_D codes of eight elements of a row, low nibble first.
__device__ __forceinline__ uint32_t rtn_codes8(const bf16x8_raw& x, uint32_t byte)
{
    const float s = scale_operand(byte);
    const uint32_t first = ties_to_larger(x[0]);
    uint32_t p = cvt_fp4_bf16<0>(first, first, s);
    p = cvt_fp4_bf16<1>(p, ties_to_larger(x[1]), s);
    p = cvt_fp4_bf16<2>(p, ties_to_larger(x[2]), s);
    return cvt_fp4_bf16<3>(p, ties_to_larger(x[3]), s);
}

__device__ __forceinline__ uint32_t rtn_codes8(const F8& x, uint32_t byte) { return rtn_codes8_f32(x.v, byte); }

}  // namespace mxd

namespace mxl {

// Sums the per-block column sums in a fixed order: a workgroup of 256 owns 32 columns; each of its 8 parts
// (32 lanes) adds up a contiguous eighth of the blocks in index order (independent loads, 128 bytes
// per row of 32 lanes), then the eight parts are added in order.
__device__ __forceinline__ void column_sum_finish(const ColumnSumTail& a, uint32_t block)
{
    __shared__ float part[8][32];
    const uint32_t lc = threadIdx.x & 31u, p = threadIdx.x >> 5;
    const uint32_t c = block * 32u + lc;
    const uint32_t per = (a.blocks + 7u) / 8u;
    float s = 0.f;
    if (c < a.cols) {
        const uint32_t b0 = min(a.blocks, p * per), b1 = min(a.blocks, b0 + per);
        const float* p0 = a.partials + (size_t)b0 * a.cols + c;
        uint32_t b = b0;
        for (; b + 8u <= b1; b += 8u, p0 += (size_t)8 * a.cols) {           // eight loads in flight, added in order
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p0[(size_t)i * a.cols];
#pragma unroll
            for (int i = 0; i < 8; ++i) s += v[i];
        }
        for (; b < b1; ++b, p0 += a.cols) s += *p0;
    }
    part[p][lc] = s;
    __syncthreads();
    if (p == 0 && c < a.cols) {
        float t = part[0][lc];
#pragma unroll
        for (int q = 1; q < 8; ++q) t += part[q][lc];
        if (a.out_bf16) static_cast<__bf16*>(a.out)[c] = (__bf16)t;
        else            static_cast<float*>(a.out)[c] = t;
    }
}

}  // namespace mxl
