// Device-side helpers shared by the gfx950 kernels of libtorq.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

namespace torq {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(int)))) int i32x8;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// A raw buffer of `bytes` bytes as four words, and a load of 16 bytes per lane from it, at voff + soff, straight into LDS at
// lds_addr + 16 * lane (lds_addr uniform over the wave).  Inline assembly: the compiler neither waits for it nor knows that
// it writes, so a kernel counts these loads in its own waits.  FENCE: the compiler's own memory accesses stay on their
// side of it (a kernel that places its LDS reads itself does without, and its products may move past).
__device__ __forceinline__ i32x4 raw_buffer(const void *p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return i32x4{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xFFFFu), (int)bytes, 0x00020000};
}
// ONCE: the non-temporal hint (see ONE_PASS_INPUT_BYTES).
#define TORQ_LOAD_TO_LDS16 "s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
#define TORQ_LOAD_TO_LDS16_ONCE "s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
template <bool FENCE = true, bool ONCE = false>
__device__ __forceinline__ void load_to_lds16(i32x4 rsrc, uint32_t lds_addr, int voff, int soff) {
  static_assert(FENCE || !ONCE);
  if constexpr (ONCE) asm volatile(TORQ_LOAD_TO_LDS16_ONCE :: "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "m0", "memory");
  else if constexpr (FENCE) asm volatile(TORQ_LOAD_TO_LDS16 :: "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "m0", "memory");
  else asm volatile(TORQ_LOAD_TO_LDS16 :: "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "m0");
}
#undef TORQ_LOAD_TO_LDS16
#undef TORQ_LOAD_TO_LDS16_ONCE
// the same hint as the cache policy of a buffer load builtin
template <bool ONCE>
constexpr int LOAD_POLICY = ONCE ? 2 : 0;

// The output tile of a GEMM workgroup whose wave holds acc[j][i][r] = out[m0 + 32 (wy WM + i) + lane % 32][n0 + 32 (wx WN
// + j) + 8 (r / 4) + 4 (lane / 32) + r % 4] (m0, n0: the tile's corner; wy, wx: the wave's place in it).
// The fp32 sums of a k piece: 16 bytes per lane and register quad, straight from the accumulators (N a multiple of 8).
template <int WM, int WN>
__device__ __forceinline__ void store_sums(const f32x16 (&acc)[WN][WM], float *piece, int64_t m0, int64_t n0, int wy,
                                           int wx, int64_t M, int64_t N, int lrow, int g) {
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int64_t m = m0 + (wy * WM + i) * 32 + lrow;
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int64_t n = n0 + (wx * WN + j) * 32 + 8 * rr + 4 * g;
        if (m < M && n + 4 <= N)
          *reinterpret_cast<f32x4 *>(piece + m * N + n) =
              f32x4{acc[j][i][4 * rr], acc[j][i][4 * rr + 1], acc[j][i][4 * rr + 2], acc[j][i][4 * rr + 3]};
      }
  }
}
// bf16 outputs.  A lane holds 8-byte pieces of one output row; stored directly, every 128-byte line of the output arrives
// in 16 separate partial writes, so the wave first transposes its piece through its own LDS at ep (32 WM rows of 64 WN + 16
// bytes, free by now) and then stores 16 bytes per lane, with 8 adjacent lanes covering one full line.
template <int WM, int WN>
__device__ __forceinline__ void store_bf16(const f32x16 (&acc)[WN][WM], char *ep, uint16_t *out, int64_t m0, int64_t n0,
                                           int wy, int wx, int64_t M, int64_t N, int64_t ldc, int lane, int lrow, int g) {
  constexpr int ROW_E = 64 * WN;               // bytes of one output row of this wave's piece
  constexpr int PITCH_E = ROW_E + 16;
  constexpr int CH_ROW = ROW_E / 16;           // 16-byte chunks per row
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (__bf16)acc[j][i][4 * rr + e];
        *reinterpret_cast<bf16x4 *>(ep + (i * 32 + lrow) * PITCH_E + (32 * j + 8 * rr + 4 * g) * 2) = v;
      }
  const bool vec_ok = (ldc & 7) == 0;           // (out itself is 16-byte aligned: checked by the host)
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int t = 0; t < 32 * CH_ROW / 64; ++t) {
      const int idx = t * 64 + lane, row = idx / CH_ROW, ch = idx % CH_ROW;
      const u32x4 v = *reinterpret_cast<const u32x4 *>(ep + (i * 32 + row) * PITCH_E + ch * 16);
      const int64_t m = m0 + (wy * WM + i) * 32 + row, n = n0 + wx * WN * 32 + ch * 8;
      if (m < M) {
        uint16_t *dst = out + m * ldc + n;
        if (vec_ok && n + 8 <= N) {
          *reinterpret_cast<u32x4 *>(dst) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (n + e < N) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
      }
    }
}

// ---------------------------------------------------------------------------
// MXFP4 quantiser for one microscaling block (Section 4, Eq. 1; Algorithm 3,
// step 4).  The shared scale is the E8M0 byte with 2^(byte-127) =
// 2^(floor(log2 amax) - 2): for a normal fp32 amax that is the exponent field
// minus 2, clamped at 0 (amax is finite, so the field is at most 254).

__device__ __forceinline__ uint32_t e8m0_from_amax(float amax) {
  int field = (int)((__float_as_uint(amax) >> 23) & 0xFFu);
  int b = field - 2;
  return (uint32_t)(b < 0 ? 0 : b);
}

// 2^(byte-127) as an fp32 value; byte 0 is the subnormal 2^-127.
__device__ __forceinline__ float e8m0_to_f32(uint32_t byte) {
  return __uint_as_float(byte ? (byte << 23) : 0x00400000u);
}

// Eight consecutive elements of a block -> eight e2m1 nibbles in one dword,
// element 0 in the lowest nibble.  v_cvt_scalef32_pk_fp4_f32 divides its two
// inputs by `scale`, rounds to the nearest e2m1 value with ties to the even
// code, saturates at 6, keeps the sign bit, and writes one byte of the result.
__device__ __forceinline__ uint32_t pack8_e2m1(const float z[8], float scale) {
  uint32_t r = 0;
  r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, z[0], z[1], scale, 0);
  r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, z[2], z[3], scale, 1);
  r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, z[4], z[5], scale, 2);
  r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, z[6], z[7], scale, 3);
  return r;
}

__device__ __forceinline__ float amax8(const float z[8]) {
  float a = fmaxf(fmaxf(fabsf(z[0]), fabsf(z[1])), fabsf(z[2]));
  a = fmaxf(fmaxf(a, fabsf(z[3])), fabsf(z[4]));
  a = fmaxf(fmaxf(a, fabsf(z[5])), fabsf(z[6]));
  return fmaxf(a, fabsf(z[7]));
}

// ---------------------------------------------------------------------------
// The other 4-bit block formats of Section 6 ("Generalizability to Other Formats").  The paper names
// them without defining them; the readings are those of include/torq.h.

constexpr int FMT_NONE = -1, FMT_MXFP4 = 0, FMT_MXINT4 = 1, FMT_NVFP4 = 2;

// MXINT4: eight values -> eight two's-complement nibbles.  inv_scale = 2^(127 - byte) (the product is
// exact), round to nearest even, clamp to [-7, 7].
__device__ __forceinline__ float e8m0_inverse_f32(uint32_t byte) {   // byte <= 252 for finite input
  return __uint_as_float((254u - byte) << 23);
}
// Adding 1.5 * 2^23 rounds a small value to the nearest integer, ties to even, leaving it in two's
// complement in the low mantissa bits; the product with a power of two is exact, so one fused
// multiply-add rounds exactly what a multiply followed by that add would.  Clamping to [-7, 7] commutes
// with the rounding (the bounds are integers) and is done on the sum.
__device__ __forceinline__ uint32_t pack8_int4(const float z[8], float inv_scale) {
  uint32_t r = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float t = __builtin_amdgcn_fmed3f(__builtin_fmaf(z[i], inv_scale, 12582912.0f), 12582905.0f, 12582919.0f);
    r |= (__float_as_uint(t) & 15u) << (4 * i);
  }
  return r;
}

// OCP FP8 E4M3 (bias 7, largest value 448 = 0x7E, 0x7F is NaN) of t >= 0: round to nearest even
// on three mantissa bits, saturating.  Below 2^-6 the codes are the multiples of 2^-9.
__device__ __forceinline__ uint32_t e4m3_from_f32(float t) {
  if (t < 0.015625f) return (uint32_t)rintf(t * 512.0f);          // 0 .. 8; 8 is the first normal
  uint32_t u = __float_as_uint(t);
  u += 0x7FFFFu + ((u >> 20) & 1u);
  const uint32_t code = (u >> 20) - (120u << 3);
  return code < 0x7Eu ? code : 0x7Eu;
}
__device__ __forceinline__ float e4m3_to_f32(uint32_t code) {     // code <= 0x7E
  return (code >> 3) ? __uint_as_float(((code >> 3) + 120u) << 23 | (code & 7u) << 20)
                     : (float)code * 0.001953125f;
}
// NVFP4's block scale: the E4M3 code of amax / (6 * tensor scale), an IEEE division by definition.  As in
// pack_nvfp4 below the division is carried out only where it can matter: the conversion is monotone, so
// where both ends of a bracket around the quotient convert to the same code the quotient does too.  The hardware converts
// both at once (e4m3_from_f32 up to 448, where that saturates; a NaN amax saturates too).
__device__ __forceinline__ uint32_t nvfp4_scale_code(float amax, float six_gs) {
  if (six_gs >= 0x1p-100f && six_gs <= 0x1p100f) {
    const float t = amax * __builtin_amdgcn_rcpf(six_gs);
    const uint32_t c = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(fminf(t * 0.99999904632568359375f, 448.0f),
                                                                 fminf(t * 1.00000095367431640625f, 448.0f), 0, false);
    const uint32_t lo = c & 255u;
    if (lo == (c >> 8)) return lo;
  }
  return e4m3_from_f32(__fdiv_rn(amax, six_gs));
}

// NVFP4: 8 N values z[i] = v[i] f (rounded to fp32; f in (0, 1]) of a block with effective scale S = e4m3 value * tensor
// scale.  IEEE division, then the e2m1 rounding of pack8_e2m1; a block whose scale rounded to zero keeps signs.
// The division is only carried out where it can matter.  With r = 1 / S to one ulp, v (r (1 - 2^-20) f) and
// v (r (1 + 2^-20) f), rounded wherever they are (z, r, three products and the quotient: 7 * 2^-24 in all, relative), enclose
// the IEEE quotient q = z / S in magnitude; the e2m1 rounding is monotone, so where both ends round to the same code it is
// q's.  Otherwise (a quotient within 2^-20 of a rounding boundary, ties among them: a few values in a million) the lane
// divides.  S outside [2^-100, 2^100] or f below 2^-20: always divides.
// Two products and two halves of a conversion per value and none for z itself, which only a division needs: the butterfly
// rotation to NVFP4 (bound by its vector instructions), X [4096, 8192],
// 24.4 -> 23.4 us at G = 128, 25.8 -> 22.1 at G = 32, 11.6 -> 10.9 for X [512, 8192] at G = 256.
template <int N>
__device__ __forceinline__ void pack_nvfp4(const float *v, float f, float S, uint32_t (&c)[N]) {
  if (S >= 0x1p-100f && S <= 0x1p100f && f >= 0x1p-20f) {
    const float r = __builtin_amdgcn_rcpf(S);
    const float r_lo = r * 0.99999904632568359375f * f, r_hi = r * 1.00000095367431640625f * f;      // 1 -+ 2^-20
    uint32_t differ = 0;
    float a[8];
#pragma unroll
    for (int n = 0; n < N; ++n) {
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = v[8 * n + i] * r_lo;
      c[n] = pack8_e2m1(a, 1.0f);
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = v[8 * n + i] * r_hi;
      differ |= c[n] ^ pack8_e2m1(a, 1.0f);
    }
    if (differ == 0) return;
  }
  if (!(S > 0.0f)) {                       // (also where a tile has no block row: not the way of the divisions)
    float a[8 * N];
#pragma unroll
    for (int i = 0; i < 8 * N; ++i) a[i] = copysignf(0.0f, v[i]);
#pragma unroll
    for (int n = 0; n < N; ++n) c[n] = pack8_e2m1(a + 8 * n, 1.0f);
    return;
  }
  // (rarely reached: a value at a time, so that it does not ask for registers the way above has no use for)
  auto divide = [&](float value) {
    const float q = __fdiv_rn(__fmul_rn(value, f), S);
    __builtin_amdgcn_sched_barrier(0);
    return q;
  };
#pragma unroll
  for (int n = 0; n < N; ++n) {
    uint32_t r = 0;
#define TORQ_DIVIDE_PAIR(I_)                                                                                         \
  {                                                                                                                  \
    const float q0 = divide(v[8 * n + 2 * I_]), q1 = divide(v[8 * n + 2 * I_ + 1]);                                   \
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, q0, q1, 1.0f, I_);                                                \
  }
    TORQ_DIVIDE_PAIR(0) TORQ_DIVIDE_PAIR(1) TORQ_DIVIDE_PAIR(2) TORQ_DIVIDE_PAIR(3)
#undef TORQ_DIVIDE_PAIR
    c[n] = r;
  }
}

// bf16 <-> fp32 bit moves
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

}  // namespace torq
