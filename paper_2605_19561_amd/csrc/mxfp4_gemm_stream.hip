// mxfp4_gemm for few activation rows and wide layers (decode, M <= 64): the W4A4 linear layer of Section 5 / Algorithm 3
// ("Return"), same arithmetic as mxfp4_gemm_skinny.hip and the same bits.
//
// Bound: HBM, the weights read once.  The other two forms of few rows end a workgroup, or a turn of it, with a drain: its
// requests are answered, multiplied and added up before the next ones go out.  Here a workgroup takes one strip of 16 weight
// rows after the other and its requests run through the strips' ends:
//   * the activations' codes and scale bytes are read once and stay in registers (2 PT MT operands; d <= 2048 PT);
//   * a wave reads its line pairs w, w + 8, ... of every strip in whole lines straight into its own ring of R items in LDS
//     (a CU's requests in flight are counted in lines, so half lines in the operand's layout bring half as much), refilled as
//     soon as an item is in registers: R x 16 KB of a CU are always on their way;
//   * one barrier a strip: it says that the strip's scale bytes are in LDS and that the partial tiles of the strip before are,
//     which one wave per activation tile, the waves in turn, adds in the order 0 + 1 + ... + 7 and stores.
#include "torq_device.h"
#include "torq_internal.h"

namespace torq {

namespace {

typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2;
constexpr int WAVES = 8;
constexpr int STREAM_RING = 4;                    // items of a wave's ring: 3 and 5 measured 1 - 4 % slower, 2, 6 and 8 more
constexpr size_t STREAM_MAX_LDS = 160 * 1024;
constexpr int OOB_VOFF = 0x7FFFFFF0;              // rejected by the range check of any buffer here: zeros

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// 16-byte units of a scale row in LDS: an odd number, so that the lanes of a k-step, which read one byte of 16 rows each,
// find them in different banks
__host__ __device__ constexpr int stream_scale_units(int d) { return (d / 512) | 1; }
// buffers of scale rows: the one in use and those of the strips that the ring reaches ahead into
__host__ __device__ constexpr int stream_scale_buffers(int PT, int R) { return (R + PT - 1) / PT + 1; }

size_t stream_lds_bytes(int MT, int PT, int R, int d) {
  const size_t per = (16 * (size_t)stream_scale_units(d) + WAVES - 1) / WAVES * WAVES * 16;
  return (size_t)WAVES * R * 2048 + stream_scale_buffers(PT, R) * per + (size_t)2 * WAVES * MT * 1024;
}

}  // namespace

template <int MT, int PT, int R>
__global__ void __launch_bounds__(64 * WAVES)
mxfp4_gemm_stream_kernel(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                         const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int N, int d, int strips_each, int strips_over) {
  constexpr int BUFS = stream_scale_buffers(PT, R);
  static_assert(2 * R + BUFS <= 63, "the counter of loads in flight has six bits");
  // LDS: [rings | BUFS buffers of scale rows | two buffers of partial tiles]
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int row_bytes = d / 2, srow_bytes = d / 32, KP = d / 256;
  const int pu = stream_scale_units(d), s_pitch = pu * 16, per_wave = (16 * pu + WAVES - 1) / WAVES;
  const int sc_bytes = per_wave * WAVES * 16;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t ring0 = lds0 + wave * R * 2048, sc0 = lds0 + WAVES * R * 2048;
  const unsigned char *const ring = smem + wave * R * 2048;
  const unsigned char *const sc = smem + WAVES * R * 2048;
  f32x4 *const red = reinterpret_cast<f32x4 *>(smem + WAVES * R * 2048 + BUFS * sc_bytes);   // [2][WAVES][MT][64]

  const int first = blockIdx.x, step = gridDim.x;
  const int count = strips_each + (first < strips_over ? 1 : 0);    // strips of this workgroup, at least one

  // ---- requests.  Exactly two loads an item and one a strip's scale rows, whatever they bring: past the end of the k range
  // or of the strips they come from empty buffers
  const int l_row = lane >> 3;
  const int v0 = l_row * row_bytes + ((lane & 7) ^ (l_row >> 1)) * 16;
  const int v1 = (l_row + 8) * row_bytes + ((lane & 7) ^ (l_row >> 1) ^ 4) * 16;
  const int s_unit = wave * per_wave + lane;
  const int s_row = (int)(((float)s_unit + 0.5f) * __builtin_amdgcn_rcpf((float)pu)), s_col = s_unit - s_row * pu;   // (unit / pu)
  const int vs = s_row < 16 && s_col < srow_bytes / 16 ? s_row * srow_bytes + s_col * 16 : OOB_VOFF;
  // strip number s of the workgroup: tile s of the activations, then the weight strips
  auto row_of = [&](int s) { return s < MT ? 16 * s : s < MT + count ? (first + (s - MT) * step) * 16 : 0; };
  auto rows_of = [&](int s) {
    const int left = (s < MT ? M : s < MT + count ? N : 0) - row_of(s);
    return left < 16 ? left : 16;
  };
  // (the four words are the same in all lanes; the compiler takes some of them through vector registers)
  auto uniform = [](i32x4 v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = __builtin_amdgcn_readfirstlane(v[j]);
    return v;
  };
  auto request = [&](int s, int i, int slot) {
    const int kp = wave + 8 * i;
    const i32x4 rs = uniform(raw_buffer((s < MT ? A_q : W_q) + (int64_t)row_of(s) * row_bytes, kp < KP ? (uint32_t)rows_of(s) * row_bytes : 0u));
    load_to_lds16(rs, ring0 + slot * 2048, v0, kp * 128);
    load_to_lds16(rs, ring0 + slot * 2048 + 1024, v1, kp * 128);
  };
  auto request_scales = [&](int s) {
    const i32x4 rs = uniform(raw_buffer((s < MT ? A_s : W_s) + (int64_t)row_of(s) * srow_bytes, (uint32_t)rows_of(s) * srow_bytes));
    if (lane < per_wave) load_to_lds16(rs, sc0 + (s % BUFS) * sc_bytes + wave * per_wave * 16, vs, 0);
  };
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (j % PT == 0) request_scales(j / PT);
    request(j / PT, j % PT, j);
  }

  const int f_off[2] = {r16 * 128 + ((q ^ ((r16 >> 1) & 7)) * 16), r16 * 128 + (((4 + q) ^ ((r16 >> 1) & 7)) * 16)};
  // the partial tiles of strip s: added and stored by the waves whose turn it is
  auto reduce = [&](int s) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (((s * MT + t) & (WAVES - 1)) != wave) continue;           // uniform over the wave
      const f32x4 *p = red + ((s & 1) * WAVES * MT + t) * 64 + lane;
      f32x4 sum = p[0];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) {
        const f32x4 v = p[w * MT * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] += v[r];
      }
      bf16x4 o;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = (__bf16)sum[r];
      const int m = t * 16 + r16;
      const int nn = row_of(MT + s) + 4 * q;
      if (m < M) {
        uint16_t *dst = out + (int64_t)m * N + nn;
        if ((N & 3) == 0 && nn + 4 <= N) {
          *reinterpret_cast<bf16x4 *>(dst) = o;
        } else {
          const uint64_t bits = __builtin_bit_cast(uint64_t, o);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (nn + r < N) dst[r] = (uint16_t)(bits >> (16 * r));
        }
      }
    }
  };

  int slot = 0;
  const unsigned char *srow = sc;
  u32x4 f0, f1;                                    // item i of strip s: its two operands and their scales
  int w0, w1;
  // the items younger than number i of a strip: R - 1, and the scale rows of the strips that begin among them
  auto take = [&](auto i_c, int s, auto at_start) {
    constexpr int i = decltype(i_c)::value;
    wait_vm<2 * (R - 1) + (i + R - 1) / PT>();
    if constexpr (i == 0) {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      srow = sc + (s % BUFS) * sc_bytes + r16 * s_pitch + q;
      at_start();
    }
    const int kp = wave + 8 * i, so = kp < KP ? kp * 8 : 0;
    f0 = *reinterpret_cast<const u32x4 *>(ring + slot * 2048 + f_off[0]);
    f1 = *reinterpret_cast<const u32x4 *>(ring + slot * 2048 + f_off[1]);
    w0 = srow[so];
    w1 = srow[so + 4];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // read: the slot can be filled again
    if constexpr ((i + R) % PT == 0) request_scales(s + (i + R) / PT);
    request(s + (i + R) / PT, (i + R) % PT, slot);
    slot = slot + 1 == R ? 0 : slot + 1;
  };

  // ---- the activations: operand (i, e, t) = line pair wave + 8 i, k-step e of it, tile t; zeros past M and d
  u32x4 aq[PT][2][MT];
  int as[PT][MT];                                  // bytes 0 and 1: the lane's scales of the two k-steps
  static_for<MT>([&](auto t_c) {
    constexpr int t = decltype(t_c)::value;
    static_for<PT>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      take(i_c, t, []() {});
      aq[i][0][t] = f0;
      aq[i][1][t] = f1;
      as[i][t] = w0 | w1 << 8;
    });
  });

  // ---- the strips
  for (int s = 0; s < count; ++s) {
    f32x4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    static_for<PT>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      take(i_c, MT + s, [&]() { if (s > 0) reduce(s - 1); });
#pragma unroll
      for (int t = 0; t < MT; ++t)
        acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
            i32x8{(int)f0[0], (int)f0[1], (int)f0[2], (int)f0[3], 0, 0, 0, 0},
            i32x8{(int)aq[i][0][t][0], (int)aq[i][0][t][1], (int)aq[i][0][t][2], (int)aq[i][0][t][3], 0, 0, 0, 0},
            acc[t], 4, 4, 0, w0, 0, as[i][t]);
#pragma unroll
      for (int t = 0; t < MT; ++t)
        acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
            i32x8{(int)f1[0], (int)f1[1], (int)f1[2], (int)f1[3], 0, 0, 0, 0},
            i32x8{(int)aq[i][1][t][0], (int)aq[i][1][t][1], (int)aq[i][1][t][2], (int)aq[i][1][t][3], 0, 0, 0, 0},
            acc[t], 4, 4, 0, w1, 1, as[i][t]);
    });
#pragma unroll
    for (int t = 0; t < MT; ++t) red[(((s & 1) * WAVES + wave) * MT + t) * 64 + lane] = acc[t];
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");       // nothing is on its way into the LDS any more
  reduce(count - 1);
}

template <int MT, int PT, int R>
static hipError_t launch_cfg(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M,
                             int64_t N, int d, hipStream_t stream) {
  const size_t lds = stream_lds_bytes(MT, PT, R, d);
  if (lds > STREAM_MAX_LDS) return hipErrorInvalidValue;
  if (lds > 64 * 1024) {
    static std::atomic<uint64_t> raised{0};
    const hipError_t e =
        raise_lds_limit(reinterpret_cast<const void *>(mxfp4_gemm_stream_kernel<MT, PT, R>), STREAM_MAX_LDS, raised);
    if (e != hipSuccess) return e;
  }
  const int64_t strips = (N + 15) / 16;
  const int64_t grid = strips < 256 ? strips : 256;
  hipLaunchKernelGGL((mxfp4_gemm_stream_kernel<MT, PT, R>), dim3((unsigned)grid), dim3(64 * WAVES), lds, stream, A_q, A_s, W_q, W_s,
                     reinterpret_cast<uint16_t *>(out), (int)M, (int)N, d, (int)(strips / grid), (int)(strips % grid));
  return hipGetLastError();
}

// Whether the product (d a multiple of 512, 16-byte aligned scale rows) is one for strips through a ring where the whole-line
// form does not take it: line pairs of two to four per wave and strip (d = 2560 ... 8192; the activations' operands would not
// fit the registers beyond), and strips enough for a workgroup's start, the activations through its ring, to be paid off.
// Weights from HBM, us, what the planner took before against this form:
//   8 - 16 rows past 1600 strips (two strips a workgroup, persistent): [8, 8192] x 28672 27.8 / 25.8, [16, 8192] x 28672 28.7 /
//     26.4; below that the whole-line form stays, and below 8 rows the strips straight to registers ([1, 8192] x 28672 24.4 /
//     25.1)
//   17 - 32 rows past 1536 strips (tiles): [17, 5120] x 28672 18.8 / 17.0, [32, 8192] x 25600 29.8 / 25.0, [32, 2560] x 28672
//     11.0 / 10.6; d = 2048 9.1 / 9.3, left to the tiles
//   33 - 64 rows (tiles, cut or not), where it is ahead by more than the two were apart in other runs:
//     640 to 768 and 1024 to 1536 strips, which 64 x 64 and 64 x 128 tiles fill badly: [48, 5120] x 12288 12.0 / 10.3, [64,
//       7168] x 12288 18.3 / 14.1, [48, 4096] x 12288 9.5 / 8.7, [33, 8192] x 20480 26.2 / 21.2, [64, 2560] x 20480 10.8 / 10.5;
//       d = 3072 x 12288 7.7 / 7.8
//     elsewhere past 640 strips where every wave has its full share of line pairs, d a multiple of 2048: [48, 6144] x 14336 14.4
//       / 12.8, [48, 8192] x 25600 30.6 / 26.1, [64, 4096] x 28672 16.4 / 16.3, but [33, 4096] x 16384 9.5 / 10.3; between them,
//       [64, 5120] x 16384 13.8 / 13.0, [64, 7168] x 28672 26.0 / 26.2, [64, 2560] x 28672 11.8 / 12.8, the tiles keep theirs
bool mxfp4_gemm_stream_takes(int64_t M, int64_t N, int d) {
  if (M < 8 || M > 64 || d % 512 != 0 || d < 2560 || d > 8192 || N > (1 << 30)) return false;
  const int64_t strips = (N + 15) / 16;
  if (M <= 16) return strips > 1600;
  if (M <= 32) return strips > 1536;
  if (strips > 640 && strips <= 768) return d >= 3584;
  if (strips > 1024 && strips <= 1536) return true;
  return strips > 640 && d % 2048 == 0 && (d > 4096 || strips > 1024);
}

int mxfp4_gemm_stream_strips(int d) { return stream_scale_buffers((d / 256 + WAVES - 1) / WAVES, STREAM_RING); }

// mxfp4_gemm_stream_takes(M, N, d), 16-byte aligned scale rows
hipError_t launch_mxfp4_gemm_stream(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out,
                                    int64_t M, int64_t N, int d, hipStream_t stream) {
  const int MT = (int)((M + 15) / 16), PT = (d / 256 + WAVES - 1) / WAVES;
#define TORQ_STREAM(MT_, PT_) \
  if (MT == MT_ && PT == PT_) return launch_cfg<MT_, PT_, STREAM_RING>(A_q, A_s, W_q, W_s, out, M, N, d, stream);
  TORQ_STREAM(1, 2) TORQ_STREAM(1, 3) TORQ_STREAM(1, 4) TORQ_STREAM(2, 2) TORQ_STREAM(2, 3) TORQ_STREAM(2, 4)
  TORQ_STREAM(3, 2) TORQ_STREAM(3, 3) TORQ_STREAM(3, 4) TORQ_STREAM(4, 2) TORQ_STREAM(4, 3) TORQ_STREAM(4, 4)
#undef TORQ_STREAM
  return hipErrorInvalidValue;
}

}  // namespace torq
