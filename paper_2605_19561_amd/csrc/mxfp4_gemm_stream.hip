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
#include "rotate32_resident.h"
#include "torq_device.h"
#include "torq_internal.h"

namespace torq {

namespace {

constexpr int WAVES = 8;
constexpr int STREAM_RING = 4;                    // items of a wave's ring: 3 and 5 measured 1 - 4 % slower, 2, 6 and 8 more
constexpr size_t STREAM_MAX_LDS = 160 * 1024;
constexpr int OOB_VOFF = 0x7FFFFFF0;              // rejected by the range check of any buffer here: zeros

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// 16-byte units of a scale row in LDS: an odd number, so that the lanes of a k-step, which read one byte of 16 rows each,
// find them in different banks, but no more than the workgroup loads in one go, 512 for the 16 rows (up to d = 16384)
__host__ __device__ constexpr int stream_scale_units(int d) { return (d / 512 | 1) <= 32 ? d / 512 | 1 : d / 512; }
// buffers of scale rows: the one in use and those of the strips that the ring reaches ahead into
__host__ __device__ constexpr int stream_scale_buffers(int PT, int R) { return (R + PT - 1) / PT + 1; }

size_t stream_lds_bytes(int MT, int PT, int R, int d) {
  const size_t per = (16 * (size_t)stream_scale_units(d) + WAVES - 1) / WAVES * WAVES * 16;
  return (size_t)WAVES * R * 2048 + stream_scale_buffers(PT, R) * per + (size_t)2 * WAVES * MT * 1024;
}

}  // namespace

// What a wave of the two kernels below works with.  AT: how many activation tiles come through the ring ahead of the strips
// (the "strips" 0 ... AT - 1 of a workgroup; its weight strips follow).
// ONCE: the weights' codes with the non-temporal hint (ONE_PASS_WEIGHT_BYTES; the activations come from the L2 in every workgroup and
// go without: with it [64, 8192] x 20480 23.4 -> 24.5 us).
// LDS from `mem` on: [rings | buffers of scale rows | two buffers of partial tiles]
template <int MT, int PT, int R, int AT, bool ONCE>
struct Stream {
  static constexpr int BUFS = stream_scale_buffers(PT, R);
  static_assert(2 * R + BUFS <= 63, "the counter of loads in flight has six bits");
  const uint8_t *A_q, *A_s, *W_q, *W_s;
  uint16_t *out;
  int M, N, KP, row_bytes, srow_bytes;
  int lane, wave, r16, q;
  int first, step, count;                          // the workgroup's weight strips: first, first + step, ...
  int s_pitch, per_wave, sc_bytes, v0, v1, vs;
  int f_off[2];
  uint32_t ring0, sc0;
  const unsigned char *ring, *sc, *srow;
  f32x4 *red;                                      // [2][WAVES][MT][64]
  int slot = 0;
  u32x4 f0, f1;                                    // the item taken last: its two operands and their scales
  int w0, w1;

  __device__ __forceinline__ Stream(const uint8_t *A_q_, const uint8_t *A_s_, const uint8_t *W_q_, const uint8_t *W_s_, uint16_t *out_,
                                    int M_, int N_, int d, int strips_each, int strips_over, unsigned char *mem)
      : A_q(A_q_), A_s(A_s_), W_q(W_q_), W_s(W_s_), out(out_), M(M_), N(N_) {
    const int tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    r16 = lane & 15;
    q = lane >> 4;
    row_bytes = d / 2;
    srow_bytes = d / 32;
    KP = d / 256;
    first = blockIdx.x;
    step = gridDim.x;
    count = strips_each + (first < strips_over ? 1 : 0);           // at least one
    const int pu = stream_scale_units(d);
    s_pitch = pu * 16;
    per_wave = (16 * pu + WAVES - 1) / WAVES;
    sc_bytes = per_wave * WAVES * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)mem;
    ring0 = lds0 + wave * R * 2048;
    sc0 = lds0 + WAVES * R * 2048;
    ring = mem + wave * R * 2048;
    sc = srow = mem + WAVES * R * 2048;
    red = reinterpret_cast<f32x4 *>(mem + WAVES * R * 2048 + BUFS * sc_bytes);
    // chunks of an item swizzled by the row, as the operands' reads expect
    const int l_row = lane >> 3;
    v0 = l_row * row_bytes + ((lane & 7) ^ (l_row >> 1)) * 16;
    v1 = (l_row + 8) * row_bytes + ((lane & 7) ^ (l_row >> 1) ^ 4) * 16;
    f_off[0] = r16 * 128 + ((q ^ ((r16 >> 1) & 7)) * 16);
    f_off[1] = r16 * 128 + (((4 + q) ^ ((r16 >> 1) & 7)) * 16);
    const int unit = wave * per_wave + lane;
    const int row = (int)(((float)unit + 0.5f) * __builtin_amdgcn_rcpf((float)pu)), col = unit - row * pu;   // (unit / pu)
    vs = row < 16 && col < srow_bytes / 16 ? row * srow_bytes + col * 16 : OOB_VOFF;
  }

  __device__ __forceinline__ int row_of(int s) const { return s < AT ? 16 * s : s < AT + count ? (first + (s - AT) * step) * 16 : 0; }
  __device__ __forceinline__ int rows_of(int s) const {
    const int left = (s < AT ? M : s < AT + count ? N : 0) - row_of(s);
    return left < 16 ? left : 16;
  }
  // (the four words are the same in all lanes; the compiler takes some of them through vector registers)
  static __device__ __forceinline__ i32x4 uniform(i32x4 v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = __builtin_amdgcn_readfirstlane(v[j]);
    return v;
  }
  // Exactly two loads an item and one a strip's scale rows, whatever they bring: past the end of the k range or of the strips
  // they come from empty buffers.
  __device__ __forceinline__ void request(int s, int i, int to) {
    const int kp = wave + 8 * i;
    const i32x4 rs = uniform(raw_buffer((s < AT ? A_q : W_q) + (int64_t)row_of(s) * row_bytes, kp < KP ? (uint32_t)rows_of(s) * row_bytes : 0u));
    if (ONCE && s >= AT) {
      load_to_lds16<true, true>(rs, ring0 + to * 2048, v0, kp * 128);
      load_to_lds16<true, true>(rs, ring0 + to * 2048 + 1024, v1, kp * 128);
    } else {
      load_to_lds16(rs, ring0 + to * 2048, v0, kp * 128);
      load_to_lds16(rs, ring0 + to * 2048 + 1024, v1, kp * 128);
    }
  }
  __device__ __forceinline__ void request_scales(int s) {
    const i32x4 rs = uniform(raw_buffer((s < AT ? A_s : W_s) + (int64_t)row_of(s) * srow_bytes, (uint32_t)rows_of(s) * srow_bytes));
    if (lane < per_wave) load_to_lds16(rs, sc0 + (s % BUFS) * sc_bytes + wave * per_wave * 16, vs, 0);
  }
  // the ring's first R items, from item number H of the workgroup on
  template <int H>
  __device__ __forceinline__ void start() {
    static_for<R>([&](auto j_c) {
      constexpr int j = H + decltype(j_c)::value;
      if constexpr (j % PT == 0) request_scales(j / PT);
      request(j / PT, j % PT, j - H);
    });
  }
  // strip s begins: its scale rows have landed (this wave's part: the caller has waited), the strip before's partial tiles too
  __device__ __forceinline__ void meet(int s) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    srow = sc + (s % BUFS) * sc_bytes + r16 * s_pitch + q;
  }
  __device__ __forceinline__ void scales_of(int i) {
    const int kp = wave + 8 * i, so = kp < KP ? kp * 8 : 0;
    w0 = srow[so];
    w1 = srow[so + 4];
  }
  // Item i of strip s into f0, f1, w0, w1, and the request of the one R further on.  The items younger than it: R - 1, and
  // the scale rows of the strips that begin among them.
  template <int i, class F>
  __device__ __forceinline__ void take(int s, F &&at_start) {
    wait_vm<2 * (R - 1) + (i + R - 1) / PT>();
    if constexpr (i == 0) {
      meet(s);
      at_start();
    }
    f0 = *reinterpret_cast<const u32x4 *>(ring + slot * 2048 + f_off[0]);
    f1 = *reinterpret_cast<const u32x4 *>(ring + slot * 2048 + f_off[1]);
    scales_of(i);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // read: the slot can be filled again
    if constexpr ((i + R) % PT == 0) request_scales(s + (i + R) / PT);
    request(s + (i + R) / PT, (i + R) % PT, slot);
    slot = slot + 1 == R ? 0 : slot + 1;
  }
  __device__ __forceinline__ void multiply(f32x4 (&acc)[MT], const u32x4 (&a)[2][MT], const int (&as)[MT]) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
      acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
          i32x8{(int)f0[0], (int)f0[1], (int)f0[2], (int)f0[3], 0, 0, 0, 0},
          i32x8{(int)a[0][t][0], (int)a[0][t][1], (int)a[0][t][2], (int)a[0][t][3], 0, 0, 0, 0}, acc[t], 4, 4, 0, w0, 0, as[t]);
#pragma unroll
    for (int t = 0; t < MT; ++t)
      acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
          i32x8{(int)f1[0], (int)f1[1], (int)f1[2], (int)f1[3], 0, 0, 0, 0},
          i32x8{(int)a[1][t][0], (int)a[1][t][1], (int)a[1][t][2], (int)a[1][t][3], 0, 0, 0, 0}, acc[t], 4, 4, 0, w1, 1, as[t]);
  }
  // the wave's partial tiles of the workgroup's weight strip number s; and, one barrier later, their sums, added and stored
  // by the waves whose turn it is
  __device__ __forceinline__ void leave(int s, const f32x4 (&acc)[MT]) {
#pragma unroll
    for (int t = 0; t < MT; ++t) red[(((s & 1) * WAVES + wave) * MT + t) * 64 + lane] = acc[t];
  }
  __device__ __forceinline__ void reduce(int s) {
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
      const int nn = row_of(AT + s) + 4 * q;
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
  }
  // weight strips s0 ... of the workgroup, all of their items through the ring; nothing is in flight at the end
  __device__ __forceinline__ void strips(int s0, const u32x4 (&aq)[PT][2][MT], const int (&as)[PT][MT]) {
    for (int s = s0; s < count; ++s) {
      f32x4 acc[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      static_for<PT>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        take<i>(AT + s, [&]() { if (s > 0) reduce(s - 1); });
        multiply(acc, aq[i], as[i]);
      });
      leave(s, acc);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    reduce(count - 1);
  }
};

template <int MT, int PT, int R, bool ONCE>
__global__ void __launch_bounds__(64 * WAVES)
mxfp4_gemm_stream_kernel(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                         const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int N, int d, int strips_each, int strips_over) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  Stream<MT, PT, R, MT, ONCE> st(A_q, A_s, W_q, W_s, out, M, N, d, strips_each, strips_over, smem);
  st.template start<0>();
  // the activations: operand (i, e, t) = line pair wave + 8 i, k-step e of it, tile t; zeros past M and d
  u32x4 aq[PT][2][MT];
  int as[PT][MT];                                  // bytes 0 and 1: the lane's scales of the two k-steps
  static_for<MT>([&](auto t_c) {
    constexpr int t = decltype(t_c)::value;
    static_for<PT>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      st.template take<i>(t, []() {});
      aq[i][0][t] = st.f0;
      aq[i][1][t] = st.f1;
      as[i][t] = st.w0 | st.w1 << 8;
    });
  });
  st.strips(0, aq, as);
}

// ---------------------------------------------------------------------------------------------
// torq_linear in one launch for one to four token-groups (G = 112 or 128) and more weights than torq_linear_local_kernel
// (mxfp4_gemm_skinny.hip) is for.  As there every workgroup rotates and quantises the rows itself, into LDS, and the packed
// activations never leave the chip (workgroup 0 stores a copy for the caller).  The strips come through the ring as above.
// Only the first H items of a wave (H x 16 KB a CU) are requested together with the rotation's operands, and the ring starts
// when R_inter has been used: requested all at once, the weights keep the rotation's operands away until most of
// them have come.
template <int PT, int H, int R>
__global__ void __launch_bounds__(64 * WAVES)
torq_linear_stream_kernel(const uint4 *__restrict__ x, int TG, int G, const uint4 *__restrict__ inter_hi,
                          const uint4 *__restrict__ inter_lo, const uint4 *__restrict__ intra_hi_frag,
                          const uint4 *__restrict__ intra_lo_frag, uint8_t *__restrict__ A_q, uint8_t *__restrict__ A_s,
                          const uint8_t *__restrict__ W_q, const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int N,
                          int d, int strips_each, int strips_over) {
  static_assert(H >= 1 && H <= PT, "items of the first strip");
  // LDS: [stream_lds_bytes | scale rows of the activations, 16 | their codes, M rows padded by 16 bytes | token-groups, 4 x 8 KB]
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  Stream<1, PT, R, 0, false> st(nullptr, nullptr, W_q, W_s, out, M, N, d, strips_each, strips_over, smem);
  const int s_stride = st.srow_bytes + 4, a_stride = st.row_bytes + 16;
  unsigned char *const s_a = reinterpret_cast<unsigned char *>(st.red + 2 * WAVES * 64);
  unsigned char *const a_c = s_a + 16 * s_stride;
  unsigned char *const xs = a_c + M * a_stride;
  st.request_scales(0);
  for (int i = threadIdx.x; i < 4 * s_stride; i += 64 * WAVES) reinterpret_cast<uint32_t *>(s_a)[i] = 0u;

  u32x4 head[H][2];                                // strip 0's first items, in the operand's layout
  {
    LocalSink sink;
    sink.a_c = a_c;
    sink.s_a = s_a;
    sink.a_stride = a_stride;
    sink.s_stride = s_stride;
    sink.bpr = st.srow_bytes;
    sink.codes_g = blockIdx.x == 0 ? reinterpret_cast<uint2 *>(A_q) : nullptr;
    sink.scales_g = A_s;
    auto first_items = [&]() {
      // (the waves meet so that every wave's rotation reads are in the CU's memory pipeline before any wave's weights)
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<uint8_t *>(W_q) + (int64_t)st.row_of(0) * st.row_bytes, 0, st.rows_of(0) * st.row_bytes, 0x00020000);
#pragma unroll
      for (int i = 0; i < H; ++i) {
        // (a pair past the k range: out of range by arithmetic, a branch would leave the compiler's count of these loads open)
        const int kp = st.wave + 8 * i, voff = st.r16 * st.row_bytes + st.q * 16 + (((st.KP - 1 - kp) >> 31) & 0x70000000);
#pragma unroll
        for (int e = 0; e < 2; ++e) head[i][e] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, kp * 128 + e * 64, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto ring = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0x0F70);          // the compiler's own loads, and this wave's part of strip 0's scale rows
      st.template start<H>();
      __builtin_amdgcn_sched_barrier(0);
    };
    // (barriers inside: the first orders the clearing above before any scale byte, the last makes the results visible)
    rotate32_resident(x, TG, G, inter_hi, inter_lo, intra_hi_frag, intra_lo_frag, reinterpret_cast<char *>(xs), sink, first_items, ring);
  }
  u32x4 aq[PT][2][1];
  int as[PT][1];
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int kp = st.wave + 8 * i;
    const bool ok = kp < st.KP && st.r16 < M;
    const unsigned char *const c = a_c + st.r16 * a_stride + kp * 128 + st.q * 16, *const b = s_a + st.r16 * s_stride + kp * 8 + st.q;
    aq[i][0][0] = ok ? *reinterpret_cast<const u32x4 *>(c) : u32x4{0u, 0u, 0u, 0u};
    aq[i][1][0] = ok ? *reinterpret_cast<const u32x4 *>(c + 64) : u32x4{0u, 0u, 0u, 0u};
    as[i][0] = ok ? b[0] | b[4] << 8 : 0;
  }
  st.srow = st.sc + st.r16 * st.s_pitch + st.q;
  f32x4 acc[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
  static_for<PT>([&](auto i_c) {
    constexpr int i = decltype(i_c)::value;
    if constexpr (i < H) {
      st.f0 = head[i][0];
      st.f1 = head[i][1];
      st.scales_of(i);
    } else {
      st.template take<i>(0, []() {});
    }
    st.multiply(acc, aq[i], as[i]);
  });
  st.leave(0, acc);
  st.strips(1, aq, as);
}

template <int MT, int PT, int R, bool ONCE>
static hipError_t launch_cfg(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M,
                             int64_t N, int d, hipStream_t stream) {
  const size_t lds = stream_lds_bytes(MT, PT, R, d);
  if (lds > STREAM_MAX_LDS) return hipErrorInvalidValue;
  auto kernel = mxfp4_gemm_stream_kernel<MT, PT, R, ONCE>;
  if (lds > 64 * 1024) {
    static std::atomic<uint64_t> raised{0};
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(kernel), STREAM_MAX_LDS, raised);
    if (e != hipSuccess) return e;
  }
  const int64_t strips = (N + 15) / 16;
  const int64_t grid = strips < 256 ? strips : 256;
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * WAVES), lds, stream, A_q, A_s, W_q, W_s,
                     reinterpret_cast<uint16_t *>(out), (int)M, (int)N, d, (int)(strips / grid), (int)(strips % grid));
  return hipGetLastError();
}

// Whether the product (d a multiple of 512, 16-byte aligned scale rows) is one for strips through a ring where the whole-line
// form does not take it: line pairs of two to four per wave and strip (d = 2560 ... 8192; the activations' operands would not
// fit the registers beyond), and strips enough for a workgroup's start, the activations through its ring, to be paid off.
// Weights from HBM, us, what the planner took before against this form:
//   8 - 16 rows past 1600 strips (two strips a workgroup, persistent): [8, 8192] x 28672 27.8 / 25.8, [16, 8192] x 28672 28.7 /
//     23.8; below that the whole-line form stays
//   fewer than 8 rows (strips straight to registers, which are 3 % ahead of this form without the non-temporal hint): weights
//     that take the hint, [1, 8192] x 28672 24.8 / 23.6, x 24576 21.3 / 20.4, [4, 8192] x 28672 27.1 / 23.9, [7, 8192] x 26624
//     27.2 / 22.8
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
  if (d % 512 != 0 || d < 2560 || d > 8192 || N > (1 << 30)) return false;
  if (M < 8) return (double)N * (double)d * 0.53125 > ONE_PASS_WEIGHT_BYTES;
  if (M > 64) return false;
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
  const bool once = (double)N * (double)d * 0.53125 > ONE_PASS_WEIGHT_BYTES;
  // (one activation tile of d > 6144 has as much wherever the rule takes it)
  if (MT == 1 && PT == 4) return launch_cfg<1, 4, STREAM_RING, true>(A_q, A_s, W_q, W_s, out, M, N, d, stream);
#define TORQ_STREAM(MT_, PT_)                                                                                                   \
  if (MT == MT_ && PT == PT_)                                                                                                  \
    return once ? launch_cfg<MT_, PT_, STREAM_RING, true>(A_q, A_s, W_q, W_s, out, M, N, d, stream)                            \
                : launch_cfg<MT_, PT_, STREAM_RING, false>(A_q, A_s, W_q, W_s, out, M, N, d, stream);
  TORQ_STREAM(1, 2) TORQ_STREAM(1, 3) TORQ_STREAM(2, 2) TORQ_STREAM(2, 3) TORQ_STREAM(2, 4)
  TORQ_STREAM(3, 2) TORQ_STREAM(3, 3) TORQ_STREAM(3, 4) TORQ_STREAM(4, 2) TORQ_STREAM(4, 3) TORQ_STREAM(4, 4)
#undef TORQ_STREAM
  return hipErrorInvalidValue;
}

static size_t linear_stream_lds_bytes(int64_t M, int d, int PT) {
  return stream_lds_bytes(1, PT, STREAM_RING, d) + 16 * (size_t)(d / 32 + 4) + (size_t)M * (d / 2 + 16) + 4 * 8192;
}

template <int PT>
static hipError_t launch_linear_cfg(const torq_rotation *r, const void *x, uint8_t *A_q, uint8_t *A_s, const uint8_t *W_q,
                                    const uint8_t *W_s, void *out, int64_t M, int64_t N, hipStream_t stream) {
  const size_t lds = linear_stream_lds_bytes(M, r->d, PT);
  if (lds > STREAM_MAX_LDS) return hipErrorInvalidValue;
  auto kernel = torq_linear_stream_kernel<PT, 2, STREAM_RING>;
  static std::atomic<uint64_t> raised{0};
  const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(kernel), STREAM_MAX_LDS, raised);
  if (e != hipSuccess) return e;
  const int64_t strips = (N + 15) / 16, grid = strips < 256 ? strips : 256;
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * WAVES), lds, stream, reinterpret_cast<const uint4 *>(x),
                     (int)(M * (int64_t)(r->d / 32 / r->G)), r->G, reinterpret_cast<const uint4 *>(r->inter32f_hi),
                     reinterpret_cast<const uint4 *>(r->inter32f_lo), reinterpret_cast<const uint4 *>(r->intra32_hi),
                     reinterpret_cast<const uint4 *>(r->intra32_lo), A_q, A_s, W_q, W_s, reinterpret_cast<uint16_t *>(out), (int)M,
                     (int)N, r->d, (int)(strips / grid), (int)(strips % grid));
  return hipGetLastError();
}

// Where it takes the place of torq_linear_local_kernel (and, with more weights than that form is for, of two launches).  One
// launch of this form against the faster of those, weights from HBM, us:
//   one or two token-groups, up to 80 MB of weights ([1, 4096] x 14336 10.9 / 9.9, x 28672 16.9 / 14.5, [2, 4096] x 14336 10.9 /
//     9.9, [1, 8192] x 1024 6.6 / 6.1, x 14336 17.9 / 15.7, [1, 3584] x 4096 6.9 / 6.3, [1, 7168] x 4096 9.0 / 7.4; [1, 8192] x
//     28672 27.5 / 26.4 replayed from a graph, but 25.7 / 26.3 called one after the other) but where a workgroup's share is
//     a strip that the other form requests all at once, in one full trip of each wave ([1, 4096] x 4096 5.7 / 6.5, x 1024 5.2 / 5.6;
//     d = 3584 does not fill the trip, its loads there are under a condition, and a strip of d = 8192 is 64 KB)
//   three or four: up to a strip a workgroup of d <= 7168, up to half as many beyond: [4, 3584] x 4096 8.4 / 7.6, [2, 7168] x
//     4096 10.5 / 9.2, [1, 14336] x 2048 10.7 / 9.0, but [4, 4096] x 4096 7.1 / 8.0 (all at once), [2, 8192] x 4096 9.2 / 9.4, [1, 14336] x
//     4096 11.3 / 10.5 to 12.2 (and not beyond seven line pairs a wave, the most that are built); with more strips the second token-group of a wave keeps the ring waiting ([4, 4096] x 14336 11.0 /
//     11.4, [2, 7168] x 14336 15.1 / 16.2)
// (the first strip's items requested with the rotation's operands, one / two / three / four: [1, 8192] x 28672 26.3 / 26.4 / 26.0 /
// 25.7, x 1024 6.0 / 6.1 / 6.4 / 6.8, [1, 14336] x 4096 11.6 / 10.5 / 10.5 / 11.1)
bool torq_linear_stream_takes(const torq_rotation *r, int64_t M, int64_t N, const uint8_t *W_s) {
  if (!torq_linear_local_fits(r, M) || N < 1 || N > (1 << 30) || r->d % 512 != 0 || (reinterpret_cast<uintptr_t>(W_s) & 15u)) return false;
  const int64_t token_groups = M * (int64_t)(r->d / 32 / r->G), strips = (N + 15) / 16;
  // the other form's EXACT loop on two line pairs a wave or fewer: a strip of 32 KB at most
  const int trip = 256 * WAVES;
  const bool at_once = r->d % trip == 0 && r->d <= 2 * trip;
  if (token_groups <= 2) return !(at_once && strips <= 256) && (double)N * (double)r->d * 0.53125 <= 80e6;
  return !at_once && r->d <= 7 * trip && strips <= (r->d <= 7168 ? 256 : 128);
}

hipError_t launch_torq_linear_stream(const torq_rotation *r, const void *x, uint8_t *A_q, uint8_t *A_s, const uint8_t *W_q,
                                     const uint8_t *W_s, void *out, int64_t M, int64_t N, hipStream_t stream) {
  // (d is a multiple of 32 G with at most four token-groups a row: 3584, 4096 and their multiples up to 14336)
  switch ((r->d / 256 + WAVES - 1) / WAVES) {
    case 2: return launch_linear_cfg<2>(r, x, A_q, A_s, W_q, W_s, out, M, N, stream);
    case 4: return launch_linear_cfg<4>(r, x, A_q, A_s, W_q, W_s, out, M, N, stream);
    case 6: return launch_linear_cfg<6>(r, x, A_q, A_s, W_q, W_s, out, M, N, stream);
    case 7: return launch_linear_cfg<7>(r, x, A_q, A_s, W_q, W_s, out, M, N, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace torq
