// mxfp4_gemm for products of few tiles: the tiled W4A4 product of mxfp4_gemm.hip (Section 5; Algorithm 3, "Return";
// the same arithmetic in the same order of the k-steps, the same bits) with its operands staged in a ring.
//
// Bound: the latency of a workgroup's own loads.  A CU keeps about 32 KB on their way (measured: 57 bytes/ns from HBM
// with 32 KB in flight or with 256, 85 from the Infinity Cache, 148 from the L2), the matrix cores want 32 KB every
// 0.21 us for a 128 x 128 tile, and up to a few hundred tiles nothing else hides the difference.  So the next three
// iterations are always on their way, straight into LDS (no staging registers, no LDS stores, one barrier an
// iteration), and tiles go down to 64 x 64, which cut the output finely and leave a CU room for two.  Against the form
// that staged through registers (128 x 128 and 128 x 64 tiles, two or three iterations ahead, two barriers), us, weights
// from HBM: [100, 4096] x 4096 11.2 -> 6.8, [300, 1024] x 520 5.2 -> 4.0, [512, 4096] x 4096 11.9 -> 9.9,
// [333, 14336] x 4096 33.0 -> 30.3; over 320 random shapes of 65 ... 2048 rows 1.19 times faster on average.
// Six and eight stages measured the same or slower (one workgroup a CU), two stages slower beyond 1024 elements,
// loads that only bring the next iterations' lines into the L2 slower (they take their share of the 32 KB).
#include "torq_device.h"
#include "torq_internal.h"

namespace torq {

namespace {

// every DMA but the youngest N of this wave has landed, every LDS read of it has returned; then the workgroup meets
template <int N>
__device__ __forceinline__ void ring_meet() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// n / D for 0 <= n < 2^31 by a product: mul = ceil(2^(31 + s) / D), 2^s the power of two at or above D
struct Quotient {
  uint32_t mul, shift;
};
static Quotient quotient_by(int64_t D) {
  uint32_t s = 0;
  while ((int64_t)1 << s < D) ++s;
  return Quotient{(uint32_t)((((uint64_t)1 << (31 + s)) + (uint64_t)D - 1) / (uint64_t)D), 31 + s};
}
__device__ __forceinline__ int quotient(int n, Quotient q) { return (int)(((uint64_t)(uint32_t)n * q.mul) >> q.shift); }

constexpr int NST = 4, NSB = 2;       // stages of codes, buffers of scale bytes

}  // namespace

// Workgroup = 4 waves (2 x 2); wave tiles, fragments, LDS swizzle and scales as in mxfp4_gemm_kernel.  An iteration is
// 256 elements of k; iteration k's codes go to stage k % 4, the scale bytes of iterations 2 q and 2 q + 1 to buffer
// q % 2.  At the barrier inside iteration k, behind the last fragment read of its stage, every wave waits for its own
// part of iteration k + 1 and, once all have met, requests iteration k + 4 into the stage just freed (odd k: the next
// but one pair's scale bytes first).  Requests return in order, so "iteration k + 1 is here" is a count of the younger
// ones: the codes of k + 2 and k + 3, and for even k the scale bytes requested in between.  The loop's loads are inline
// assembly, which keeps the compiler from waiting for all of them in front of every LDS read; past the end the
// requests go to empty buffers, so that the count holds.
// SPLIT: blockIdx.y is the piece of the k range, its fp32 sums go to partial[blockIdx.y][M][N].
template <int WM, int WN, bool SPLIT>
__global__ void __launch_bounds__(256)
mxfp4_gemm_ring_kernel(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                       const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, float *__restrict__ partial, int64_t M,
                       int64_t N, int d, int tiles_m, int tiles_n, int64_t ldc, Quotient by_columns, Quotient by_rows) {
  constexpr int BM = 64 * WM, BN = 64 * WN;
  constexpr int A_CH = BM / 32, W_CH = BN / 32, C = A_CH + W_CH;   // DMA instructions of a wave per iteration
  constexpr int ROWS = (BM + BN + 255) / 256 * 256, S = ROWS / 256;  // scale rows (padded), DMA instructions per pair
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128, SBUF = ROWS * 16, S_BASE = NST * STAGE;
  extern __shared__ __attribute__((aligned(16))) char lds[];

  const int total = tiles_m * tiles_n;
  int lid = blockIdx.x;
  if (total % 8 == 0) lid = (lid % 8) * (total / 8) + lid / 8;     // contiguous runs of tiles per XCD
  // Down eight tile rows, then the next column, as in mxfp4_gemm_kernel: the tiles that an XCD runs at a time share rows of A
  // as well as of W, and where the tile count is no multiple of 8 every eighth tile is on the same tile row.  Down all
  // rows first each XCD fetched most of A once a column: tall products, best ring form, us: [1826, 21504] x 640 33.7 ->
  // 28.3, [8733, 2048] x 392 15.3 -> 12.1, [17308, 3072] x 132 22.5 -> 18.1.
  // (Quotients by the host's multipliers, and no branch: around one the kernel's arguments arrive one after the other, 0.2 us
  // ahead of the first load.)
  const int first = quotient(lid >> 3, by_columns) * 8, rest = lid - first * tiles_n;      // (0 up to eight tile rows)
  const int rows = min(tiles_m - first, 8), by_last = quotient(rest, by_rows);
  const int tn = rows == 8 ? rest >> 3 : by_last, tm = first + rest - tn * rows;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int rows_a = (M - m0 < BM) ? (int)(M - m0) : BM, rows_w = (N - n0 < BN) ? (int)(N - n0) : BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wy = wave >> 1, wx = wave & 1;
  const int lrow = lane & 31, g = lane >> 5;
  const int row_bytes = d / 2, srow_bytes = d / 32;
  const int KT = d / 256;
  const int count = SPLIT ? KT / (int)gridDim.y : KT;      // even
  const int kt0 = SPLIT ? (int)blockIdx.y * count : 0;

  const i32x4 a_rs = raw_buffer(A_q + m0 * row_bytes, (uint32_t)rows_a * row_bytes);
  const i32x4 w_rs = raw_buffer(W_q + n0 * row_bytes, (uint32_t)rows_w * row_bytes);
  const i32x4 as_rs = raw_buffer(A_s + m0 * srow_bytes, (uint32_t)rows_a * srow_bytes);
  const i32x4 ws_rs = raw_buffer(W_s + n0 * srow_bytes, (uint32_t)rows_w * srow_bytes);
  const int c_row = tid >> 3;
  const int c_voff = c_row * row_bytes + (((tid & 7) ^ ((c_row >> 1) & 7)) * 16);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;

  auto empty = [](i32x4 r, bool ok) { r[2] = ok ? r[2] : 0; return r; };
  // chunk c (32 rows of a wave's DMA each) of an iteration's codes into stage slot: the weights first
  auto code_chunk = [&](int c, i32x4 ra, i32x4 rw, int ko, int slot) {
    const int i = c < W_CH ? c : c - W_CH;
    load_to_lds16<false>(c < W_CH ? rw : ra, lds0 + slot * STAGE + (c < W_CH ? A_BYTES : 0) + i * 4096 + wave * 1024, c_voff, ko + i * 32 * row_bytes);
  };
  auto load_codes = [&](int k, int slot) {
    const bool ok = k < count;
    const i32x4 ra = empty(a_rs, ok), rw = empty(w_rs, ok);
#pragma unroll
    for (int c = 0; c < C; ++c) code_chunk(c, ra, rw, (kt0 + k) * 128, slot);
  };
  // scale bytes of iterations 2 q and 2 q + 1 into scale buffer sb
  auto load_scales = [&](int q, int sb) {
    const bool ok = 2 * q < count;
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int r0 = i * 256 + wave * 64;                          // BM is a multiple of 64
      const bool is_a = r0 < BM;
      const i32x4 rs = empty(is_a ? as_rs : ws_rs, ok && r0 < BM + BN);
      load_to_lds16<false>(rs, lds0 + S_BASE + sb * SBUF + r0 * 16, lane * srow_bytes, (is_a ? r0 : r0 - BM) * srow_bytes + (kt0 / 2 + q) * 16);
    }
  };

  // fragments and scale bytes: the addresses of mxfp4_gemm_kernel, relative to a stage or buffer
  const int f_sw = (lrow >> 1) & 7;
  int fa_off[4], fw_off[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int ch = ((4 * g + ks) ^ f_sw) * 16;
    fa_off[ks] = (wy * WM * 32 + lrow) * 128 + ch;
    fw_off[ks] = A_BYTES + (wx * WN * 32 + lrow) * 128 + ch;
  }
  const int sa_off = S_BASE + (wy * WM * 32 + lrow) * 16 + 4 * g;
  const int sw_off = S_BASE + (BM + wx * WN * 32 + lrow) * 16 + 4 * g;

  f32x16 acc[WN][WM];
#pragma unroll
  for (int j = 0; j < WN; ++j)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  i32x4 fa[2][WM], fw[2][WN];
  uint32_t sa[2][WM], sw[2][WN];
  auto frags = [&](int set, int slot, int ks) {
    const char *p = lds + slot * STAGE;
#pragma unroll
    for (int i = 0; i < WM; ++i) fa[set][i] = *reinterpret_cast<const i32x4 *>(p + fa_off[ks] + i * 4096);
#pragma unroll
    for (int j = 0; j < WN; ++j) fw[set][j] = *reinterpret_cast<const i32x4 *>(p + fw_off[ks] + j * 4096);
  };
  auto scale_regs = [&](int par, int sb) {
    const char *p = lds + sb * SBUF + par * 8;
#pragma unroll
    for (int i = 0; i < WM; ++i) sa[par][i] = *reinterpret_cast<const uint32_t *>(p + sa_off + i * 512);
#pragma unroll
    for (int j = 0; j < WN; ++j) sw[par][j] = *reinterpret_cast<const uint32_t *>(p + sw_off + j * 512);
  };
#define RING_MFMA_ONE(SET_, PAR_, KS_, J_, I_)                                                    \
  acc[J_][I_] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(                                  \
      i32x8{fw[SET_][J_][0], fw[SET_][J_][1], fw[SET_][J_][2], fw[SET_][J_][3], 0, 0, 0, 0},      \
      i32x8{fa[SET_][I_][0], fa[SET_][I_][1], fa[SET_][I_][2], fa[SET_][I_][3], 0, 0, 0, 0},      \
      acc[J_][I_], 4, 4, KS_, sw[PAR_][J_], KS_, sa[PAR_][I_]);
#define RING_MFMA(SET_, PAR_, KS_)                                                                \
  _Pragma("unroll") for (int j = 0; j < WN; ++j) _Pragma("unroll") for (int i = 0; i < WM; ++i) { RING_MFMA_ONE(SET_, PAR_, KS_, j, i) }

#pragma unroll
  for (int k = 0; k < NST; ++k) {
    if (k & 1) load_scales(k / 2, k / 2);
    load_codes(k, k);
  }
  ring_meet<(NST - 1) * C + (NSB - 1) * S>();
  scale_regs(0, 0);
  frags(0, 0, 0);

  int slot = 0, sb = 0;
#define SGB(MASK_, N_) __builtin_amdgcn_sched_group_barrier(MASK_, N_, 0);
#define SG_MFMA 0x008
#define SG_DS_RD 0x100
#define RING_ITER(PAR_, KT_)                                                                      \
  {                                                                                               \
    const int nslot = slot + 1 == NST ? 0 : slot + 1, nsb = sb + 1 == NSB ? 0 : sb + 1;           \
    frags(1, slot, 1);                                                                            \
    RING_MFMA(0, PAR_, 0)                                                                         \
    frags(0, slot, 2);                                                                            \
    RING_MFMA(1, PAR_, 1)                                                                         \
    frags(1, slot, 3);                                                                            \
    RING_MFMA(0, PAR_, 2)                                                                         \
    _Pragma("unroll") for (int n_ = 0; n_ < 3; ++n_) {                                            \
      _Pragma("unroll") for (int q_ = 0; q_ < WM * WN; ++q_) { SGB(SG_MFMA, 1) SGB(SG_DS_RD, 2) } \
    }                                                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    ring_meet<(NST - 2) * C + (NSB - (PAR_ ? 2 : 1)) * S>();         \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    scale_regs((PAR_) ^ 1, (PAR_) ? nsb : sb);                                                    \
    frags(0, nslot, 0);                                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    if (PAR_) load_scales((KT_) / 2 + NSB, sb);                                                   \
    const bool ok_ = (KT_) + NST < count;                                                         \
    const i32x4 ra_ = empty(a_rs, ok_), rw_ = empty(w_rs, ok_);                                   \
    const int ko_ = (kt0 + (KT_) + NST) * 128;                                                    \
    _Pragma("unroll") for (int q_ = 0; q_ < WM * WN; ++q_) {                                      \
      RING_MFMA_ONE(1, PAR_, 3, q_ / WM, q_ % WM)                                                 \
      _Pragma("unroll") for (int c_ = q_ * C / (WM * WN); c_ < (q_ + 1) * C / (WM * WN); ++c_)    \
        code_chunk(c_, ra_, rw_, ko_, slot);                                                      \
      __builtin_amdgcn_sched_barrier(0);                                                          \
    }                                                                                             \
    if (PAR_) sb = nsb;                                                                           \
    slot = nslot;                                                                                 \
  }
  for (int kt = 0; kt < count; kt += 2) {
    RING_ITER(0, kt)
    RING_ITER(1, kt + 1)
  }
#undef RING_ITER
#undef RING_MFMA
#undef RING_MFMA_ONE
#undef SGB
  ring_meet<0>();                                  // (what follows reuses the stages) nothing is on its way into the LDS any more

  if constexpr (SPLIT)
    store_sums<WM, WN>(acc, partial + (size_t)blockIdx.y * (size_t)M * (size_t)N, m0, n0, wy, wx, M, N, lrow, g);
  else
    store_bf16<WM, WN>(acc, lds + wave * (32 * WM) * (64 * WN + 16), out, m0, n0, wy, wx, M, N, ldc, lane, lrow, g);
}

template <int WM, int WN>
static hipError_t launch_ring(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out,
                              float *partial, int splits, int64_t M, int64_t N, int d, int64_t ldc, hipStream_t stream) {
  constexpr int BM = 64 * WM, BN = 64 * WN, ROWS = (BM + BN + 255) / 256 * 256;
  constexpr size_t lds = (size_t)NST * (BM + BN) * 128 + (size_t)NSB * ROWS * 16;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  if (tiles_m * tiles_n > 0x7FFFFFFF) return hipErrorInvalidValue;
  auto go = [&](auto kern, std::atomic<uint64_t> &raised) {
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(kern), lds, raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n), splits), dim3(256), lds, stream, A_q, A_s, W_q, W_s,
                       reinterpret_cast<uint16_t *>(out), partial, M, N, d, (int)tiles_m, (int)tiles_n, ldc,
                       tiles_m > 8 ? quotient_by(tiles_n) : Quotient{0, 0}, quotient_by(tiles_m > 8 && tiles_m % 8 ? tiles_m % 8 : tiles_m));
    return hipGetLastError();
  };
  static std::atomic<uint64_t> raised[2];
  return splits > 1 ? go(mxfp4_gemm_ring_kernel<WM, WN, true>, raised[1]) : go(mxfp4_gemm_ring_kernel<WM, WN, false>, raised[0]);
}

hipError_t launch_mxfp4_gemm_ring(int tile_m, int tile_n, const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q,
                                  const uint8_t *W_s, void *out, float *partial, int splits, int64_t M, int64_t N, int d,
                                  int64_t ldc, hipStream_t stream) {
#define TORQ_RING(WM_, WN_)                      \
  if (tile_m == 64 * WM_ && tile_n == 64 * WN_)  \
    return launch_ring<WM_, WN_>(A_q, A_s, W_q, W_s, out, partial, splits, M, N, d, ldc, stream);
  TORQ_RING(2, 2) TORQ_RING(2, 1) TORQ_RING(1, 2) TORQ_RING(1, 1)
#undef TORQ_RING
  return hipErrorInvalidValue;
}

}  // namespace torq
