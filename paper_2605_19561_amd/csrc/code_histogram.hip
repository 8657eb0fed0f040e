// torq_code_histogram: the column-wise codebook histogram of the intra-block calibration
// (Appendix A.5, N_j^(k); Section 5.2, the occupancy that the equilibrium loss is made of):
//
//   counts[k][j] = number of 32-element blocks whose element k carries the magnitude codeword j
//
// over the packed e2m1 codes that the quantiser wrote (the sign bit of a code is ignored).
//
// One lane = one block = one 16-byte load; dword w of it holds the elements 8 w .. 8 w + 7, one per
// nibble, element 8 w in the lowest.  Nothing is decoded element by element.  With b0 b1 b2 the
// three magnitude bits of a nibble, the lane counts, per nibble position, the seven monomials
//   b0, b1, b2, b0 b1, b0 b2, b1 b2, b0 b1 b2
// eight positions at a time with whole-dword AND / shift / ADD into nibble-packed counters (nine
// logic operations and seven additions per dword).  The eight codeword counts follow from the
// monomial sums and the number of blocks by inclusion-exclusion, once, in the final kernel.
// Nibble counters hold 15: after 12 blocks the lanes of the wave are added by the matrix cores
// (add_lanes), into 32-bit sums.  Loads are buffer loads in groups of four with two groups in flight
// beyond the one being counted; a block past the end of the input reads as zeros (the buffer's range
// check), and a zero nibble adds to no monomial.  Every workgroup writes its 224 totals; the final kernel
// adds them (integers: any order gives the same result).
// HBM bound: half a byte per element, read once; the counting is 64 vector operations per block and
// wave, 3.4 us of the vector units' time at 2^21 blocks, beside 6 us of reading.  What follows the last load is
// not hidden by anything, so it is kept short.  An earlier form widened the nibbles into byte counters after
// 15 blocks and added the lanes through LDS: 14.7 us for the
// call at 2^21 blocks (codes of [8192, 8192]), 7.5 us at 512; this one 11.8 us and 5.6 us.  The loads carry the non-temporal
// hint at any size, us without / with it: from HBM 2^21 blocks 12.7 / 12.3, 2^23 29.8 / 27.5, 2^25 97.0 / 83.7, 31000 6.65 / 6.0; one
// input again the same up to 2^21 and 18.2 / 16.0 at 2^22; codes that the rotation has just packed, with the rotation, 17.6 /
// 16.9 at 2^18, 61.9 / 63.1 (a run's spread is 6) at 2^21, and of eight inputs rotated one after the other and counted then, a
// pair, 63.6 / 61.9 at 2^21 and 109.3 / 107.6 at 2^22 (codes that a plain element-wise kernel has
// just written, with it, 17.0 / 18.3 at 2^20, 37.8 / 39.2 at 2^22, 124 / 121 at 2^24).
#include "torq_device.h"
#include "torq_internal.h"

namespace torq {

constexpr int HIST_THREADS = 256;
constexpr int HIST_MAX_WG = 512;          // two resident workgroups per CU: one round
constexpr int HIST_GROUP = 4;             // blocks per lane per group of loads
constexpr int HIST_CHUNK = 3 * HIST_GROUP; // blocks per lane between two additions of the lanes
constexpr int HIST_MONO = 7;
constexpr int HIST_QUADS = 2 * HIST_MONO; // quadruples of byte words per lane, one matrix product each
constexpr int HIST_PARTIAL = HIST_MONO * 32;   // per workgroup: [monomial][position]
static_assert(HIST_CHUNK <= 15, "counter width");

typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4_t;

__global__ void __launch_bounds__(HIST_THREADS)
code_histogram_kernel(const uint8_t *__restrict__ codes, int64_t nblk, uint32_t *__restrict__ partial) {
  __shared__ uint32_t lds[HIST_THREADS / 16][HIST_PARTIAL];

  const int tid = threadIdx.x;
  const int64_t lanes = (int64_t)gridDim.x * HIST_THREADS;
  const int64_t per_lane = (nblk + lanes - 1) / lanes;                // uniform trip count
  const int ngroup = (int)((per_lane + HIST_GROUP - 1) / HIST_GROUP);
  // the workgroup's blocks are one contiguous span: [wg_first, wg_end)
  const int64_t wg_first = (int64_t)blockIdx.x * per_lane * HIST_THREADS;
  const int64_t wg_end = (wg_first + per_lane * HIST_THREADS < nblk) ? wg_first + per_lane * HIST_THREADS : nblk;
  const int voff = tid * 16;
  constexpr int ROW_BYTES = HIST_THREADS * 16;                        // one block per lane
  constexpr uint32_t K1 = 0x11111111u, KB = 0x0F0F0F0Fu;

  // Group g = the blocks wg_first + (HIST_GROUP g + i) * 256 + lane, i < HIST_GROUP: consecutive lanes
  // read consecutive 16-byte blocks.  The buffer resource starts at the group's first block and
  // ends at the end of the span, so a block past the end reads as zeros.
  auto load_group = [&](u32x4 (&v)[HIST_GROUP], int g) {
    const int64_t first = wg_first + (int64_t)g * HIST_GROUP * HIST_THREADS, left = (wg_end - first) * 16;
    const uint32_t records = left <= 0 ? 0u : (left > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)left);
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(codes) + (left <= 0 ? 0 : first * 16), 0, (int)records, 0x00020000);
#pragma unroll
    for (int i = 0; i < HIST_GROUP; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, i * ROW_BYTES, LOAD_POLICY<true>);
  };

  uint32_t nib[HIST_MONO][4];
  auto count_group = [&](const u32x4 (&v)[HIST_GROUP]) {
#pragma unroll
    for (int i = 0; i < HIST_GROUP; ++i)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t x = v[i][w], y = x >> 1, z = x >> 2;
        const uint32_t m0 = x & K1, m1 = y & K1, m2 = z & K1;
        const uint32_t m01 = m0 & y, m02 = m0 & z, m12 = m1 & z, m012 = m01 & z;
        nib[0][w] += m0;
        nib[1][w] += m1;
        nib[2][w] += m2;
        nib[3][w] += m01;
        nib[4][w] += m02;
        nib[5][w] += m12;
        nib[6][w] += m012;
      }
  };

  // Sums over lanes by v_mfma_i32_16x16x64_i8.  As A, lane l holds row l % 16 and, of the 64 k, the sixteen
  // of its quarter l / 16: four words of byte counters, byte j of them k = 16 (l / 16) + j.  B has a one where
  // k % 16 is the column, so D[row][j] += the byte j of the four lanes that share the row.  Quad 2 m has the even
  // nibbles of monomial m (bytes 4 w + s: position 8 w + 2 s), 2 m + 1 the odd ones.
  i32x4_t sum[HIST_QUADS];
#pragma unroll
  for (int q = 0; q < HIST_QUADS; ++q) sum[q] = i32x4_t{0, 0, 0, 0};
  i32x4_t pick;
#pragma unroll
  for (int w = 0; w < 4; ++w) pick[w] = ((tid & 15) >> 2) == w ? 1 << (8 * (tid & 3)) : 0;
  auto add_lanes = [&]() {
#pragma unroll
    for (int m = 0; m < HIST_MONO; ++m) {
      i32x4_t even, odd;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        even[w] = (int)(nib[m][w] & KB);
        odd[w] = (int)((nib[m][w] >> 4) & KB);
      }
      sum[2 * m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(even, pick, sum[2 * m], 0, 0, 0);
      sum[2 * m + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(odd, pick, sum[2 * m + 1], 0, 0, 0);
    }
  };

  u32x4 v0[HIST_GROUP], v1[HIST_GROUP], v2[HIST_GROUP];   // two groups in flight beyond the one being counted
  load_group(v0, 0);
  load_group(v1, 1);
  for (int g = 0; g < ngroup; g += 3) {
#pragma unroll
    for (int m = 0; m < HIST_MONO; ++m)
#pragma unroll
      for (int w = 0; w < 4; ++w) nib[m][w] = 0;
    load_group(v2, g + 2);
    count_group(v0);
    load_group(v0, g + 3);
    if (g + 1 < ngroup) count_group(v1);
    load_group(v1, g + 4);
    if (g + 2 < ngroup) count_group(v2);
    add_lanes();
  }

  // D: lane l holds column l % 16, rows 4 (l / 16) + r.  Sixteen partial sums per column and quad are left in the
  // workgroup, one per quarter of a wave.
#pragma unroll
  for (int q = 0; q < HIST_QUADS; ++q) lds[tid >> 4][16 * q + (tid & 15)] = sum[q][0] + sum[q][1] + sum[q][2] + sum[q][3];
  __syncthreads();
  if (tid < HIST_PARTIAL) {
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < HIST_THREADS / 16; ++i) total += lds[i][tid];
    // byte 4 w + s of quad 2 m + odd.  The partial sums are stored counter-major, [counter][workgroup], for the
    // final kernel's coalesced reads.
    const int m = tid >> 5, odd = (tid >> 4) & 1, w = (tid >> 2) & 3, s = tid & 3;
    partial[(size_t)(m * 32 + 8 * w + 2 * s + odd) * HIST_MAX_WG + blockIdx.x] = total;
  }
}

// Workgroup k of 32, a wave per monomial m (and an idle eighth): each lane adds the partial sums of eight
// workgroups, the wave adds its lanes, and eight threads turn
// (N, s0, s1, s2, s01, s02, s12, s012) into the eight codeword counts of position k by
// inclusion-exclusion.  All latency: the launch, one trip to memory, the wave's six exchanges.  (With 128 slices
// added in LDS by one thread per monomial it took 3.8 us of a call at 2^21 blocks, this takes about 2.5.)
__global__ void __launch_bounds__(512)
code_histogram_final_kernel(const uint32_t *__restrict__ partial, int n_partial, uint64_t nblk,
                            uint64_t *__restrict__ counts) {
  __shared__ uint64_t s[8];
  const int tid = threadIdx.x, k = blockIdx.x, m = tid >> 6, lane = tid & 63;
  if (m < HIST_MONO) {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(partial + (size_t)(m * 32 + k) * HIST_MAX_WG);
    u32x4 v[HIST_MAX_WG / 256];
#pragma unroll
    for (int i = 0; i < HIST_MAX_WG / 256; ++i)
      v[i] = (4 * lane + 256 * i < n_partial) ? src[lane + 64 * i] : u32x4{0, 0, 0, 0};
    uint64_t acc = 0;
#pragma unroll
    for (int i = 0; i < HIST_MAX_WG / 256; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc += (4 * lane + 256 * i + c < n_partial) ? v[i][c] : 0u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) acc += __shfl_xor((unsigned long long)acc, off);
    if (lane == 0) s[m] = acc;
  }
  __syncthreads();
  if (tid < 8) {
    const uint64_t s0 = s[0], s1 = s[1], s2 = s[2], s01 = s[3], s02 = s[4], s12 = s[5], s012 = s[6];
    uint64_t c;
    switch (tid) {   // codeword j = b0 + 2 b1 + 4 b2
      case 0: c = nblk - s0 - s1 - s2 + s01 + s02 + s12 - s012; break;
      case 1: c = s0 - s01 - s02 + s012; break;
      case 2: c = s1 - s01 - s12 + s012; break;
      case 3: c = s01 - s012; break;
      case 4: c = s2 - s02 - s12 + s012; break;
      case 5: c = s02 - s012; break;
      case 6: c = s12 - s012; break;
      default: c = s012; break;
    }
    counts[k * 8 + tid] = c;
  }
}

size_t code_histogram_workspace_bytes() { return (size_t)HIST_MAX_WG * HIST_PARTIAL * sizeof(uint32_t); }

// nblk >= 0 blocks of 16 bytes (none: all counts zero); counts: 256 uint64 on the device; workspace as above
hipError_t launch_code_histogram(const uint8_t *codes, int64_t nblk, uint64_t *counts, void *workspace,
                                 hipStream_t stream) {
  // a workgroup per 256 * 4 blocks (one group of loads per lane) while that leaves CUs free; beyond, all
  // the workgroups that can be resident at once, each with a longer span
  int64_t want = (nblk + (int64_t)HIST_THREADS * HIST_GROUP - 1) / ((int64_t)HIST_THREADS * HIST_GROUP);
  const int n_wg = (int)(want < 1 ? 1 : (want > HIST_MAX_WG ? HIST_MAX_WG : want));
  uint32_t *partial = static_cast<uint32_t *>(workspace);
  hipLaunchKernelGGL(code_histogram_kernel, dim3(n_wg), dim3(HIST_THREADS), 0, stream, codes, nblk, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(code_histogram_final_kernel, dim3(32), dim3(512), 0, stream, partial, n_wg, (uint64_t)nblk,
                     counts);
  return hipGetLastError();
}

}  // namespace torq
