// Host-side declarations shared by the translation units of libtorq.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/torq.h"

struct torq_rotation {
  int d;
  int G;
  int KS;            // ceil(G / 32): k-steps of the inter-block contraction
  int device;        // device the tables live on
  // R_inter as bf16 hi and lo parts, [G][KS*32] row-major, zero-padded columns
  uint16_t *inter_hi, *inter_lo;
  // the same values in the order in which the lanes of v_mfma_f32_32x32x16_bf16 take them as B operand,
  // [tile NW = ceil(G/32)][k-step 2 NW][lane 64][8], zero past G, so that a wave's load of one operand is
  // 1 KiB of consecutive bytes (from the row-major table it touches 32 cache lines)
  uint16_t *inter32f_hi, *inter32f_lo;
  // R_intra^T rows permuted for the accumulator layout, bf16 hi and lo, [32][32]
  uint16_t *intra_hi, *intra_lo;
  // the same matrix as the A operand of v_mfma_f32_32x32x16_bf16 (two k-steps), bf16 hi and lo
  uint16_t *intra32_hi, *intra32_lo;
  // optional: R_inter as a butterfly of plane rotations (rotate_butterfly.hip), the per-lane
  // coefficient table [butterfly_coef_count(G)][32]; nullptr for a dense R_inter
  float *butterfly;
  // DECODE_CTR_WORDS counters (zero between launches) on which torq_linear_single_launch synchronises
  // its rotating and its multiplying workgroups (mxfp4_gemm_skinny.hip)
  unsigned *decode_ctr;
};
constexpr int DECODE_CTR_WORDS = 32 * 131;
constexpr int DECODE_ERR = 32 * 130;      // the sticky "a workgroup gave up" word among them

namespace torq {

// What a kernel reads once and is larger than this is read with the non-temporal hint.  From HBM the hint is worth 8 % (117 MB
// into LDS at 7.4 TB/s against 6.8; the sc bits change nothing): such loads leave the 256 MB Infinity Cache alone.  What a
// program finds in that cache is read slower with it.
// Inputs (Gram, rotations) may have been written just before the call, or read by one, so the line lies where none of three
// ways of use loses by more than its runs differ (1 - 2 %), us without / with the hint, from HBM, one input again, and just written (with the writing):
//   Gram d = 8192: 134 MB 34.4 / 33.0, 30.2 / 32.3, 70.0 / 73.9; 180 MB 42.8 / 40.0, 37.1 / 39.0, 93.6 / 92.9; 235 MB 54.4 / 49.9,
//     45.2 / 50.9, 128.8 / 126.0; 262 MB 57.0 / 52.1, 51.5 / 51.1, 139.5 / 134.7; 512 MB 101 / 91, 100 / 89, 278 / 261
//   butterfly to MXFP4, G = 32 and G = 128: 134 MB 34.9 / 33.2, 30.7 / 34.2, 69.4 / 74.7 and 39.8 / 39.6, 37.7 / 40.1, 74.3 / 77.5;
//     220 MB 55.7 / 53.3, 48.9 / 53.3, 125 / 118 and 59.2 / 58.5, 57.4 / 58.1, 134 / 121; 250 MB 64.0 / 60.5, 61.2 / 59.8, 145 / 137
//     and 70.4 / 65.0, 66.8 / 65.2, 154 / 137; 512 MB 133 / 118, 134 / 116, 300 / 281 and 140 / 130, 139 / 127, 304 / 283
//   dense rotation to MXFP4, G = 128 and G = 80: 134 MB 50.3 / 51.5, 50.6 / 52.0, 84.7 / 86.4 and 48.2 / 49.2, 48.0 / 50.6, 91.2 / 91.3;
//     260 MB 90.6 / 88.9, 90.0 / 89.9, 172 / 166 and 89.6 / 88.6, 89.6 / 90.2, 181 / 181; 470 MB 159 / 157, 162 / 157, 303 / 294 and
//     160 / 156, 158 / 156, 321 / 323
constexpr double ONE_PASS_INPUT_BYTES = 240.0 * 1024 * 1024;
// In torq_linear the packed activations and the output come right behind, and the cache is better left to them: the line is where
// it would not hold all of it.  Whole calls without / with the hint, us, three layers in turn, one again, and in turn with the input
// just written, dense G = 128: [8192, 8192] x 28672 991 / 984, 991 / 985, 1041 / 1044, x 8192 332 / 327, 324 / 320, 373 / 370, x
// 1024 97.0 / 95.6, 91.7 / 94.1, 137.4 / 134.7; [12288, 8192] x 8192 477 / 477, 476 / 472, 542 / 538; butterfly G = 32 [8192, 8192] x
// 8192 323 / 315, 311 / 306, 364 / 352, x 1024 84.2 / 80.7, 75.2 / 81.5, 123.5 / 123.8; at 105 MB, [6400, 8192] x 8192, dense 278 /
// 278, 272 / 274, 310 / 308
constexpr double ONE_PASS_LINEAR_INPUT_BYTES = 96.0 * 1024 * 1024;
// Weights come round again when the program has read its other layers, so the way of use that counts is from HBM; a layer this
// large that is multiplied again at once loses.  us without / with, from HBM, then the same layer again: [16, 8192] 95 MB 22.2 /
// 20.2, 17.8 / 20.4, 128 MB 28.0 / 25.4, 24.2 / 25.3, 230 MB 46.3 / 43.1, 39.4 / 43.0, 300 MB 62.0 / 55.0, 59.1 / 55.0; [1, 8192]
// 128 MB 25.9 / 23.9, 23.7 / 23.5, 230 MB 43.2 / 40.2, 38.5 / 40.7; whole lines [16, 28672] 128 MB 34.7 / 33.0, 22.2 / 32.9, 230 MB
// 44.6 / 39.7, 36.8 / 38.9.  (From HBM layers of 4 to 70 MB would gain 3 - 10 % too; smaller models have theirs in the cache.)
constexpr double ONE_PASS_WEIGHT_BYTES = 96.0 * 1024 * 1024;

// Raises a kernel's dynamic LDS limit to `bytes`, once for each device it is launched on (the limit belongs to
// the function on one device, and the call is slow).  `raised`: the caller's, one per kernel, a bit a device;
// a failed call leaves the bit clear, so the next launch tries again.
inline hipError_t raise_lds_limit(const void *kernel, size_t bytes, std::atomic<uint64_t> &raised) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (raised.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) raised.fetch_or(bit, std::memory_order_release);
  return e;
}

// fp32 rows -> a 4-bit block format (FMT_* of torq_device.h = TORQ_FMT_* of torq.h).  nblk = number
// of 32-element blocks (M * d / 32); global_scale is NVFP4's tensor-wide scale, else ignored.
hipError_t launch_quantize_f32(const float *z, int64_t nblk, int format, float global_scale, uint8_t *codes,
                               uint8_t *scales, hipStream_t stream);

// Two-level rotation (+ quantisation).  Exactly one of (codes, scales) / z_out is used:
// z_out != nullptr writes the rotated fp32 values instead of quantising to `format`.  once: an input that is read past the
// cache (where the kernel has a form for it).
hipError_t launch_rotate(const torq_rotation *r, const void *x_bf16, int64_t M, int format, float global_scale,
                         uint8_t *codes, uint8_t *scales, float *z_out, bool once, hipStream_t stream);

// The same for a handle whose R_inter is a butterfly (r->butterfly != nullptr; G in 32, 64, 128, 256).
int butterfly_coef_count(int G);
hipError_t launch_rotate_butterfly(const torq_rotation *r, const void *x_bf16, int64_t M, int format,
                                   float global_scale, uint8_t *codes, uint8_t *scales, float *z_out, bool once,
                                   hipStream_t stream);

// workspace: optional device scratch of mxfp4_gemm_workspace_bytes(M, N, d) bytes; with it, shapes
// with few output tiles and a long reduction are cut along k (fp32 pieces added in a fixed order).
size_t mxfp4_gemm_workspace_bytes(int64_t M, int64_t N, int d);
// what launch_mxfp4_gemm would do with a workspace of that size (operands assumed 16-byte aligned)
void mxfp4_gemm_plan(int64_t M, int64_t N, int d, size_t workspace_bytes, int *skinny, int *tile_m, int *tile_n,
                     int *splits);
// torq_diag_gemm_form: the form behind the plan
void mxfp4_gemm_form(int64_t M, int64_t N, int d, size_t workspace_bytes, int *staging, int *strips, int *items, int *padded);
// The tiled kernel with its operands staged in a ring (mxfp4_gemm_ring.hip): tiles 128x128, 128x64, 64x128 and 64x64,
// d a multiple of 512, scale arrays 16-byte aligned.  splits > 1: the pieces' fp32 sums go to partial[splits][M][N] and out is not
// written.  d / 512 divisible by splits.
hipError_t launch_mxfp4_gemm_ring(int tile_m, int tile_n, const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q,
                                  const uint8_t *W_s, void *out, float *partial, int splits, int64_t M, int64_t N, int d,
                                  int64_t ldc, hipStream_t stream);
hipError_t launch_mxfp4_gemm_ring_forced(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                                         void *out_bf16, int64_t M, int64_t N, int d, int tile_m, int tile_n, int k_pieces,
                                         void *workspace, size_t workspace_bytes, hipStream_t stream);
// the tiled kernel on a given plan: tile 0 ... 3 = 256x256, 256x128, 128x128, 128x64 (always in a ring); k_pieces > 1 needs the workspace (k_pieces * M * N floats) and d / 512 divisible by it; deep: tile 2's deeper load
// pipeline where it is not cut
hipError_t launch_mxfp4_gemm_forced(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                                    void *out_bf16, int64_t M, int64_t N, int d, int tile, int k_pieces, int deep,
                                    void *workspace, size_t workspace_bytes, hipStream_t stream);
// N, or the leading output columns that a first launch of whole rounds of 256 x 256 tiles takes (the plan
// above is then that launch's; the remaining columns are a product of their own with its own plan)
int64_t mxfp4_gemm_main_columns(int64_t M, int64_t N, int d, size_t workspace_bytes);
hipError_t launch_mxfp4_gemm(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q,
                             const uint8_t *W_s, void *out_bf16, int64_t M, int64_t N, int d,
                             void *workspace, size_t workspace_bytes, hipStream_t stream);

// The same product for 1 <= M <= 64 (weight-streaming layout); called by launch_mxfp4_gemm when
// mxfp4_gemm_skinny_fits (the scale rows it stages fit the LDS).
int mxfp4_gemm_skinny_strips(int64_t M, int64_t N, int d);   // 16-row weight strips per workgroup
int mxfp4_gemm_lines_strips(int64_t M, int64_t N, int d);    // the same of its whole-line form, 0: not taken
bool mxfp4_gemm_lines_form(int64_t M, int64_t N, int d, int *strips, int *items, int *padded);
bool mxfp4_gemm_skinny_fits(int64_t M, int d);
hipError_t launch_mxfp4_gemm_skinny(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q,
                                    const uint8_t *W_s, void *out_bf16, int64_t M, int64_t N, int d,
                                    hipStream_t stream);
// The same product for wide layers, strip after strip through a ring (mxfp4_gemm_stream.hip): where it is taken, how many
// strips a workgroup has under way at a time, and the launch (scale arrays 16-byte aligned).
bool mxfp4_gemm_stream_takes(int64_t M, int64_t N, int d);
int mxfp4_gemm_stream_strips(int d);
hipError_t launch_mxfp4_gemm_stream(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out_bf16,
                                    int64_t M, int64_t N, int d, hipStream_t stream);
// torq_linear for at most 64 rows in one launch: rotate + quantise (the 16-block body, G = 128) in the
// first workgroups of the weight-streaming GEMM.  Preconditions: r->G == 128, dense R_inter,
// 1 <= M <= 64, mxfp4_gemm_skinny_fits(M, r->d); A_q / A_s are the workspace's code and scale areas.
// spin_limit: polls before a waiting workgroup gives up; raise_ready = 0 withholds the hand-off
// (test of the give-up path: every workgroup still exits).
hipError_t launch_torq_linear_decode(const torq_rotation *r, const void *x_bf16, uint8_t *A_q, uint8_t *A_s,
                                     const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M, int64_t N,
                                     int spin_limit, int raise_ready, hipStream_t stream);
// torq_linear for a few token-groups with rotate + quantise inside every workgroup of the GEMM's launch
// (no hand-off between workgroups, the packed activations stay in LDS; workgroup 0 leaves a copy in
// A_q / A_s).  torq_linear_local_fits: dense R_inter, G = 112 or 128, at most four token-groups.
bool torq_linear_local_fits(const torq_rotation *r, int64_t M);
// ... and is measured faster than the two launches (what torq_linear itself then does)
bool torq_linear_local_pays(const torq_rotation *r, int64_t M, int64_t N, const uint8_t *W_s);
hipError_t launch_torq_linear_local(const torq_rotation *r, const void *x_bf16, uint8_t *A_q, uint8_t *A_s,
                                    const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M, int64_t N,
                                    hipStream_t stream);
// The same with the weight strips one after the other through a ring (mxfp4_gemm_stream.hip): where it takes the place of
// the form above (its preconditions among them), and the launch.
bool torq_linear_stream_takes(const torq_rotation *r, int64_t M, int64_t N, const uint8_t *W_s);
hipError_t launch_torq_linear_stream(const torq_rotation *r, const void *x_bf16, uint8_t *A_q, uint8_t *A_s, const uint8_t *W_q,
                                     const uint8_t *W_s, void *out_bf16, int64_t M, int64_t N, hipStream_t stream);
// all of the handle's counters back to zero, the sticky error word included
hipError_t launch_decode_ctr_reset(const torq_rotation *r, hipStream_t stream);

// Block Gram matrix of the runs of G blocks (block_gram.hip), or the 32 of them kept apart by position:
// TG token-groups of G * 32 bf16 each.
size_t block_gram_workspace_bytes(int G);
size_t block_gram_workspace_least(int G);   // accepted, at the price of speed
hipError_t launch_block_gram(const void *x_bf16, int64_t TG, int G, bool positions, double *Sigma, void *workspace,
                             size_t workspace_bytes, hipStream_t stream);

// Codeword histogram per in-block position (code_histogram.hip): nblk blocks of 16 code bytes.
size_t code_histogram_workspace_bytes();
hipError_t launch_code_histogram(const uint8_t *codes, int64_t nblk, uint64_t *counts, void *workspace,
                                 hipStream_t stream);

// Host side of the intra-block calibration (intra_calib.hip).
void intra_pair_scores(const uint64_t *counts, double lambda, double *h, double *H);
int64_t intra_best_angle(const double *u, const double *v, int64_t n, const uint64_t rest[8], double *theta,
                         double *loss);
void intra_rotation(const float *X, int64_t n, int max_iter, int k_top, int P, double lambda, double eps,
                    double *R_out, double *losses, int *n_eval);

// 1024 x 256 lanes issue iters x 16 MFMAs each on operands taken from `words` (see diag.hip).
hipError_t launch_mfma_burn(int kind, const uint32_t *words, uint32_t n_words, int iters, float *sink,
                            hipStream_t stream);

// The two headline kernels with parts of their work left out (SKIP bits documented at the kernels):
// what each part costs in time on this machine.  Outputs are meaningless by design.
hipError_t launch_mxfp4_gemm_ablated(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                                     void *out_bf16, int64_t M, int64_t N, int d, int skip, hipStream_t stream);
// the persistent form of the tiled GEMM (tile 0: 256 x 256, 1: 256 x 128) on `workgroups` workgroups
hipError_t launch_mxfp4_gemm_persistent(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                                        void *out_bf16, int64_t M, int64_t N, int d, int tile, int workgroups,
                                        hipStream_t stream);
hipError_t launch_rotate_ablated(const torq_rotation *r, const void *x, int64_t M, uint8_t *codes, uint8_t *scales,
                                 int skip, hipStream_t stream);
// plain copy of `bytes` (a multiple of 16) device bytes, the traffic counters' yardstick (diag.hip)
hipError_t launch_diag_copy(const void *src, void *dst, size_t bytes, hipStream_t stream);

}  // namespace torq
