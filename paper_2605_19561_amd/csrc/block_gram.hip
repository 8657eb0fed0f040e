// torq_block_gram / torq_block_gram_positions: the statistics that the inter-block calibration starts
// from (Section 5.1, Algorithm 1 input; Section 4.2, sigma_b^2 = E ||z_b||^2 and the Sigma_k of Theorem 4.1):
//
//   Sigma[b][b']    = mean over token-groups of  sum_k X[b][k] X[b'][k]
//   Sigma_k[b][b']  = mean over token-groups of  X[b][k] X[b'][k]
//
// where a token-group is one run of G consecutive 32-element blocks of one row, i.e. G rows of
// 64 contiguous bytes.  Both are products of a matrix with its own transpose on the matrix cores, of which
// only the 16 x 16 tiles (r, c) with r <= c are computed; the reduce kernel writes both triangles.
//
// Sigma: the contraction index is the position inside a block (K = 32 = one instruction), the operand
//   of tile row r is 16 block rows x 64 bytes = 1 KiB of consecutive input.  Two forms, both one pass
//   over the input: waves that work alone, and waves that share each token-group through LDS.
//   bf16 products are exact in fp32; the sums are fp32 along a chain of instructions and double across them.
// Sigma_k: the contraction index is the token-group; the workgroup transposes its input on the way
//   into LDS (below).  The sums are double throughout.
//
// Partial sums: packed tiles, [tile][lane][4 floats or doubles] as the accumulators hold them.
#include "torq_device.h"
#include "torq_internal.h"

namespace torq {

typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

constexpr int GRAM_WAVES = 8;
constexpr int GRAM_MAX_WG = 256;      // Sigma, waves alone: one workgroup per CU
constexpr int GRAM_MAX_TILES = 36;    // ... and 144 accumulator registers
constexpr int GRAM_SHARED_WG = 512;   // Sigma, shared token-groups: two workgroups per CU
constexpr int GRAM_SHARED_U = 2;      // ... and token-groups per trip
constexpr int GRAM_POS_TILES = 9;     // Sigma_k: tiles of a wave, 72 registers

// the tiles (r, c), r <= c < NT, row by row
template <int NT>
struct GramTiles {
  static constexpr int N = NT * (NT + 1) / 2;
  int r[N] = {}, c[N] = {};
  constexpr GramTiles() {
    int i = 0;
    for (int a = 0; a < NT; ++a)
      for (int b = a; b < NT; ++b) {
        r[i] = a;
        c[i] = b;
        ++i;
      }
  }
};

// how many of a wave's tiles go through LDS at once when the waves of a workgroup add theirs
constexpr int gram_box_tiles(int tiles) { return tiles * GRAM_WAVES <= 144 ? tiles : (tiles + 1) / 2; }

// tile number i of the triangle -> its row; i becomes its place in that row (column - row)
__device__ __forceinline__ int gram_tile_row(int nt, int &i) {
  int r = 0;
  while (i >= nt - r) i -= nt - r++;
  return r;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gram_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// Sigma, G <= 128.  Bound: HBM, 2 bytes per element, read once.  Every wave takes token-groups of its own (U at a
// time, about 8 KiB), straight from memory into the operand registers: nothing is staged or shared, there
// is no barrier in the loop, and two steps are in flight beyond the one being multiplied (128 KiB per CU).
// A token-group past the end reads as zeros through the buffer's range check and adds nothing.  The
// workgroup's waves add their tiles at the end: 256 partial results instead of the 512 of the form that
// shares each token-group.  X [16384, 8192], G = 128: this kernel 51 us against 64 (5.2 TB/s, the rate of a copy).
// ONCE: loads with the non-temporal hint (ONE_PASS_INPUT_BYTES), X [16384, 8192] 55.4 -> 50.5 us with the reduction.
template <int NT, bool ONCE>
__global__ void __launch_bounds__(64 * GRAM_WAVES)
block_gram_kernel(const uint4 *__restrict__ x, int64_t TG, f32x4 *__restrict__ partial) {
  constexpr GramTiles<NT> tiles;
  constexpr int G = 16 * NT, COUNT = GramTiles<NT>::N, U = NT < 8 ? 8 / NT : 1;
  extern __shared__ __attribute__((aligned(16))) char lds[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int voff = (lane & 15) * 64 + (lane >> 4) * 16;
  // the workgroup's steps are one contiguous span, dealt to its waves in turn
  const int64_t steps = (TG + U - 1) / U;
  const int64_t per = (steps + gridDim.x - 1) / gridDim.x;
  const int64_t s_end = (int64_t)(blockIdx.x + 1) * per < steps ? (int64_t)(blockIdx.x + 1) * per : steps;

  f32x4 acc[COUNT];
#pragma unroll
  for (int i = 0; i < COUNT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto load = [&](u32x4 (&v)[U][NT], int64_t s) {
    const int64_t left = s < s_end ? TG - s * U : 0;
    const __amdgpu_buffer_rsrc_t rsrc =
        gram_rsrc(x + (left > 0 ? s * U : 0) * (4 * G), (uint32_t)(left < U ? left : U) * (G * 64));
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int f = 0; f < NT; ++f)
        v[u][f] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, u * (G * 64) + f * 1024, LOAD_POLICY<ONCE>);
  };
  auto multiply = [&](const u32x4 (&v)[U][NT]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < COUNT; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, v[u][tiles.r[i]]),
            __builtin_bit_cast(bf16x8, v[u][tiles.c[i]]), acc[i], 0, 0, 0);
  };

  u32x4 v[3][U][NT];
  int64_t s = (int64_t)blockIdx.x * per + wave;
  load(v[0], s);
  load(v[1], s + GRAM_WAVES);
  for (; s < s_end; s += 3 * GRAM_WAVES) {
    load(v[2], s + 2 * GRAM_WAVES);
    multiply(v[0]);
    load(v[0], s + 3 * GRAM_WAVES);
    multiply(v[1]);
    load(v[1], s + 4 * GRAM_WAVES);
    multiply(v[2]);
  }

  // The waves' tiles meet in LDS, half of them at a time where they do not all fit, and are added in double: one
  // rounding to fp32 for each partial sum, so that it is the waves' chains alone that round.
  constexpr int BATCH = gram_box_tiles(COUNT);
  f32x4 *const box = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
  for (int t0 = 0; t0 < COUNT; t0 += BATCH) {
    constexpr int THR = 64 * GRAM_WAVES;
    if (t0) __syncthreads();
#pragma unroll
    for (int i = t0; i < t0 + BATCH && i < COUNT; ++i) box[(wave * BATCH + i - t0) * 64 + lane] = acc[i];
    __syncthreads();
    const int quads = (COUNT - t0 < BATCH ? COUNT - t0 : BATCH) * 64;
    for (int i = threadIdx.x; i < quads; i += THR) {
      double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int w = 0; w < GRAM_WAVES; ++w) {
        const f32x4 v = box[w * BATCH * 64 + i];
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += (double)v[e];
      }
      partial[((size_t)blockIdx.x * COUNT + t0) * 64 + i] = f32x4{(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
    }
  }
}

// Sigma for short inputs and for G > 128, where one wave's registers do not hold the tiles and splitting them over
// launches reads the input once for each (two launches at G = 144 to five at 256).  The workgroup shares each
// token-group through LDS: wave w owns the block rows 32 w .. 32 w + 31 (two tile rows) against all NT columns, trips of two
// token-groups go global -> registers -> LDS with two stages and one barrier a trip.  Workgroups are
// persistent, two per CU; only the tiles of the triangle are written.  Bound: HBM, read once.  X [16384, 8192],
// G = 256, with the reduction: 98 us against 208 in five launches; G = 160 (X [16384, 5120]): 44 against 65.
template <int NT>
__global__ void __launch_bounds__(64 * ((NT + 1) / 2))
block_gram_shared_kernel(const uint4 *__restrict__ x, int64_t TG, f32x4 *__restrict__ partial) {
  constexpr int G = 16 * NT, NTHR = 64 * ((NT + 1) / 2), U = GRAM_SHARED_U;
  constexpr int CHUNKS = 4 * G;                          // 16-byte chunks of one token-group
  constexpr int CH = (CHUNKS + NTHR - 1) / NTHR;         // chunks per thread per token-group (2)
  constexpr int TG_BYTES = G * 64, STAGE_BYTES = U * TG_BYTES;
  __shared__ __attribute__((aligned(16))) char lds[2 * STAGE_BYTES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, q = lane >> 4;
  const int rt0 = 2 * wave, rt1 = 2 * wave + 1;          // this wave's tile rows; rt1 may not exist
  const bool has1 = rt1 < NT;

  f32x4 acc0[NT], acc1[NT];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) acc0[ct] = acc1[ct] = f32x4{0.f, 0.f, 0.f, 0.f};

  // chunk c of a token-group = (block row c / 4, elements 8 (c % 4) .. + 7).  In LDS the chunk index inside a
  // 64-byte row is XORed with (row >> 2) & 3, so that the 16 lanes that read one operand (16 consecutive rows,
  // same chunk) hit 16 different bank groups; for a tile's rows 16 t + m that term is (m >> 2) & 3
  const int frag_off = m * 64 + ((q ^ ((m >> 2) & 3)) * 16);
  int st_off[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = tid + i * NTHR, r = c >> 2;
    st_off[i] = r * 64 + (((c & 3) ^ ((r >> 2) & 3)) * 16);
  }

  const int64_t ntrip = (TG + U - 1) / U;                // dealt to the workgroups round robin
  uint4 regs[U][CH];
  auto load_trip = [&](int64_t trip) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int c = tid + i * NTHR;
        regs[u][i] = (trip * U + u < TG && c < CHUNKS) ? x[(trip * U + u) * CHUNKS + c] : make_uint4(0, 0, 0, 0);
      }
  };
  auto store_trip = [&](int stage) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < CH; ++i)
        if (tid + i * NTHR < CHUNKS)
          *reinterpret_cast<uint4 *>(lds + stage * STAGE_BYTES + u * TG_BYTES + st_off[i]) = regs[u][i];
  };

  int64_t trip = blockIdx.x;
  if (trip < ntrip) {
    load_trip(trip);
    store_trip(0);
  }
  __syncthreads();
  int stage = 0;
  for (; trip < ntrip; trip += gridDim.x, stage ^= 1) {
    const int64_t next = trip + gridDim.x;
    const bool have_next = next < ntrip;
    if (have_next) load_trip(next);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const char *g = lds + stage * STAGE_BYTES + u * TG_BYTES + frag_off;
      const bf16x8 a0 = *reinterpret_cast<const bf16x8 *>(g + rt0 * 1024);
      const bf16x8 a1 = *reinterpret_cast<const bf16x8 *>(g + (has1 ? rt1 : rt0) * 1024);
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) {
        const bf16x8 col = *reinterpret_cast<const bf16x8 *>(g + ct * 1024);
        acc0[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, col, acc0[ct], 0, 0, 0);
        acc1[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, col, acc1[ct], 0, 0, 0);
      }
    }
    if (have_next) store_trip(stage ^ 1);
    __syncthreads();
  }

  f32x4 *const out = partial + (size_t)blockIdx.x * (GramTiles<NT>::N * 64) + lane;
  const int row0 = rt0 * NT - rt0 * (rt0 - 1) / 2 - rt0, row1 = rt1 * NT - rt1 * (rt1 - 1) / 2 - rt1;
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    if (ct >= rt0) out[(row0 + ct) * 64] = acc0[ct];
    if (has1 && ct >= rt1) out[(row1 + ct) * 64] = acc1[ct];
  }
}

// Sigma_k: how a launch is cut.  256 or 512 workgroups of nearly equal work (four chunks x parts x slices) for at
// most GRAM_POS_TILES tiles a part; the slices are a multiple of the XCDs.
constexpr int gram_pos_parts(int nt) {
  const int tiles = nt * (nt + 1) / 2, fit = (tiles + GRAM_POS_TILES - 1) / GRAM_POS_TILES;
  return fit > 8 ? 16 : fit > 4 ? 8 : tiles < 4 ? tiles : 4;
}
constexpr int gram_pos_slices(int nt) { return nt == 1 ? 64 : gram_pos_parts(nt) <= 4 ? 16 : 8; }

// The tiles of part PART of gram_pos_parts(NT).  A wave widens the operands of its tiles' rows and columns once a step, so a
// part's tiles are to share them: the parts are consecutive runs of the triangle gone through by blocks of 2 x 2 tiles, down
// the columns of each (NT = 8: 22 operands for the 36 tiles of four parts; by rows 25, by blocks of 3 x 3 26, each tile its
// own 72).
template <int NT, int PART>
struct GramPart {
  static constexpr int TILES = NT * (NT + 1) / 2, PARTS = gram_pos_parts(NT);
  static constexpr int FIRST = TILES * PART / PARTS, COUNT = TILES * (PART + 1) / PARTS - FIRST;
  int operands = 0;
  int row[2 * GRAM_POS_TILES] = {};                             // operand -> tile row of the block rows
  int a[GRAM_POS_TILES] = {}, b[GRAM_POS_TILES] = {};           // tile -> its operands
  int place[GRAM_POS_TILES] = {};                               // tile -> its number in the triangle, row by row
  constexpr int operand(int r) {
    for (int o = 0; o < operands; ++o)
      if (row[o] == r) return o;
    row[operands] = r;
    return operands++;
  }
  constexpr GramPart() {
    int i = 0;
    for (int r0 = 0; r0 < NT; r0 += 2)
      for (int c0 = r0; c0 < NT; c0 += 2)
        for (int c = c0; c < NT && c < c0 + 2; ++c)
          for (int r = r0; r < NT && r < r0 + 2; ++r) {
            if (r > c) continue;
            if (i >= FIRST && i < FIRST + COUNT) {
              a[i - FIRST] = operand(r);
              b[i - FIRST] = operand(c);
              place[i - FIRST] = r * NT - r * (r - 1) / 2 + c - r;
            }
            ++i;
          }
  }
};

// Sigma_k, all 32 positions in one pass.  A workgroup takes the eight positions of one 16-byte chunk of
// every block, a slice of the token-groups and a part of the tiles; the workgroups of a slice share the
// input's lines through the L2 of the XCD that all of them are on.  Wave j owns position 8 chunk + j.  The
// contraction runs over token-groups, so an operand register holds one position of one block row for eight
// of them: a thread loads its block's chunk of eight token-groups, pairs up their halves with byte
// permutes and writes one 16-byte operand piece for each position to LDS, [position][octet][block row],
// which is written and read in whole consecutive runs (no bank conflicts).  A stage holds KST steps of 32
// token-groups so that the 512 threads have one chunk column each.
//
// v_mfma_f64_16x16x4_f64, eight of them for 32 token-groups: the four k of an instruction are the four octets
// (any order of the token-groups will do, as long as both operands have the same).  Products and sums are double:
// bf16 instructions round 32 products at a time to 24 bits and lose the small ones beside an outlier, 5.5e-8 against
// 2.1e-8 relative for sums of one product after the other (activations with outlier channels, X [8192, 8192],
// G = 128), and still 2.5e-8 with eight products a sum, added up in double.  Bound: the matrix cores at the double rate,
// an instruction in 64 cycles, and no vector instruction runs beside it, so every conversion is paid for.  Each tile's
// operands widened for it alone / those of a part's rows once for all its tiles, with the reduction: X [4096, 4096], G = 128,
// 68.2 / 58.5 us (31 are the products; 7.5 the reduction; the first loads, the transposition and the stores are the rest),
// [2048, 14336], G = 112, 92.5 / 77.8, [1024, 8192], G = 256, 100 / 85.  Eight parts and eight slices at G = 128 take 66 (each
// part reads the lines from the L2 and widens again).
template <int NT, int PART>
__device__ __forceinline__ void gram_positions_part(const uint4 *__restrict__ x, int64_t TG, int chunk, int slice, int slices,
                                                    f64x4 *__restrict__ partial, char *lds) {
  constexpr GramPart<NT, PART> part;
  constexpr int COUNT = GramPart<NT, PART>::COUNT;
  constexpr int G = 16 * NT, TILES = NT * (NT + 1) / 2;
  constexpr int KST = NT < 8 ? 8 / NT : 1;          // steps of 32 token-groups per stage
  constexpr int ITEMS = 4 * KST * G;                // (octet of token-groups, block row)
  constexpr int THR = 64 * GRAM_WAVES, IT = (ITEMS + THR - 1) / THR;
  constexpr int PLANE = ITEMS * 16, STAGE = 8 * PLANE;
  constexpr bool TWO = 2 * STAGE <= 128 * 1024;     // two LDS stages, one barrier per stage

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t stages = (TG + 32 * KST - 1) / (32 * KST);
  const int64_t st0 = stages * slice / slices, st1 = stages * (slice + 1) / slices;

  int voff[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int item = tid + i * THR;
    voff[i] = item < ITEMS ? ((item / G) * 8 * G + item % G) * 64 + chunk * 16 : 0x7FFFFFF0;
  }
  u32x4 v[IT][8];
  auto load = [&](int64_t st) {                     // a token-group past the end reads as zeros
    const int64_t tg0 = st * (32 * KST), left = TG - tg0 < 32 * KST ? TG - tg0 : 32 * KST;
    const __amdgpu_buffer_rsrc_t rsrc = gram_rsrc(x + tg0 * (4 * G), (uint32_t)left * (G * 64));
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int t = 0; t < 8; ++t) v[i][t] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff[i], t * (G * 64), 0);
  };
  auto store = [&](char *stage) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (ITEMS % THR != 0 && tid + i * THR >= ITEMS) continue;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        u32x4 even, odd;                            // positions 2 w and 2 w + 1 of the chunk
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          even[p] = __builtin_amdgcn_perm(v[i][2 * p + 1][w], v[i][2 * p][w], 0x05040100u);
          odd[p] = __builtin_amdgcn_perm(v[i][2 * p + 1][w], v[i][2 * p][w], 0x07060302u);
        }
        *reinterpret_cast<u32x4 *>(stage + (2 * w) * PLANE + (tid + i * THR) * 16) = even;
        *reinterpret_cast<u32x4 *>(stage + (2 * w + 1) * PLANE + (tid + i * THR) * 16) = odd;
      }
    }
  };

  f64x4 acc[COUNT];
#pragma unroll
  for (int i = 0; i < COUNT; ++i) acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};

  const int f_off = wave * PLANE + ((lane >> 4) * G + (lane & 15)) * 16;
  if (st0 < st1) load(st0);
  int buf = 0;
  for (int64_t st = st0; st < st1; ++st) {
    char *const stage = lds + (TWO ? buf * STAGE : 0);
    store(stage);
    if (st + 1 < st1) load(st + 1);
    __syncthreads();
#pragma unroll 1
    for (int ks = 0; ks < KST; ++ks) {
      const char *const f = stage + f_off + ks * (4 * G * 16);
      u32x4 v[part.operands];
#pragma unroll
      for (int o = 0; o < part.operands; ++o) v[o] = *reinterpret_cast<const u32x4 *>(f + part.row[o] * 256);
#pragma unroll
      for (int h = 0; h < 8; ++h) {                 // token-groups h of the octets
        double wide[part.operands];
#pragma unroll
        for (int o = 0; o < part.operands; ++o)
          wide[o] = (double)__builtin_bit_cast(float, h & 1 ? v[o][h / 2] & 0xFFFF0000u : v[o][h / 2] << 16);
#pragma unroll
        for (int i = 0; i < COUNT; ++i)
          acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(wide[part.a[i]], wide[part.b[i]], acc[i], 0, 0, 0);
      }
    }
    if (!TWO) __syncthreads();
    buf ^= 1;
  }
  f64x4 *const out = partial + ((size_t)slice * 32 + chunk * 8 + wave) * TILES * 64 + lane;
#pragma unroll
  for (int i = 0; i < COUNT; ++i) out[part.place[i] * 64] = acc[i];
}

template <int NT>
__global__ void __launch_bounds__(64 * GRAM_WAVES)
block_gram_positions_kernel(const uint4 *__restrict__ x, int64_t TG, int slices, f64x4 *__restrict__ partial) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int PARTS = gram_pos_parts(NT);
  // workgroup id mod 8 is the XCD: the chunks and parts of a slice share one
  const int id = blockIdx.x, units = 4 * PARTS, unit = (id >> 3) % units, chunk = unit & 3, part = unit >> 2;
  const int slice = (id >> 3) / units * 8 + (id & 7);
  if (slice >= slices) return;
  static_for<PARTS>([&](auto p) {                   // (uniform: one branch taken)
    if (part == p) gram_positions_part<NT, decltype(p)::value>(x, TG, chunk, slice, slices, partial, lds);
  });
}

// Adds n partial results in double and in a fixed order, divides by the number of token-groups and writes
// both triangles.  A workgroup adds QUADS accumulator quads: thread (slice = t / QUADS, quad = t % QUADS) every
// SLICES-th partial, then the slices meet in LDS.  Sigma: 16 quads, so that its few tiles make four times as
// many workgroups, and 16 slices for 256 or 512 partials; Sigma_k: whole tiles, at most 64 partials.
// blockIdx.y: the position (1 or 32 of them); a partial result holds gridDim.y * tiles * 64 quads.
// A lane's quad: column lane % 16, and four rows of the tile: 4 (lane / 16) + e of a 32-bit accumulator,
// lane / 16 + 4 e of a 64-bit one.
template <typename Quad, int QUADS>
__global__ void __launch_bounds__(256)
block_gram_reduce_kernel(const Quad *__restrict__ partial, int n, int nt, double inv_groups, double *__restrict__ Sigma) {
  constexpr int SLICES = 256 / QUADS, PER_TILE = 64 / QUADS;
  constexpr bool F64_ROWS = sizeof(Quad) == 32;
  static_assert(QUADS == (F64_ROWS ? 64 : 16), "the transposed store's rows");
  const int G = 16 * nt;
  __shared__ double part[SLICES][QUADS][4];
  __shared__ double sum[QUADS][4];
  const int t = threadIdx.x, quad = t % QUADS, slice = t / QUADS;
  const size_t per_position = (size_t)gridDim.x * QUADS, stride = gridDim.y * per_position;
  const Quad *src = partial + blockIdx.y * per_position + blockIdx.x * QUADS + quad;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  constexpr int FLY = QUADS == 16 ? 8 : 4;          // loads in flight, added in order
  int p = slice;
  for (; p + (FLY - 1) * SLICES < n; p += FLY * SLICES) {
    Quad q[FLY];
#pragma unroll
    for (int u = 0; u < FLY; ++u) q[u] = src[(size_t)(p + SLICES * u) * stride];
#pragma unroll
    for (int u = 0; u < FLY; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += (double)q[u][e];
  }
  for (; p < n; p += SLICES) {
    const Quad q = src[(size_t)p * stride];
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += (double)q[e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[slice][quad][e] = s[e];
  __syncthreads();
  int place = blockIdx.x / PER_TILE;
  const int tile_row = gram_tile_row(nt, place), lane0 = blockIdx.x % PER_TILE * QUADS;
  const int r = tile_row * 16, c = (tile_row + place) * 16;
  auto row = [&](int lane, int e) { return F64_ROWS ? lane / 16 + 4 * e : lane / 16 * 4 + e; };
  double *const out = Sigma + (size_t)blockIdx.y * G * G;
  if (t < 4 * QUADS) {
    const int e = t / QUADS;
    double total = 0.0;
#pragma unroll
    for (int i = 0; i < SLICES; ++i) total += part[i][quad][e];
    total *= inv_groups;
    sum[quad][e] = total;
    out[(size_t)(r + row(lane0 + quad, e)) * G + c + (quad & 15)] = total;
  }
  __syncthreads();
  // the other triangle, along its rows: column j of the tile, the workgroup's rows of it
  if (t < 4 * QUADS && place != 0) {
    const int j = t / (QUADS / 4), i = t % (QUADS / 4);              // QUADS / 4 rows of the tile
    const int q = F64_ROWS ? (i & 3) * 16 + j : (i >> 2) * 16 + j, e = F64_ROWS ? i >> 2 : i & 3;
    out[(size_t)(c + j) * G + r + row(lane0 + q, e)] = sum[q][e];
  }
}

// the larger of the two statistics' partial results: Sigma_k's slices of 32 positions, Sigma's workgroups
size_t block_gram_workspace_bytes(int G) {
  const int nt = G / 16;
  const size_t tiles = (size_t)nt * (nt + 1) / 2;
  const size_t pos = (size_t)gram_pos_slices(nt) * 32 * tiles * 2048, sigma = (size_t)GRAM_SHARED_WG * tiles * 1024;
  return pos > sigma ? pos : sigma;
}

// The least that is accepted: what earlier sizes of this scratch came to, for programs that keep one.  A launch then
// has fewer slices or workgroups (X [4096, 4096], G = 128: 15 slices instead of 16).
size_t block_gram_workspace_least(int G) {
  const size_t earlier = G <= 128 ? (size_t)2176 * G * G : (size_t)23 << 20, now = block_gram_workspace_bytes(G);
  return earlier < now ? earlier : now;
}

template <typename Quad, int QUADS>
static hipError_t launch_reduce(const Quad *partial, int n, int nt, int positions, int64_t TG, double *Sigma, hipStream_t stream) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((block_gram_reduce_kernel<Quad, QUADS>), dim3(nt * (nt + 1) / 2 * (64 / QUADS), positions), dim3(256), 0, stream,
                     partial, n, nt, 1.0 / (double)TG, Sigma);
  return hipGetLastError();
}

template <int NT>
static hipError_t launch_sigma(const uint4 *x, int64_t TG, double *Sigma, void *workspace, size_t workspace_bytes,
                               hipStream_t stream) {
  f32x4 *const partial = static_cast<f32x4 *>(workspace);
  constexpr int TILES = GramTiles<NT>::N;
  if constexpr (TILES <= GRAM_MAX_TILES) {
    // Waves alone where each wave of 256 workgroups has a step.  Shorter inputs take the other form, which spreads them
    // over up to 512 partial sums: with fewer workgroups than CUs this one is further from the sum in 64 bits, 1.8
    // times at X [512, 4096], G = 128, and seven times at [512, 1024], G = 32, of Gaussian values.  us, this form
    // against the other: [64, 4096] 11.5 / 6.7, [4096, 512] 9.3 / 7.3, [1024, 4096] 13.9 / 17.4 (the price of the
    // smaller error), [2048, 4096] 15.1 / 17.8, [16384, 512] 9.1 / 12.7.
    constexpr int U = NT < 8 ? 8 / NT : 1;
    if (TG / U >= GRAM_WAVES * GRAM_MAX_WG) {
      constexpr size_t lds = (size_t)GRAM_WAVES * gram_box_tiles(TILES) * 1024;
      auto go = [&](auto kernel, std::atomic<uint64_t> &raised) {
        if constexpr (lds > 64 * 1024) {
          const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(kernel), lds, raised);
          if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3(GRAM_MAX_WG), dim3(64 * GRAM_WAVES), lds, stream, x, TG, partial);
        return hipSuccess;
      };
      static std::atomic<uint64_t> raised[2];
      const hipError_t e = (double)TG * (1024.0 * NT) > ONE_PASS_INPUT_BYTES ? go(block_gram_kernel<NT, true>, raised[1])
                                                                       : go(block_gram_kernel<NT, false>, raised[0]);
      if (e != hipSuccess) return e;
      return launch_reduce<f32x4, 16>(partial, GRAM_MAX_WG, NT, 1, TG, Sigma, stream);
    }
  }
  const int64_t trips = (TG + GRAM_SHARED_U - 1) / GRAM_SHARED_U;
  const int64_t room = (int64_t)(workspace_bytes / ((size_t)TILES * 1024)), most = room < GRAM_SHARED_WG ? room : GRAM_SHARED_WG;
  const int n = (int)(trips < most ? trips : most);
  hipLaunchKernelGGL((block_gram_shared_kernel<NT>), dim3(n), dim3(64 * ((NT + 1) / 2)), 0, stream, x, TG, partial);
  return launch_reduce<f32x4, 16>(partial, n, NT, 1, TG, Sigma, stream);
}

template <int NT>
static hipError_t launch_positions(const uint4 *x, int64_t TG, double *Sigma, void *workspace, size_t workspace_bytes,
                                   hipStream_t stream) {
  constexpr int KST = NT < 8 ? 8 / NT : 1;
  constexpr size_t stage = (size_t)8 * 4 * KST * 16 * NT * 16, lds = 2 * stage <= 128 * 1024 ? 2 * stage : stage;
  f64x4 *const partial = static_cast<f64x4 *>(workspace);
  const int64_t stages = (TG + 32 * KST - 1) / (32 * KST);
  const int64_t room = (int64_t)(workspace_bytes / ((size_t)32 * GramTiles<NT>::N * 2048));
  const int64_t most = room < gram_pos_slices(NT) ? room : gram_pos_slices(NT);
  constexpr int parts = gram_pos_parts(NT);
  const int n = (int)(stages < most ? stages : most);
  static std::atomic<uint64_t> raised{0};
  const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(block_gram_positions_kernel<NT>), lds, raised);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((block_gram_positions_kernel<NT>), dim3((n + 7) / 8 * 8 * 4 * parts), dim3(64 * GRAM_WAVES), lds,
                     stream, x, TG, n, partial);
  return launch_reduce<f64x4, 64>(partial, n, NT, 32, TG, Sigma, stream);
}

// G a multiple of 16 in [16, 256], TG > 0 token-groups, workspace of at least block_gram_workspace_least(G) bytes
// positions: the 32 matrices Sigma_k instead of Sigma
hipError_t launch_block_gram(const void *x_bf16, int64_t TG, int G, bool positions, double *Sigma, void *workspace,
                             size_t workspace_bytes, hipStream_t stream) {
  const uint4 *x = static_cast<const uint4 *>(x_bf16);
  switch (G / 16) {
#define TORQ_GRAM_CASE(NT_) \
  case NT_:                                                                                          \
    return positions ? launch_positions<NT_>(x, TG, Sigma, workspace, workspace_bytes, stream)       \
                     : launch_sigma<NT_>(x, TG, Sigma, workspace, workspace_bytes, stream);
    TORQ_GRAM_CASE(1) TORQ_GRAM_CASE(2) TORQ_GRAM_CASE(3) TORQ_GRAM_CASE(4)
    TORQ_GRAM_CASE(5) TORQ_GRAM_CASE(6) TORQ_GRAM_CASE(7) TORQ_GRAM_CASE(8)
    TORQ_GRAM_CASE(9) TORQ_GRAM_CASE(10) TORQ_GRAM_CASE(11) TORQ_GRAM_CASE(12)
    TORQ_GRAM_CASE(13) TORQ_GRAM_CASE(14) TORQ_GRAM_CASE(15) TORQ_GRAM_CASE(16)
#undef TORQ_GRAM_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace torq
