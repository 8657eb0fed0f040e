// mxfp4_gemm for few activation rows (decode, M <= 64): the W4A4 linear layer of Section 5
// (weight fusion) / Algorithm 3 ("Return"), same arithmetic as mxfp4_gemm.hip:
//
//   out[m][n] = sum_kb 2^(A_s[m][kb] + W_s[n][kb] - 254) * sum_{k<32} val(A[m][32kb+k]) val(W[n][32kb+k])
//
// With so few rows the work is reading the weights once, so the layout of the job follows the
// memory system, not the matrix cores: one workgroup per strip of 16 weight rows (or two or four strips),
// so that every CU streams; its 8 waves split the k range between them;
// the codes go global -> registers directly in the operand layout of
// v_mfma_scale_f32_16x16x128_f8f6f4 (lane = (row l % 16, microscaling block l / 16), 16 code
// bytes), all loads of a trip in flight at once; the scale bytes of the strip and of the
// activation rows are copied to LDS once per workgroup; and the eight partial 16 x 16 tiles are
// added through LDS at the end.  Activations (at most 64 rows) are re-read by every workgroup
// from the L2.
//
// The first MFMA operand is the weight strip and the second the activations, so an accumulator
// lane holds out[m = l % 16][n = n0 + 4 (l / 16) + 0..3]: four consecutive outputs of one row.
#include "rotate16_body.h"
#include "rotate32_resident.h"
#include "torq_device.h"
#include "torq_internal.h"

namespace torq {

namespace {

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

#define LDSP(x) ((__attribute__((address_space(3))) void *)(x))

constexpr int WAVES = 8;              // waves per workgroup = ways the k range is split
constexpr size_t SKINNY_MAX_LDS = 160 * 1024;
constexpr int LOCAL_MAX_TG = 4;       // token-groups that torq_linear_local_kernel rotates in every workgroup
constexpr int SKINNY_MIN_GROUPS = 384; // fewer workgroups than this leave CUs without work (256 CUs)

// a voffset that the range check of any buffer used here rejects (the load then delivers zeros)
constexpr int OOB_VOFF = 0x7FFFFFF0;

// what the decode form of torq_linear needs on top of the GEMM's arguments
struct DecodeArgs {
  const uint4 *x;
  int64_t TG;
  const uint4 *inter_hi, *inter_lo;            // R_inter in lane order, R_intra as the 32x32x16 operand
  const uint4 *intra_hi_frag, *intra_lo_frag;
  uint8_t *A_q, *A_s;          // written by the first P workgroups, read by the others
  int P;
  unsigned *ctr;
  int spin_limit;              // polls of the "ready" word before a waiting workgroup gives up
  int raise_ready;             // 0: the producers never raise "ready" (host-driven test of the give-up path)
};

}  // namespace

// The end of both kernels: add the waves' partial tiles through LDS and store.  Every wave's partial
// tiles go through LDS (red_mem: WAVES NS MT KiB) and the NS MT output tiles are shared out over the
// waves (tile k to wave k % WAVES), each added in the same fixed order, wave 0 + 1 + ... + 7: the same
// bits whichever wave does it (one wave adding up to eight tiles took a microsecond while seven waited).
template <int MT, int NS>
__device__ __forceinline__ void skinny_reduce_store(f32x4 (&acc)[NS][MT], unsigned char *red_mem, uint16_t *__restrict__ out,
                                                    int M, int64_t N, int64_t n0, int wave, int lane) {
  const int r16 = lane & 15, q = lane >> 4;
  __syncthreads();                                 // everybody is done with the scales
  float *red = reinterpret_cast<float *>(red_mem); // [WAVES][NS][MT][4][64]
#pragma unroll
  for (int n = 0; n < NS; ++n)
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[(((wave * NS + n) * MT + t) * 4 + r) * 64 + lane] = acc[n][t][r];
  __syncthreads();
#pragma unroll
  for (int n = 0; n < NS; ++n) {
    const int64_t nn = n0 + n * 16 + 4 * q;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if ((n * MT + t) % WAVES != wave) continue;  // uniform over the wave
      bf16x4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float sum = red[((n * MT + t) * 4 + r) * 64 + lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) sum += red[(((w * NS + n) * MT + t) * 4 + r) * 64 + lane];
        v[r] = (__bf16)sum;
      }
      const int m = t * 16 + r16;
      if (m < M) {
        uint16_t *dst = out + (int64_t)m * N + nn;
        if ((N & 3) == 0 && nn + 4 <= N) {
          *reinterpret_cast<bf16x4 *>(dst) = v;
        } else {
          const uint64_t bits = __builtin_bit_cast(uint64_t, v);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (nn + r < N) dst[r] = (uint16_t)(bits >> (16 * r));
        }
      }
    }
  }
}

// MT = number of 16-row activation tiles (M <= 16 MT); NS = 16-row weight strips per workgroup
// (1, 2 or 4; they share the activation loads); PT = line pairs per wave and trip.
// PERSIST: a workgroup takes the strip groups blockIdx.x, blockIdx.x + gridDim.x, ... and loads the
// activations' codes (and scale bytes) ONCE, keeping the codes in registers across its groups; only
// when one trip covers the k range (d / 256 <= PT * WAVES line pairs), where those registers are the
// trip's own.  Every workgroup otherwise re-reads all activation rows from the L2, which at 8 - 16 rows
// is half as many bytes again as the weights it streams.  Same arithmetic in the same order: the
// outputs are bit-identical.
template <int MT, int NS, int PT, bool PERSIST = false>
__global__ void __launch_bounds__(64 * WAVES)
mxfp4_gemm_skinny_kernel(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s,
                         const uint8_t *__restrict__ W_q, const uint8_t *__restrict__ W_s,
                         uint16_t *__restrict__ out, int M, int64_t N, int d, int wide) {
  // dynamic LDS: scale bytes of the weight strips (16 NS rows) and of the activation rows (16 MT),
  // d / 32 bytes each, every row padded by 4 or 16 bytes (the lanes of a k-step read one byte of 16
  // different rows); the waves' partial tiles are overlaid on it after the k loop
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int row_bytes = d / 2, srow_bytes = d / 32;
  const int KS = d / 128;                          // k-steps of one MFMA (128 elements, 4 blocks)
  const int KP = (KS + 1) / 2;                     // pairs of k-steps = whole 128-byte lines of a row
  const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(A_q, (uint32_t)M * row_bytes);
  const __amdgpu_buffer_rsrc_t as_rsrc = make_rsrc(A_s, (uint32_t)M * srow_bytes);
  const int c_voff = r16 * row_bytes + q * 16;     // codes: + 64 per k-step

  // ---- scales: copied to LDS by buffer loads with an LDS destination (no registers, nothing to
  // wait for before the code loads go out).  Such an instruction writes lane l's 4 or 16 bytes at (base + 4 l or
  // 16 l), the global address per lane is free: unit j of a region is (row j / pu, column j % pu) of the padded layout,
  // the pad column and rows past the end load zeros.  Their addresses hold the code loads up, so units of 16 bytes (wide)
  // take a quarter of the instructions where the rows allow it (us, by 4 and by 16, weights from HBM: [16, 28672] x 8192
  // 29.8 -> 28.3, [16, 4096] x 14336 10.0 -> 9.5, [45, 8192] x 5120 13.9 -> 13.3, [1, 14336] x 4096 9.6 -> 9.1; issued
  // behind the codes instead they come last and everything waits for them, [16, 8192] x 8192 10.7 -> 12.5).
  // (the unit as a shift: the compiler divides by a variable in 30 instructions ahead of the first load, 1 % of the products
  // of up to 16 rows and d <= 1024 at the median, 4 % at the 95th percentile)
  const int lg = wide ? 4 : 2, unit = 1 << lg;
  const int pu = (srow_bytes >> lg) + 1;           // units per padded row
  const int pd = pu << (lg - 2);                   // dwords per padded row
  const int w_ins = (16 * NS * pu + 63) / 64;      // instructions for the weight strips
  const int a_ins = (16 * MT * pu + 63) / 64;      // ... and for the activation rows
  const int ws_off = r16 * pd * 4 + q;             // this lane's scale byte: + 4 per k-step
  const int as_off = w_ins * 64 * unit + r16 * pd * 4 + q;
  // the waves' partial tiles: over the scales (one group per workgroup), behind them (PERSIST:
  // the activations' scale bytes stay)
  unsigned char *const red_mem = PERSIST ? smem + (w_ins + a_ins) * 64 * unit : smem;

  // j / pu in float: j < 2^17 and a quotient at least 1 / (2 pu) from an integer, pu < 2^11
  const float per_unit = __builtin_amdgcn_rcpf((float)pu);
  auto load_scales = [&](int i0, int i1, const __amdgpu_buffer_rsrc_t ws_rs) {
    for (int i = i0 + wave; i < i1; i += WAVES) {
      const bool is_w = i < w_ins;
      const int j = (is_w ? i : i - w_ins) * 64 + lane;
      const int row = (int)(((float)j + 0.5f) * per_unit), col = j - row * pu;
      const bool ok = col < pu - 1 && row < (is_w ? 16 * NS : 16 * MT);
      const int voff = ok ? row * srow_bytes + col * unit : OOB_VOFF;
      if (wide) __builtin_amdgcn_raw_ptr_buffer_load_lds(is_w ? ws_rs : as_rsrc, LDSP(smem + i * 1024), 16, voff, 0, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(is_w ? ws_rs : as_rsrc, LDSP(smem + i * 256), 4, voff, 0, 0, 0);
    }
  };
  // the activation codes of the k-steps of the trip that starts at line pair p0_
#define TORQ_LOAD_A(DST_, P0_)                                                                    \
  _Pragma("unroll") for (int u = 0; u < 2 * PT; ++u) {                                            \
    const int ks = 2 * ((P0_) + (u >> 1) * WAVES) + (u & 1);                                      \
    const bool in = ks < KS;                                                                      \
    _Pragma("unroll") for (int t = 0; t < MT; ++t)                                                \
        DST_[u][t] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, in ? c_voff : OOB_VOFF,        \
                                                           in ? ks * 64 + t * 16 * row_bytes : 0, 0); \
  }
  u32x4 aq_keep[PERSIST ? 2 * PT : 1][MT];
  if constexpr (PERSIST) {
    load_scales(w_ins, w_ins + a_ins, as_rsrc);
    TORQ_LOAD_A(aq_keep, wave)
  }

  const int64_t groups = (N + 16 * NS - 1) / (16 * NS);
  for (int64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {   // one group unless PERSIST
    const int64_t n0 = grp * 16 * NS;
    const int rows_w = (N - n0 < 16 * NS) ? (int)(N - n0) : 16 * NS;
    // rows past N or M are outside the buffers: their loads deliver zeros
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(W_q + n0 * row_bytes, (uint32_t)rows_w * row_bytes);
    const __amdgpu_buffer_rsrc_t ws_rsrc = make_rsrc(W_s + n0 * srow_bytes, (uint32_t)rows_w * srow_bytes);
    load_scales(0, PERSIST ? w_ins : w_ins + a_ins, ws_rsrc);

    f32x4 acc[NS][MT];
#pragma unroll
    for (int n = 0; n < NS; ++n)
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Wave w takes the line pairs w, w + WAVES, ...; PT pairs (2 PT k-steps) per trip, all of their
    // loads issued before the first MFMA.  Pairs past the end (and the second k-step of the last
    // pair when KS is odd) load zeros through the range check instead of branching.
    bool first = true;
    for (int p0 = wave; p0 < KP; p0 += PT * WAVES) {
      u32x4 wq[2 * PT][NS], aq_trip[PERSIST ? 1 : 2 * PT][MT];
#pragma unroll
      for (int u = 0; u < 2 * PT; ++u) {
        const int ks = 2 * (p0 + (u >> 1) * WAVES) + (u & 1);
        const bool in = ks < KS;
        const int cv = in ? c_voff : OOB_VOFF;
        const int co = in ? ks * 64 : 0;
#pragma unroll
        for (int n = 0; n < NS; ++n)
          wq[u][n] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, cv, co + (in ? n * 16 * row_bytes : 0), 0);
      }
      if constexpr (!PERSIST) { TORQ_LOAD_A(aq_trip, p0) }
      __builtin_amdgcn_sched_barrier(0);           // every load of the trip is in flight before the first wait
      if (first) {
        __syncthreads();                           // the scales are in LDS
        first = false;
      }
#pragma unroll
      for (int u = 0; u < 2 * PT; ++u) {
        const int ks = 2 * (p0 + (u >> 1) * WAVES) + (u & 1);
        const int sb = (ks < KS ? ks : 0) * 4;
        int asc[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) asc[t] = smem[as_off + t * 16 * pd * 4 + sb];
#pragma unroll
        for (int n = 0; n < NS; ++n) {
          const int wsc = smem[ws_off + n * 16 * pd * 4 + sb];
#pragma unroll
          for (int t = 0; t < MT; ++t) {
            const u32x4 av = PERSIST ? aq_keep[PERSIST ? u : 0][t] : aq_trip[PERSIST ? 0 : u][t];
            acc[n][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                i32x8{(int)wq[u][n][0], (int)wq[u][n][1], (int)wq[u][n][2], (int)wq[u][n][3], 0, 0, 0, 0},
                i32x8{(int)av[0], (int)av[1], (int)av[2], (int)av[3], 0, 0, 0, 0},
                acc[n][t], 4, 4, 0, wsc, 0, asc[t]);
          }
        }
      }
    }
    if (first) __syncthreads();                    // a wave without any pair still meets the others

    skinny_reduce_store<MT, NS>(acc, red_mem, out, M, N, n0, wave, lane);
    // PERSIST: the next group's scale bytes replace this group's, which every wave has read (first
    // barrier of the reduction); its partial tiles replace these once the adding waves have
    // arrived at the next group's barrier
  }
#undef TORQ_LOAD_A
}

// One lane of a consumer workgroup that is done with ctr[0] (see torq_linear_decode_kernel).
__device__ __forceinline__ void decode_consumer_done(unsigned *ctr, int gid, int groups) {
  const int stripes = groups < 64 ? groups : 64;
  const int s = gid % stripes;
  const unsigned quota = (unsigned)((groups - s + stripes - 1) / stripes);    // workgroups with gid % stripes == s
  const unsigned mine = __hip_atomic_fetch_add(&ctr[32 * (1 + s)], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (mine != quota - 1u) return;
  const unsigned full = __hip_atomic_fetch_add(&ctr[32 * 65], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (full != (unsigned)stripes - 1u) return;
  __hip_atomic_store(&ctr[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = 0; i < stripes; ++i) __hip_atomic_store(&ctr[32 * (1 + i)], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&ctr[32 * 65], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = 0; i < 64; ++i) __hip_atomic_store(&ctr[32 * (66 + i)], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------------------------
// torq_linear_single_launch: torq_linear for decode sizes in ONE launch (Algorithm 3, steps 1-4 and
// "Return").  With a few
// rows, rotate + quantise is a latency of 4-5 us in front of a GEMM of 4-30 us; here it runs in the
// first P workgroups of the GEMM's own launch (rotate32_resident, one token-group each: the codes are
// torq_rotate_quantize's, bit for bit) while
// the others, one per weight strip as in mxfp4_gemm_skinny_kernel, already have their scale bytes and
// the first trip of their weight codes on the way.  The two meet at counters in device memory
// (DECODE_CTR_WORDS words, one counter per 128-byte line: read-modify-writes of one address from
// the whole device take about 80 ns each, one after the other):
//   ctr[0]                   producers done: each adds 1 once its codes and scales (stored through to
//                            device-coherent memory) have been acknowledged; the last one raises
//   ctr[32 (66 + s)], s < 64  "ready", 64 copies: consumer g polls copy g % 64, so that no address is
//                            polled by more than 1/64 of the workgroups (thousands of polls on one
//                            address delay the producers' own updates of it);
//   ctr[32 (1 + s)], s < 64   consumers finished, striped the same way; a complete stripe adds 1 to
//   ctr[32 * 65]             stripes complete; the workgroup that completes the last one sets every
//                            counter back to 0, so that the next launch (and every replay of a
//                            captured one) starts from the same state;
//   ctr[DECODE_ERR]          "a workgroup gave up": set by a consumer whose bounded wait ran out, never
//                            cleared by a launch.  Such a consumer does not count itself as finished, so
//                            the counters are not set back either (late producers may still be adding to
//                            them); every consumer of every later launch sees the word first and writes
//                            NaN instead of multiplying whatever the stale counters would let through,
//                            until decode_ctr_reset_kernel has cleared all words.
// The consumers read the activations with device-coherent loads (sc1), so neither side needs a
// cache write-back or invalidate.
// Workgroups are dispatched in index order and the producers come first, so a waiting consumer can
// never keep a producer off the machine; the wait is bounded all the same (a consumer that gives
// up writes NaN to its outputs and raises the sticky error word).  Launches that share a handle's
// counters must not overlap.
template <int MT, int NS, int PT>
__global__ void __launch_bounds__(64 * WAVES, 4)
torq_linear_decode_kernel(const uint4 *__restrict__ x, int64_t TG, const uint4 *__restrict__ inter_hi,
                          const uint4 *__restrict__ inter_lo, const uint4 *__restrict__ intra_hi_frag,
                          const uint4 *__restrict__ intra_lo_frag, uint8_t *__restrict__ A_q,
                          uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                          const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int64_t N, int d,
                          int P, int groups, unsigned *__restrict__ ctr, int spin_limit, int raise_ready) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  if ((int)blockIdx.x < P) {
    {
      // codes and scale bytes are stored through to device-coherent memory (what an atomic store of device
      // scope does), for the readers in the other workgroups of this launch
      struct CoherentSink {
        unsigned long long *codes;
        uint8_t *scales;
        int64_t first_block;
        __device__ __forceinline__ void operator()(int64_t blk, int h, uint2 packed, uint32_t byte) const {
          const int64_t b = first_block + blk;
          __hip_atomic_store(&codes[b * 2 + h], ((unsigned long long)packed.y << 32) | packed.x, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
          if (h == 0) __hip_atomic_store(&scales[b], (uint8_t)byte, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } sink{reinterpret_cast<unsigned long long *>(A_q), A_s, (int64_t)blockIdx.x * 128};
      rotate32_resident(x + (int64_t)blockIdx.x * 512, 1, 128, inter_hi, inter_lo, intra_hi_frag, intra_lo_frag,
                        reinterpret_cast<char *>(smem), sink, []() {}, []() {});
    }
    __builtin_amdgcn_s_waitcnt(0);                 // this lane's stores have been acknowledged
    __syncthreads();
    if (tid == 0) {
      const unsigned before = __hip_atomic_fetch_add(&ctr[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (before == (unsigned)P - 1u && raise_ready)   // every producer's stores were complete before its own add
        for (int s = 0; s < 64; ++s) __hip_atomic_store(&ctr[32 * (66 + s)], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int row_bytes = d / 2, srow_bytes = d / 32;
  const int KS = d / 128;
  const int KP = (KS + 1) / 2;
  const int64_t n0 = (int64_t)((int)blockIdx.x - P) * 16 * NS;
  const int rows_w = (N - n0 < 16 * NS) ? (int)(N - n0) : 16 * NS;
  const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(W_q + n0 * row_bytes, (uint32_t)rows_w * row_bytes);
  const __amdgpu_buffer_rsrc_t ws_rsrc = make_rsrc(W_s + n0 * srow_bytes, (uint32_t)rows_w * srow_bytes);
  const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(A_q, (uint32_t)M * row_bytes);
  const __amdgpu_buffer_rsrc_t as_rsrc = make_rsrc(A_s, (uint32_t)M * srow_bytes);
  const int c_voff = r16 * row_bytes + q * 16;
  const int sdw = srow_bytes / 4, pd = sdw + 1;
  const int w_ins = (16 * NS * pd + 63) / 64, a_ins = (16 * MT * pd + 63) / 64;
  const int ws_off = r16 * pd * 4 + q;
  const int as_off = w_ins * 256 + r16 * pd * 4 + q;

  // ---- the weight side goes out first: scale bytes to LDS, the first trip's codes to registers
  for (int i = wave; i < w_ins; i += WAVES) {
    const int j = i * 64 + lane;
    const int row = j / pd, col = j - row * pd;
    const bool ok = col < sdw && row < 16 * NS;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ws_rsrc, LDSP(smem + i * 256), 4, ok ? row * srow_bytes + col * 4 : OOB_VOFF, 0, 0, 0);
  }
  u32x4 wq[2 * PT][NS], aq[2 * PT][MT];
  // AUX_: cache policy of the load; 16 = sc1, a device-coherent read
#define TORQ_LOAD_TRIP(DST_, RSRC_, CNT_, P0_, AUX_)                                             \
  _Pragma("unroll") for (int u = 0; u < 2 * PT; ++u) {                                           \
    const int ks = 2 * ((P0_) + (u >> 1) * WAVES) + (u & 1);                                     \
    const bool in = ks < KS;                                                                     \
    _Pragma("unroll") for (int n = 0; n < CNT_; ++n)                                             \
        DST_[u][n] = __builtin_amdgcn_raw_buffer_load_b128(RSRC_, in ? c_voff : OOB_VOFF,        \
                                                           in ? ks * 64 + n * 16 * row_bytes : 0, AUX_); \
  }
  int p0 = wave;
  if (p0 < KP) { TORQ_LOAD_TRIP(wq, w_rsrc, NS, p0, 0) }
  __builtin_amdgcn_sched_barrier(0);

  // ---- wait for the activations' codes and scales
  if (tid == 0) {
    const unsigned *flag = &ctr[32 * (66 + (((int)blockIdx.x - P) & 63))];
    // an earlier launch on these counters gave up: they are stale, nothing they say can be trusted
    const unsigned err = __hip_atomic_load(&ctr[DECODE_ERR], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned seen = 0;
    if (!err) {
      for (int spin = 0; spin < spin_limit; ++spin) {
        seen = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (seen) break;
        __builtin_amdgcn_s_sleep(8);
      }
      if (!seen) __hip_atomic_store(&ctr[DECODE_ERR], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    reinterpret_cast<volatile unsigned *>(smem)[(w_ins + a_ins) * 64] = seen;
  }
  __syncthreads();
  const bool ready = reinterpret_cast<volatile unsigned *>(smem)[(w_ins + a_ins) * 64] != 0;
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");                   // nothing below is moved above the wait
  if (!ready) {                                    // uniform over the workgroup
    __builtin_amdgcn_s_waitcnt(0);                 // the loads already issued land before the workgroup's LDS and registers go
    // gave up (or the counters are stale): mark this strip's outputs as NaN rather than leave what the
    // buffer held; the workgroup does not count as finished, so no launch sets the counters back
    for (int e = tid; e < M * 16 * NS; e += 64 * WAVES) {
      const int m = e / (16 * NS);
      const int64_t n = n0 + e % (16 * NS);
      if (n < N) out[(int64_t)m * N + n] = 0x7FC0;
    }
    return;
  }

  for (int i = w_ins + wave; i < w_ins + a_ins; i += WAVES) {
    const int j = (i - w_ins) * 64 + lane;
    const int row = j / pd, col = j - row * pd;
    const bool ok = col < sdw && row < 16 * MT;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(as_rsrc, LDSP(smem + i * 256), 4, ok ? row * srow_bytes + col * 4 : OOB_VOFF, 0, 0, 16);
  }

  f32x4 acc[NS][MT];
#pragma unroll
  for (int n = 0; n < NS; ++n)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  bool first = true;
  for (; p0 < KP; p0 += PT * WAVES) {
    if (!first) { TORQ_LOAD_TRIP(wq, w_rsrc, NS, p0, 0) }
    TORQ_LOAD_TRIP(aq, a_rsrc, MT, p0, 16)
    __builtin_amdgcn_sched_barrier(0);
    if (first) {
      __syncthreads();                             // the scales are in LDS
      first = false;
    }
#pragma unroll
    for (int u = 0; u < 2 * PT; ++u) {
      const int ks = 2 * (p0 + (u >> 1) * WAVES) + (u & 1);
      const int sb = (ks < KS ? ks : 0) * 4;
      int asc[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) asc[t] = smem[as_off + t * 16 * pd * 4 + sb];
#pragma unroll
      for (int n = 0; n < NS; ++n) {
        const int wsc = smem[ws_off + n * 16 * pd * 4 + sb];
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[n][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              i32x8{(int)wq[u][n][0], (int)wq[u][n][1], (int)wq[u][n][2], (int)wq[u][n][3], 0, 0, 0, 0},
              i32x8{(int)aq[u][t][0], (int)aq[u][t][1], (int)aq[u][t][2], (int)aq[u][t][3], 0, 0, 0, 0},
              acc[n][t], 4, 4, 0, wsc, 0, asc[t]);
      }
    }
  }
#undef TORQ_LOAD_TRIP
  if (first) __syncthreads();                      // a wave without any pair still meets the others

  skinny_reduce_store<MT, NS>(acc, smem, out, M, N, n0, wave, lane);
  if (tid == 0) decode_consumer_done(ctr, (int)blockIdx.x - P, groups);
}

// ---------------------------------------------------------------------------------------------
// torq_linear for a few token-groups (one to four rows of a decode step) with the packed activations
// never leaving the chip: Algorithm 3, steps 1-4 and "Return", in one launch and without any hand-off
// between workgroups.  Every workgroup rotates and quantises ALL token-groups itself (rotate32_resident
// on its 8 waves, G = 112 or 128: 2.9 MFLOP per token-group, well under a microsecond) into its own LDS while the
// scale bytes and the first trip of weight codes of its first strips are on the way, and then
// streams its share of the weight strips as mxfp4_gemm_skinny_kernel<1, NS, PT, true> does, with the
// activation operand read from LDS instead of from memory.  Workgroups are persistent (the rotation is
// paid once per workgroup, not once per strip).  Workgroup 0 also stores the codes and scale bytes to
// A_q / A_s (the caller's workspace, same layout as torq_rotate_quantize), which nothing in the launch
// reads: they are what was multiplied, for the caller to inspect.
//
// One trip of a wave holds 2 PT k-steps of NS strips in registers (32 PT NS bytes per lane); the launcher
// picks NS and PT so that, where 128 registers allow, one trip is the workgroup's whole share: then every
// weight byte of the launch is requested before the rotation starts, and the rotation's latency (two
// dependent reads from memory and a chain of 22 MFMAs) hides behind the stream.
//
// LDS: [weight-strip scales | activation scales (16 rows, zero beyond M) | codes, M rows of d / 2 + 16
// bytes (the pad spreads the rows over the banks) | the token-groups' bf16 values (8 KiB each), later
// the partial tiles of the reduction (8 NS KiB)].

// The end of torq_linear_local_kernel: as skinny_reduce_store for one activation tile, but with wave n
// adding strip n (every wave's partial tile goes through LDS, red_mem = 8 NS KiB): with up to four
// strips per workgroup one wave would add 112 values per lane while seven wait.  Same order of additions
// (wave 0 + 1 + ... + 7): the same bits.
template <int NS>
__device__ __forceinline__ void local_reduce_store(f32x4 (&acc)[NS][1], unsigned char *red_mem, uint16_t *__restrict__ out,
                                                   int M, int64_t N, int64_t n0, int wave, int lane) {
  const int r16 = lane & 15, q = lane >> 4;
  __syncthreads();                                 // everybody is done with the scales and the codes
  float *red = reinterpret_cast<float *>(red_mem); // [WAVES][NS][4][64]
#pragma unroll
  for (int n = 0; n < NS; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[((wave * NS + n) * 4 + r) * 64 + lane] = acc[n][0][r];
  __syncthreads();
  if (wave < NS) {
    const int n = wave;
    const int64_t nn = n0 + n * 16 + 4 * q;
    bf16x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float sum = red[(n * 4 + r) * 64 + lane];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) sum += red[((w * NS + n) * 4 + r) * 64 + lane];
      v[r] = (__bf16)sum;
    }
    if (r16 < M) {
      uint16_t *dst = out + (int64_t)r16 * N + nn;
      if ((N & 3) == 0 && nn + 4 <= N) {
        *reinterpret_cast<bf16x4 *>(dst) = v;
      } else {
        const uint64_t bits = __builtin_bit_cast(uint64_t, v);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (nn + r < N) dst[r] = (uint16_t)(bits >> (16 * r));
      }
    }
  }
}

// EXACT: d / 256 == PT * WAVES, one trip is the k range with no k-step past the end: its loads then need
// no range predicate, compile to straight-line code, and the compiler's count of them is exact.
template <int NS, int PT, bool EXACT>
__global__ void __launch_bounds__(64 * WAVES, 2)
torq_linear_local_kernel(const uint4 *__restrict__ x, int TG, int G, const uint4 *__restrict__ inter_hi,
                         const uint4 *__restrict__ inter_lo, const uint4 *__restrict__ intra_hi_frag,
                         const uint4 *__restrict__ intra_lo_frag, uint8_t *__restrict__ A_q,
                         uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                         const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int64_t N, int d) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int row_bytes = d / 2, srow_bytes = d / 32;
  const int KS = d / 128;
  const int KP = (KS + 1) / 2;
  const int c_voff = r16 * row_bytes + q * 16;
  const int sdw = srow_bytes / 4, pd = sdw + 1;
  const int w_ins = (16 * NS * pd + 63) / 64, a_ins = (16 * pd + 63) / 64;
  const int ws_off = r16 * pd * 4 + q;
  const int as_off = w_ins * 256 + r16 * pd * 4 + q;
  const int a_stride = row_bytes + 16;
  unsigned char *const s_a = smem + w_ins * 256;
  unsigned char *const a_c = smem + (w_ins + a_ins) * 256;
  unsigned char *const xs = a_c + (M * a_stride + 255) / 256 * 256;     // TG token-groups, then partial tiles

  const int64_t groups = (N + 16 * NS - 1) / (16 * NS);
  auto load_w_scales = [&](const __amdgpu_buffer_rsrc_t ws_rs) {
    for (int i = wave; i < w_ins; i += WAVES) {
      const int j = i * 64 + lane;
      const int row = j / pd, col = j - row * pd;
      const bool ok = col < sdw && row < 16 * NS;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ws_rs, LDSP(smem + i * 256), 4, ok ? row * srow_bytes + col * 4 : OOB_VOFF, 0, 0, 0);
    }
  };
  u32x4 wq[2 * PT][NS];
#define TORQ_LOAD_W(RSRC_, P0_)                                                                   \
  _Pragma("unroll") for (int u = 0; u < 2 * PT; ++u) {                                            \
    const int ks = 2 * ((P0_) + (u >> 1) * WAVES) + (u & 1);                                      \
    const bool in = EXACT || ks < KS;                                                             \
    _Pragma("unroll") for (int n = 0; n < NS; ++n)                                                \
        wq[u][n] = __builtin_amdgcn_raw_buffer_load_b128(RSRC_, in ? c_voff : OOB_VOFF,           \
                                                         in ? ks * 64 + n * 16 * row_bytes : 0, 0); \
  }

  // ---- steps 1-4 into LDS.  The rotation's own reads from memory are requested first and the first
  // trip's weight codes right behind them (reads return in order: the rotation must not queue behind
  // the weights); the scale bytes of the rows past M are zeros
  for (int i = tid; i < a_ins * 64; i += 64 * WAVES) reinterpret_cast<uint32_t *>(s_a)[i] = 0u;
  {
    LocalSink sink;
    sink.a_c = a_c;
    sink.s_a = s_a;
    sink.a_stride = a_stride;
    sink.s_stride = pd * 4;
    sink.bpr = srow_bytes;
    sink.codes_g = blockIdx.x == 0 ? reinterpret_cast<uint2 *>(A_q) : nullptr;
    sink.scales_g = A_s;
    const int64_t n0 = (int64_t)blockIdx.x * 16 * NS;
    const int rows_w = (N - n0 < 16 * NS) ? (int)(N - n0) : 16 * NS;
    load_w_scales(make_rsrc(W_s + n0 * srow_bytes, (uint32_t)rows_w * srow_bytes));   // few bytes, ahead of everything
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(W_q + n0 * row_bytes, (uint32_t)rows_w * row_bytes);
    auto weights_first_trip = [&]() {
      // The waves meet (nothing is waited for) so that every wave's rotation reads are in the CU's
      // memory pipeline before any wave's weight reads: the pipeline takes requests in order, and a
      // later wave's 5 KB for the rotation would otherwise queue behind 16 KB of weights per earlier wave.
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (EXACT || wave < KP) { TORQ_LOAD_W(w_rsrc, wave) }
      __builtin_amdgcn_sched_barrier(0);
    };
    // (two barriers inside: the first also orders the clearing above before any scale byte, the second
    // makes the results visible)
    rotate32_resident(x, TG, G, inter_hi, inter_lo, intra_hi_frag, intra_lo_frag, reinterpret_cast<char *>(xs), sink,
                      weights_first_trip, []() {});
  }

  // ---- the strip groups of this workgroup
  bool preloaded = true;
  for (int64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    const int64_t n0 = grp * 16 * NS;
    const int rows_w = (N - n0 < 16 * NS) ? (int)(N - n0) : 16 * NS;
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(W_q + n0 * row_bytes, (uint32_t)rows_w * row_bytes);
    if (!preloaded) load_w_scales(make_rsrc(W_s + n0 * srow_bytes, (uint32_t)rows_w * srow_bytes));

    f32x4 acc[NS][1];
#pragma unroll
    for (int n = 0; n < NS; ++n) acc[n][0] = f32x4{0.f, 0.f, 0.f, 0.f};

    bool first = true;
    for (int p0 = wave; p0 < KP; p0 += PT * WAVES) {
      if (!(preloaded && first)) { TORQ_LOAD_W(w_rsrc, p0) }
      u32x4 aq[2 * PT];
#pragma unroll
      for (int u = 0; u < 2 * PT; ++u) {
        const int ks = 2 * (p0 + (u >> 1) * WAVES) + (u & 1);
        aq[u] = ((EXACT || ks < KS) && r16 < M) ? *reinterpret_cast<const u32x4 *>(a_c + r16 * a_stride + ks * 64 + q * 16)
                                     : u32x4{0u, 0u, 0u, 0u};
      }
      __builtin_amdgcn_sched_barrier(0);
      if (first) {
        __syncthreads();                           // the strip's scale bytes are in LDS
        first = false;
      }
#pragma unroll
      for (int u = 0; u < 2 * PT; ++u) {
        const int ks = 2 * (p0 + (u >> 1) * WAVES) + (u & 1);
        const int sb = ((EXACT || ks < KS) ? ks : 0) * 4;
        const int asc = smem[as_off + sb];
#pragma unroll
        for (int n = 0; n < NS; ++n) {
          const int wsc = smem[ws_off + n * 16 * pd * 4 + sb];
          acc[n][0] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              i32x8{(int)wq[u][n][0], (int)wq[u][n][1], (int)wq[u][n][2], (int)wq[u][n][3], 0, 0, 0, 0},
              i32x8{(int)aq[u][0], (int)aq[u][1], (int)aq[u][2], (int)aq[u][3], 0, 0, 0, 0},
              acc[n][0], 4, 4, 0, wsc, 0, asc);
        }
      }
    }
    if (first) __syncthreads();                    // a wave without any pair still meets the others
    preloaded = false;

    // the partial tiles go where the rotation staged its input; the next group's scale bytes replace
    // this group's once every wave has read them (first barrier of the reduction), and its partial tiles
    // these once the adding waves have arrived at the next group's barrier
    local_reduce_store<NS>(acc, xs, out, M, N, n0, wave, lane);
  }
#undef TORQ_LOAD_W
}

// scale rows of whole 16-byte units
static bool rows16(const uint8_t *A_s, const uint8_t *W_s, int d) {
  return d % 512 == 0 && ((reinterpret_cast<uintptr_t>(A_s) | reinterpret_cast<uintptr_t>(W_s)) & 15u) == 0;
}

// the scale bytes in LDS, copied by units of 4 or 16 bytes
static size_t skinny_scale_bytes(int MT, int NS, int d, int unit = 4) {
  const int pu = d / 32 / unit + 1;                // units per padded row
  return (size_t)((16 * NS * pu + 63) / 64 + (16 * MT * pu + 63) / 64) * 64 * unit;
}
static size_t skinny_red_bytes(int MT, int NS) { return (size_t)WAVES * NS * MT * 4 * 64 * sizeof(float); }

static size_t skinny_lds_bytes(int MT, int NS, int d, int unit = 4) {
  const size_t scale_bytes = skinny_scale_bytes(MT, NS, d, unit), red_bytes = skinny_red_bytes(MT, NS);
  return scale_bytes > red_bytes ? scale_bytes : red_bytes;
}

// ---------------------------------------------------------------------------------------------
// The same product where a CU has at most one workgroup's strips to stream (up to 256 workgroups): whole lines.
// An operand load of the kernel above touches 16 rows of 64 bytes, half a line each, and what a CU can have on its way is
// counted in lines (measured: a strip of 16 rows x 4 KB in 1.6 us by half lines, 1.1 by whole ones).  Here a load is 8
// rows of 128 bytes straight into LDS, where the operand layout is picked up again; the ring of R items (a line pair of
// the NS strips and of the MT activation tiles) is the wave's own, so nothing in the k loop waits for another wave.
// Same k-steps, same order, same bits.
template <int N>
__device__ __forceinline__ void lines_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// ONCE: the weights' codes with the non-temporal hint (ONE_PASS_WEIGHT_BYTES), [16, 28672] x 8192 24.2 -> 22.0 us.
template <int MT, int NS, int R, bool ONCE>
__device__ __forceinline__ void
gemm_lines(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
           const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int64_t N, int d, int pad, unsigned char *smem) {
  constexpr int T = NS + MT, OPS = 2 * T, ITEM = T * 2048;          // tiles, DMA instructions and bytes of an item
  static_assert(R * OPS <= 63, "the counter of loads in flight has six bits");
  // LDS: [rings | scale rows of the strips, then of the activation tiles, 16 bytes of padding each (pad = 1) where there
  // is room]; the waves' partial tiles over the rings at the end
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int row_bytes = d / 2, srow_bytes = d / 32, KP = d / 256;   // d is a multiple of 512
  const int64_t n0 = (int64_t)blockIdx.x * (16 * NS);
  const int rows_w = (N - n0 < 16 * NS) ? (int)(N - n0) : 16 * NS;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t sc0 = lds0 + WAVES * R * ITEM;
  const unsigned char *const sc = smem + WAVES * R * ITEM;

  // ---- scale rows first: unit j of 16 bytes is (row j / pu, column j % pu), the pad column loads zeros
  const int pu = srow_bytes / 16 + pad, s_pitch = pu * 16;
  const int w_units = 16 * NS * pu, units = w_units + 16 * MT * pu;
  {
    const i32x4 ws_rs = raw_buffer(W_s + n0 * srow_bytes, (uint32_t)rows_w * srow_bytes);
    const i32x4 as_rs = raw_buffer(A_s, (uint32_t)M * srow_bytes);
    const float per_unit = __builtin_amdgcn_rcpf((float)pu);        // (j / pu in float, as above)
    for (int i = wave; i * 64 < units; i += WAVES) {
      const int j = i * 64 + lane;
      const int row = (int)(((float)j + 0.5f) * per_unit), col = j - row * pu;
      const bool ok = col < srow_bytes / 16;
      // the lanes of an instruction may straddle the strips' and the tiles' rows: one masked load from each buffer, and
      // where only one is needed the other is an empty one
      const bool is_w = row < 16 * NS;
      if (i * 64 < w_units)
        { if (is_w) load_to_lds16(ws_rs, sc0 + i * 1024, ok ? row * srow_bytes + col * 16 : OOB_VOFF, 0); }
      if (i * 64 + 63 >= w_units)
        { if (!is_w) load_to_lds16(as_rs, sc0 + i * 1024, ok ? (row - 16 * NS) * srow_bytes + col * 16 : OOB_VOFF, 0); }
    }
  }

  // ---- items: line pair kp = wave, wave + 8, ...; chunks swizzled by the row, as the reads below expect
  const i32x4 w_rs = raw_buffer(W_q + n0 * row_bytes, (uint32_t)rows_w * row_bytes);
  const i32x4 a_rs = raw_buffer(A_q, (uint32_t)M * row_bytes);
  const int l_row = lane >> 3;
  const int v0 = l_row * row_bytes + ((lane & 7) ^ (l_row >> 1)) * 16, v1 = (l_row + 8) * row_bytes + ((lane & 7) ^ (l_row >> 1) ^ 4) * 16;
  const uint32_t ring0 = lds0 + wave * R * ITEM;
  const unsigned char *const ring = smem + wave * R * ITEM;
  auto request = [&](int kp, int slot) {
    const bool ok = kp < KP;                                        // past the k range: empty buffers, the counts hold
    i32x4 rw = w_rs, ra = a_rs;
    rw[2] = ok ? rw[2] : 0;
    ra[2] = ok ? ra[2] : 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int so = (t < NS ? t : t - NS) * 16 * row_bytes + kp * 128;
      if (ONCE && t < NS) {
        load_to_lds16<true, true>(rw, ring0 + slot * ITEM + t * 2048, v0, so);
        load_to_lds16<true, true>(rw, ring0 + slot * ITEM + t * 2048 + 1024, v1, so);
        continue;
      }
      load_to_lds16(t < NS ? rw : ra, ring0 + slot * ITEM + t * 2048, v0, so);
      load_to_lds16(t < NS ? rw : ra, ring0 + slot * ITEM + t * 2048 + 1024, v1, so);
    }
  };
#pragma unroll
  for (int i = 0; i < R; ++i) request(wave + i * WAVES, i);

  f32x4 acc[NS][MT];
#pragma unroll
  for (int n = 0; n < NS; ++n)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  lines_wait<R * OPS>();                                            // this wave's scale bytes have landed
  asm volatile("s_barrier" ::: "memory");

  const int f_off[2] = {r16 * 128 + ((q ^ ((r16 >> 1) & 7)) * 16), r16 * 128 + (((4 + q) ^ ((r16 >> 1) & 7)) * 16)};
  int slot = 0;
  for (int kp = wave; kp < KP; kp += WAVES) {
    lines_wait<(R - 1) * OPS>();                                    // the oldest item has landed
    u32x4 f[2][T];
    int fs[2][T];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        f[e][t] = *reinterpret_cast<const u32x4 *>(ring + slot * ITEM + t * 2048 + f_off[e]);
        fs[e][t] = sc[(t * 16 + r16) * s_pitch + (2 * kp + e) * 4 + q];
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // read: the slot can be filled again
    request(kp + R * WAVES, slot);
    slot = slot + 1 == R ? 0 : slot + 1;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[n][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              i32x8{(int)f[e][n][0], (int)f[e][n][1], (int)f[e][n][2], (int)f[e][n][3], 0, 0, 0, 0},
              i32x8{(int)f[e][NS + t][0], (int)f[e][NS + t][1], (int)f[e][NS + t][2], (int)f[e][NS + t][3], 0, 0, 0, 0},
              acc[n][t], 4, 4, 0, fs[e][n], 0, fs[e][NS + t]);
  }
  lines_wait<0>();                                                  // nothing is on its way into the LDS any more
  skinny_reduce_store<MT, NS>(acc, smem, out, M, N, n0, wave, lane);
}

template <int MT, int NS, int R>
__global__ void __launch_bounds__(64 * WAVES)
mxfp4_gemm_lines_kernel(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                        const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int64_t N, int d, int pad) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  gemm_lines<MT, NS, R, false>(A_q, A_s, W_q, W_s, out, M, N, d, pad, smem);
}
template <int MT, int NS, int R>
__global__ void __launch_bounds__(64 * WAVES)
mxfp4_gemm_lines_once_kernel(const uint8_t *__restrict__ A_q, const uint8_t *__restrict__ A_s, const uint8_t *__restrict__ W_q,
                             const uint8_t *__restrict__ W_s, uint16_t *__restrict__ out, int M, int64_t N, int d, int pad) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  gemm_lines<MT, NS, R, true>(A_q, A_s, W_q, W_s, out, M, N, d, pad, smem);
}

static size_t lines_lds_bytes(int MT, int NS, int R, int d, int pad) {
  const size_t units = (size_t)16 * (NS + MT) * (d / 512 + pad), rings = (size_t)WAVES * R * (NS + MT) * 2048;
  const size_t bytes = rings + (units + 63) / 64 * 1024, red = skinny_red_bytes(MT, NS);
  return bytes > red ? bytes : red;
}

static int lines_pad(int MT, int NS, int R, int d) { return lines_lds_bytes(MT, NS, R, d, 1) <= SKINNY_MAX_LDS ? 1 : 0; }

// the bytes of the widest weights that a form takes: a workgroup a CU, and the k range whose scale rows fit beside its rings
static constexpr double lines_most_weights(int MT, int NS, int R) {
  const int pieces = (int)((SKINNY_MAX_LDS - (size_t)WAVES * R * (NS + MT) * 2048) / (256 * (size_t)(NS + MT)));
  return 256.0 * 16 * NS * 512 * pieces * 0.53125;
}

// the deepest ring with room for the scale rows: 4 items of two tiles, 3 (2) of three, 2 (1) of four, 1 of five to eight;
// 0: none
static int lines_ring(int MT, int NS, int d) {
  const int T = NS + MT, most = T == 2 ? 4 : T == 3 ? 3 : T == 4 ? 2 : T <= 8 ? 1 : 0;
  for (int R = most; R >= 1 && R >= most - 1; --R)
    if (lines_lds_bytes(MT, NS, R, d, 0) <= SKINNY_MAX_LDS) return R;
  return 0;
}

// Strips per workgroup of the whole-line form, 0 where it does not take the product (d a multiple of 512, 16-byte
// aligned scale rows): as few as leave a CU at most one workgroup, which keeps every CU busy and reads the activations
// once a CU.  It is ahead almost everywhere it fits, the more the more rows and the longer the k range; us, the other
// form against this one, weights from HBM: [16, 8192] x 1024 6.6 / 4.6, [16, 8192] x 8192 10.1 / 9.9, [16, 28672] x 8192
// 28.9 / 23.2, [45, 5120] x 8192 10.6 / 8.5, [45, 8192] x 5120 13.2 / 9.9, [64, 4096] x
// 4096 8.0 / 5.3, [1, 14336] x 4096 9.0 / 8.4, [1, 4096] x 14336 8.7 / 8.2.  Short k ranges leave its waves idle (one
// line pair each is 2048 elements) and have it wait for its scale bytes: up to d = 1024 it takes only many rows, or from
// 17 rows on more than one strip a CU ([16, 1024] x 2048 0.9 times as fast, [40, 1024] x 5120 1.2, [64, 512] x 128 1.06);
// below 8 rows the other form also keeps d = 2048 (0.94 - 1.04) and rows a multiple of 4 KB apart past 448 strips
// ([1, 8192] x 28672 0.93, [1, 16384] x 16384 0.91: all workgroups walk the same columns, whose lines share channels).
// From 8 rows on past 1600 strips: seven strips a CU leave a ring of one item, and beside it the scale rows of d = 8192 at
// most.  At that length (rows 4 KB apart again) even the persistent form below was ahead, and the ring of strips
// (mxfp4_gemm_stream.hip), which takes such a product, is ahead of both: [16, 8192] x 28672 in a decoder block 29.4 / 27.5 / 25.4
// (this form, that one, the ring), alone 31.0 / 31.0 / 23.8; this form and the persistent one, whole calls [8, 8192] x 26624 30.5 / 28.4, [12, 8192] x 28672 31.8 / 30.3,
// [16, 8192] x 26624 30.7 / 29.8, but x 25600 28.2 / 29.4, x 24576 27.6 / 28.8, x 20480 22.7 / 28.7.
// Three strips of one activation tile: four measured up to 6 % ahead.
int mxfp4_gemm_lines_strips(int64_t M, int64_t N, int d) {
  if (M < 1 || M > 64 || d % 512 != 0) return 0;
  const int MT = (int)((M + 15) / 16);
  const int64_t strips = (N + 15) / 16;
  if (strips > 7 * 256) return 0;
  int NS = (int)((strips + 255) / 256);
  if (MT == 1 && NS == 3) NS = 4;
  if (NS + MT > 8 || lines_ring(MT, NS, d) == 0) return 0;
  const bool pays = MT == 4   ? true
                    : MT == 3 ? d >= 1024 || strips > 256
                    : MT == 2 ? d >= 2048 || (strips > 256 && strips <= 1024)
                    : M >= 8  ? d >= 2048 && (d < 8192 || strips <= 1600)
                              : d >= 3072 && (d % 8192 != 0 || strips <= 448);
  return pays ? NS : 0;
}

// whether the product (16-byte aligned scale rows) takes the whole-line form, and which: strips per workgroup, items in a
// wave's ring, padding of the scale rows
bool mxfp4_gemm_lines_form(int64_t M, int64_t N, int d, int *strips, int *items, int *padded) {
  const int NS = mxfp4_gemm_lines_strips(M, N, d);
  if (NS == 0) return false;
  const int MT = (int)((M + 15) / 16);
  *strips = NS;
  *items = lines_ring(MT, NS, d);
  *padded = lines_pad(MT, NS, *items, d);
  return true;
}

template <int MT, int NS, int R>
static hipError_t launch_lines(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M,
                               int64_t N, int d, hipStream_t stream) {
  const int pad = lines_pad(MT, NS, R, d);
  const size_t lds = lines_lds_bytes(MT, NS, R, d, pad);
  auto go = [&](auto kernel, std::atomic<uint64_t> &raised) {
    if (lds > 64 * 1024) {
      const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(kernel), SKINNY_MAX_LDS, raised);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)((N + 16 * NS - 1) / (16 * NS))), dim3(64 * WAVES), lds, stream, A_q, A_s, W_q, W_s,
                       reinterpret_cast<uint16_t *>(out), (int)M, N, d, pad);
    return hipGetLastError();
  };
  static std::atomic<uint64_t> raised[2];
  // (one strip a workgroup, at most 4096 rows, would be as much from d = 46000 on: no layer here)
  if constexpr (NS >= 2 && lines_most_weights(MT, NS, R) > ONE_PASS_WEIGHT_BYTES)
    if ((double)N * (double)d * 0.53125 > ONE_PASS_WEIGHT_BYTES) return go(mxfp4_gemm_lines_once_kernel<MT, NS, R>, raised[1]);
  return go(mxfp4_gemm_lines_kernel<MT, NS, R>, raised[0]);
}

template <int MT>
static hipError_t launch_lines_mt(int NS, const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s, void *out,
                                  int64_t M, int64_t N, int d, hipStream_t stream) {
  const int R = lines_ring(MT, NS, d);
#define TORQ_LINES(NS_)                                                                                                     \
  if constexpr (NS_ + MT <= 8 && !(MT == 1 && NS_ == 3))                                                                    \
    if (NS == NS_) {                                                                                                        \
      constexpr int T = NS_ + MT, MOST = T == 2 ? 4 : T == 3 ? 3 : T == 4 ? 2 : 1;                                          \
      if (R == MOST) return launch_lines<MT, NS_, MOST>(A_q, A_s, W_q, W_s, out, M, N, d, stream);                          \
      if constexpr (MOST > 1) if (R == MOST - 1) return launch_lines<MT, NS_, MOST - 1>(A_q, A_s, W_q, W_s, out, M, N, d, stream); \
    }
  TORQ_LINES(1) TORQ_LINES(2) TORQ_LINES(3) TORQ_LINES(4) TORQ_LINES(5) TORQ_LINES(6) TORQ_LINES(7)
#undef TORQ_LINES
  return hipErrorInvalidValue;
}

template <int MT, int NS, int PT>
static hipError_t launch_cfg(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                             void *out, int64_t M, int64_t N, int d, hipStream_t stream, const DecodeArgs *fused) {
  const int64_t groups = (N + 16 * NS - 1) / (16 * NS);
  if (groups > 0x7FFFFFF0) return hipErrorInvalidValue;
  const size_t scale_bytes = skinny_scale_bytes(MT, NS, d);
  size_t lds_bytes = skinny_lds_bytes(MT, NS, d);
  if constexpr (NS <= 2 && PT <= (MT + NS <= 3 ? 4 : 2)) if (fused) {
    // + the "ready" word behind the scales; at least the rotation's four token-group places
    lds_bytes = lds_bytes > scale_bytes + 16 ? lds_bytes : scale_bytes + 16;
    const size_t rot_bytes = 4 * (size_t)RotCfg<4>::TG_LDS_BYTES;
    lds_bytes = lds_bytes > rot_bytes ? lds_bytes : rot_bytes;
    if (lds_bytes > SKINNY_MAX_LDS) return hipErrorInvalidValue;
    if (lds_bytes > 64 * 1024) {
      static std::atomic<uint64_t> raised{0};
      const hipError_t e =
          raise_lds_limit(reinterpret_cast<const void *>(torq_linear_decode_kernel<MT, NS, PT>), SKINNY_MAX_LDS, raised);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((torq_linear_decode_kernel<MT, NS, PT>), dim3((unsigned)(groups + fused->P)), dim3(64 * WAVES),
                       lds_bytes, stream, fused->x, fused->TG, fused->inter_hi, fused->inter_lo, fused->intra_hi_frag,
                       fused->intra_lo_frag, fused->A_q, fused->A_s, W_q, W_s, reinterpret_cast<uint16_t *>(out), (int)M,
                       N, d, fused->P, (int)groups, fused->ctr, fused->spin_limit, fused->raise_ready);
    return hipGetLastError();
  }
  // The persistent form (activation codes loaded once per workgroup and kept in registers): 8 - 16 rows,
  // one trip over the k range, and weights enough for the re-reads to cost more than the parallelism
  // given up (measured: [16, 8192] x 28672 34.2 -> 28.4 us, [8, 8192] x 28672 32.2 -> 27.4,
  // [16, 4096] x 14336 9.2 -> 9.0; below 24 MB of weights it loses.  With 16-byte aligned scale rows d = 2560 ... 8192 go to the
  // ring of strips or to whole lines; left are d up to 2048, rows that are no whole pieces and scale rows elsewhere).  Each
  // workgroup takes `per` groups, the smallest power of two that leaves at most 256 workgroups (one per CU,
  // evenly loaded: 3 or 7 groups per workgroup measured 15 - 20 % slower than 4, and half as many
  // workgroups as CUs 30 % slower than one each).
  const int KP = (d / 128 + 1) / 2;
  // the scale bytes by units of 16 where their rows allow it and the LDS has room for the wider padding
  const bool by16 = rows16(A_s, W_s, d);
  const size_t red_bytes = skinny_red_bytes(MT, NS);
  if constexpr (MT == 1) if (M >= 8 && KP <= PT * WAVES && (double)N * (double)d * 0.53125 >= 24e6 && scale_bytes + red_bytes <= 64 * 1024) {
    const size_t p_wide = skinny_scale_bytes(MT, NS, d, 16) + red_bytes;
    const bool wide = by16 && p_wide <= 64 * 1024;
    const size_t p_bytes = wide ? p_wide : scale_bytes + red_bytes;
    int64_t per = 1;
    while ((groups + per - 1) / per > 256) per *= 2;
    if (per > 1) {
      const int64_t grid = (groups + per - 1) / per;
      hipLaunchKernelGGL((mxfp4_gemm_skinny_kernel<MT, NS, PT, true>), dim3((unsigned)grid), dim3(64 * WAVES), p_bytes,
                         stream, A_q, A_s, W_q, W_s, reinterpret_cast<uint16_t *>(out), (int)M, N, d, (int)wide);
      return hipGetLastError();
    }
  }
  const bool wide = by16 && skinny_lds_bytes(MT, NS, d, 16) <= SKINNY_MAX_LDS;
  if (wide) lds_bytes = skinny_lds_bytes(MT, NS, d, 16);
  if (lds_bytes > SKINNY_MAX_LDS) return hipErrorInvalidValue;
  if (lds_bytes > 64 * 1024) {
    static std::atomic<uint64_t> raised{0};
    const hipError_t e =
        raise_lds_limit(reinterpret_cast<const void *>(mxfp4_gemm_skinny_kernel<MT, NS, PT>), SKINNY_MAX_LDS, raised);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((mxfp4_gemm_skinny_kernel<MT, NS, PT>), dim3((unsigned)groups), dim3(64 * WAVES), lds_bytes,
                     stream, A_q, A_s, W_q, W_s, reinterpret_cast<uint16_t *>(out), (int)M, N, d, (int)wide);
  return hipGetLastError();
}

template <int MT, int NS>
static hipError_t launch_mt_ns(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                               void *out, int64_t M, int64_t N, int d, hipStream_t stream, const DecodeArgs *fused) {
  // trip depth: as deep as the k range of a wave goes, at most 4 line pairs (8 k-steps) in flight
  // (2 when the operand registers of a trip would not leave room for several workgroups per CU)
  const int pairs_per_wave = ((d / 128 + 1) / 2 + WAVES - 1) / WAVES;
  if (pairs_per_wave <= 1) return launch_cfg<MT, NS, 1>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
  if (pairs_per_wave <= 2) return launch_cfg<MT, NS, 2>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
  return launch_cfg<MT, NS, (MT + NS <= 3 ? 4 : 2)>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
}

// Strips per workgroup of the weight-streaming GEMM.  Every workgroup reads all activation rows from the L2,
// which from 17 rows on is as many bytes as its weights or more, and a CU that gets a second workgroup
// reads them a second time: the fewest strips that leave every CU at most one workgroup win, since a
// strip more in a workgroup shares those reads and a workgroup more on a CU does not.
// Up to 256 strips: one (x 4096, 24 - 64 rows: two measured 13 - 28 % slower).  Up to 512: two, from 8 rows
// on, against one, us, weights from HBM: [64, 4096] x 4224 14.5 -> 9.6, [16, 8192] x 5120 11.4 -> 9.9,
// [32, 8192] x 5120 17.1 -> 12.0, [64, 8192] x 8192 26.7 -> 18.5, [45, 5120] x 8192 14.3 -> 11.1,
// [32, 25600] x 5120 46.4 -> 32.3, [48, 28672] x 8192 61.4 -> 45.5, [16, 28672] x 8192 34.7 -> 30.6.
// Beyond, from 17 rows on: four (two workgroups a CU past 1024 strips), [32, 8192] x 8448 24.3 -> 18.1,
// [64, 4096] x 12288 22.4 -> 14.8, [48, 5120] x 25600 40.5 -> 30.0.  At 17 - 32 rows the reads saved are fewer, and
// the larger reduction of four strips or a nearly empty second round of them costs more: two from 768
// strips on up to d = 4096 ([17, 4096] x 16384 10.2 against 10.8, [17, 1024] x 14336 5.0 against 5.4) and just
// past 1024 strips, one below 768 strips and d = 2048 ([17, 1024] x 8448 4.7 against 5.1; [32, 3072] x 11264
// gains, 11.4 -> 9.4).  8 - 16 rows beyond 512 strips: two from 768 strips on, mostly in the persistent form
// (two against four, [16, 8192] x 28672 28.8 / 32.3; below 768 strips two, with trips of four, have measured ahead too,
// [16, 8192] x 8448 15.5 -> 14.1, and are not taken yet); 1 - 7 rows re-read too little to gain.
int mxfp4_gemm_skinny_strips(int64_t M, int64_t N, int d) {
  const int MT = (int)((M + 15) / 16);
  const int64_t strips = (N + 15) / 16;
  int NS = 1;
  if (M >= 8 && strips > 256 && strips <= 512) NS = 2;
  else if (MT == 1) NS = M >= 8 && strips >= 2 * SKINNY_MIN_GROUPS ? 2 : 1;
  else if (strips > 512) {
    if (MT == 2 && strips >= 2 * SKINNY_MIN_GROUPS && (d <= 4096 || (strips > 1024 && strips <= 1280))) NS = 2;
    else NS = MT == 2 && d < 2048 ? 1 : 4;
  }
  while (NS > 1 && skinny_lds_bytes(MT, NS, d) > SKINNY_MAX_LDS) NS /= 2;
  return NS;
}

template <int MT>
static hipError_t launch_mt(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                            void *out, int64_t M, int64_t N, int d, hipStream_t stream, const DecodeArgs *fused) {
  if (fused) {
    // the decode form's consumers: two strips where there are workgroups enough
    if (MT <= 2 && M >= 8 && (N + 15) / 16 >= 2 * SKINNY_MIN_GROUPS)
      return launch_mt_ns<MT, (MT <= 2 ? 2 : 1)>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
    return launch_mt_ns<MT, 1>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
  }
  if (const int lines = rows16(A_s, W_s, d) ? mxfp4_gemm_lines_strips(M, N, d) : 0)
    return launch_lines_mt<MT>(lines, A_q, A_s, W_q, W_s, out, M, N, d, stream);
  const int NS = mxfp4_gemm_skinny_strips(M, N, d);
  const int pairs_per_wave = ((d / 128 + 1) / 2 + WAVES - 1) / WAVES;
  if constexpr (MT >= 2) {
    // four strips: a deeper trip measured 1 - 8 % slower (64 accumulators and the weights leave no room)
    if (NS == 4) return launch_cfg<MT, 4, 1>(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
  }
  if (NS == 2) {
    // one trip of four pairs where it covers the k range exactly (d about 8192: [45, 8192] x 8192 15.6 -> 14.5 us
    // against two trips of two; at 64 rows 18.4 -> 20.3, its registers), else trips of two
    if (pairs_per_wave <= 1) return launch_cfg<MT, 2, 1>(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
    if constexpr (MT <= 3) {
      if (pairs_per_wave == 4) return launch_cfg<MT, 2, 4>(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
    }
    if constexpr (MT == 1) {
      // past 512 strips: the depth that lets the persistent form cover the k range
      if (pairs_per_wave > 2 && (N + 15) / 16 > 512)
        return launch_cfg<MT, 2, 4>(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
    }
    return launch_cfg<MT, 2, 2>(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
  }
  return launch_mt_ns<MT, 1>(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
}

// Whether the scale rows of (up to two) strips and of the activations fit the LDS.
bool mxfp4_gemm_skinny_fits(int64_t M, int d) {
  const int MT = (int)((M + 15) / 16), NS = MT <= 2 ? 2 : 1;
  const int pd = d / 128 + 1;
  return M >= 1 && M <= 64 &&
         (size_t)((16 * NS * pd + 63) / 64 + (16 * MT * pd + 63) / 64) * 256 <= SKINNY_MAX_LDS;
}

// 1 <= M <= 64; d a multiple of 128 with 64 rows of d / 2 bytes addressable in 32 bits (the caller
// checks both) and mxfp4_gemm_skinny_fits(M, d).
static hipError_t launch_by_rows(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q, const uint8_t *W_s,
                                 void *out, int64_t M, int64_t N, int d, hipStream_t stream, const DecodeArgs *fused) {
  switch ((M + 15) / 16) {
    case 1: return launch_mt<1>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
    case 2: return launch_mt<2>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
    case 3: return launch_mt<3>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
    case 4: return launch_mt<4>(A_q, A_s, W_q, W_s, out, M, N, d, stream, fused);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_mxfp4_gemm_skinny(const uint8_t *A_q, const uint8_t *A_s, const uint8_t *W_q,
                                    const uint8_t *W_s, void *out, int64_t M, int64_t N, int d,
                                    hipStream_t stream) {
  return launch_by_rows(A_q, A_s, W_q, W_s, out, M, N, d, stream, nullptr);
}

// torq_linear in one launch (torq_linear_single_launch); the caller has checked G = 128, a dense R_inter,
// 1 <= M <= 64, mxfp4_gemm_skinny_fits(M, r->d) and N > 0.  A_q / A_s: the workspace's code and scale areas.
hipError_t launch_torq_linear_decode(const torq_rotation *r, const void *x_bf16, uint8_t *A_q, uint8_t *A_s,
                                     const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M, int64_t N,
                                     int spin_limit, int raise_ready, hipStream_t stream) {
  DecodeArgs fz;
  fz.x = reinterpret_cast<const uint4 *>(x_bf16);
  fz.TG = M * (int64_t)(r->d / 32 / r->G);
  fz.inter_hi = reinterpret_cast<const uint4 *>(r->inter32f_hi);
  fz.inter_lo = reinterpret_cast<const uint4 *>(r->inter32f_lo);
  fz.intra_hi_frag = reinterpret_cast<const uint4 *>(r->intra32_hi);
  fz.intra_lo_frag = reinterpret_cast<const uint4 *>(r->intra32_lo);
  fz.A_q = A_q;
  fz.A_s = A_s;
  fz.P = (int)fz.TG;                               // one token-group per rotating workgroup
  fz.ctr = r->decode_ctr;
  fz.spin_limit = spin_limit;
  fz.raise_ready = raise_ready;
  return launch_by_rows(A_q, A_s, W_q, W_s, out, M, N, r->d, stream, &fz);
}

// torq_linear with the activations rotated and quantised inside every workgroup (torq_linear_local_kernel).
// Preconditions (torq_linear_local_fits): dense R_inter with 96 < G <= 128, at most LOCAL_MAX_TG
// token-groups in all, d a multiple of 128, and LDS for one strip per workgroup.
static size_t local_lds_bytes(int64_t M, int d, int NS) {
  const int pd = d / 128 + 1;
  const size_t red = (size_t)WAVES * NS * 4 * 64 * sizeof(float), rot = LOCAL_MAX_TG * (size_t)RotCfg<4>::TG_LDS_BYTES;
  return (size_t)((16 * NS * pd + 63) / 64 + (16 * pd + 63) / 64) * 256 + ((size_t)M * (d / 2 + 16) + 255) / 256 * 256 +
         (red > rot ? red : rot);
}

bool torq_linear_local_fits(const torq_rotation *r, int64_t M) {
  if (r->butterfly || r->G <= 96 || r->G > 128 || r->G % 16 != 0 || r->d % 128 != 0) return false;
  if (M < 1 || M > 16) return false;
  if (M * (int64_t)(r->d / 32 / r->G) > LOCAL_MAX_TG) return false;
  return (r->d / 128 + 1) / 2 <= 8 * WAVES * 4 && local_lds_bytes(M, r->d, 1) <= 64 * 1024;
}

// Where the one-launch form is the faster way through torq_linear: one or two token-groups up to 20 MB of packed
// weights, three or four up to 16 MB.  Measured against rotate + quantise followed by the GEMM with weights from HBM (copies
// of 600 MB in all; with six copies of a 31 MB layer the 256 MB Infinity Cache held them, and the form seemed to
// pay up to 48 MB).  One launch against two, us, HIP-graph replays: [1, 4096] x 1024 5.9 / 6.9, x 4096 6.3 / 7.4, x 8192
// 8.3 / 9.0, x 11008 11.2 / 9.9, x 14336 11.4 / 10.7; [1, 8192] x 4096 8.9 / 9.2, x 8192 12.2 / 11.6.  Three or four token-groups are within a launch's gap of each other, and which is ahead depends on who waits:
// replayed, [4, 4096] x 1024 7.1 / 7.2, x 4096 8.4 / 7.6, [2, 8192] x 2048 8.7 / 8.1, [1, 14336] x 2048 (G = 112)
// 10.7 / 9.5; called one after the other from Python, where a launch more is 3 us of the host, 7.0 / 10.0, 7.0 / 10.0,
// 7.7 / 8.6 and 10.6 / 9.1 with buffers kept by the caller, 10.3 / 13.4, 10.3 / 13.3, 9.6 / 12.3 and 10.6 / 12.1 without.
// (Where the strips come through a ring, mxfp4_gemm_stream.hip, one launch is ahead of two at any size that form takes.)
bool torq_linear_local_pays(const torq_rotation *r, int64_t M, int64_t N, const uint8_t *W_s) {
  if (!torq_linear_local_fits(r, M) || N <= 0) return false;
  if (torq_linear_stream_takes(r, M, N, W_s)) return true;
  const int64_t token_groups = M * (int64_t)(r->d / 32 / r->G);
  return (double)N * (double)r->d * 0.53125 <= (token_groups <= 2 ? 20e6 : 16e6);
}

template <int NS, int PT>
static hipError_t launch_local_cfg(const torq_rotation *r, const void *x_bf16, uint8_t *A_q, uint8_t *A_s,
                                   const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M, int64_t N,
                                   hipStream_t stream) {
  const int d = r->d;
  const int64_t groups = (N + 16 * NS - 1) / (16 * NS);
  // as for the persistent GEMM: the smallest power of two of groups per workgroup that leaves at most
  // 256 workgroups, so that every workgroup has the same share
  int64_t per = 1;
  while ((groups + per - 1) / per > 256) per *= 2;
  const int64_t grid = (groups + per - 1) / per;
  const bool exact = d % 256 == 0 && d / 256 == PT * WAVES;
  auto kernel = exact ? torq_linear_local_kernel<NS, PT, true> : torq_linear_local_kernel<NS, PT, false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * WAVES), local_lds_bytes(M, d, NS), stream,
                     reinterpret_cast<const uint4 *>(x_bf16), (int)(M * (int64_t)(d / 32 / r->G)), r->G,
                     reinterpret_cast<const uint4 *>(r->inter32f_hi), reinterpret_cast<const uint4 *>(r->inter32f_lo),
                     reinterpret_cast<const uint4 *>(r->intra32_hi),
                     reinterpret_cast<const uint4 *>(r->intra32_lo), A_q, A_s, W_q, W_s,
                     reinterpret_cast<uint16_t *>(out), (int)M, N, d);
  return hipGetLastError();
}

hipError_t launch_torq_linear_local(const torq_rotation *r, const void *x_bf16, uint8_t *A_q, uint8_t *A_s,
                                    const uint8_t *W_q, const uint8_t *W_s, void *out, int64_t M, int64_t N,
                                    hipStream_t stream) {
  if (!torq_linear_local_fits(r, M) || N <= 0) return hipErrorInvalidValue;
  if (torq_linear_stream_takes(r, M, N, W_s)) return launch_torq_linear_stream(r, x_bf16, A_q, A_s, W_q, W_s, out, M, N, stream);
  // PT: the line pairs of a wave, so that one trip covers the k range (at most 8); NS: as many strips per
  // workgroup as leave every CU a workgroup, within the registers (NS PT <= 8: 128 for the weight codes
  // of a trip) and the LDS
  const int pairs_per_wave = ((r->d / 128 + 1) / 2 + WAVES - 1) / WAVES;
  const int PT = pairs_per_wave <= 8 ? pairs_per_wave : 8;
  const int64_t strips = (N + 15) / 16;
  int NS = 1;
  while (NS < 4 && strips > 256 * NS && 2 * NS * PT <= 8 && local_lds_bytes(M, r->d, 2 * NS) <= 64 * 1024) NS *= 2;
#define TORQ_LOCAL_CASE(NS_, PT_) \
  if (NS == NS_ && PT == PT_) return launch_local_cfg<NS_, PT_>(r, x_bf16, A_q, A_s, W_q, W_s, out, M, N, stream);
  TORQ_LOCAL_CASE(1, 1) TORQ_LOCAL_CASE(1, 2) TORQ_LOCAL_CASE(1, 3) TORQ_LOCAL_CASE(1, 4)
  TORQ_LOCAL_CASE(1, 5) TORQ_LOCAL_CASE(1, 6) TORQ_LOCAL_CASE(1, 7) TORQ_LOCAL_CASE(1, 8)
  TORQ_LOCAL_CASE(2, 1) TORQ_LOCAL_CASE(2, 2) TORQ_LOCAL_CASE(2, 3) TORQ_LOCAL_CASE(2, 4)
  TORQ_LOCAL_CASE(4, 1) TORQ_LOCAL_CASE(4, 2)
#undef TORQ_LOCAL_CASE
  return hipErrorInvalidValue;
}

// every counter of a handle back to zero, the error word included (a fill kernel rather than a
// memset node, so that the call may sit in a captured graph)
__global__ void __launch_bounds__(256) decode_ctr_reset_kernel(unsigned *__restrict__ ctr) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < DECODE_CTR_WORDS) ctr[i] = 0u;
}

hipError_t launch_decode_ctr_reset(const torq_rotation *r, hipStream_t stream) {
  hipLaunchKernelGGL(decode_ctr_reset_kernel, dim3((DECODE_CTR_WORDS + 255) / 256), dim3(256), 0, stream, r->decode_ctr);
  return hipGetLastError();
}

}  // namespace torq
