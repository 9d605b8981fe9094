// keepkv_match: nearest retained key by cosine similarity for every to-be-evicted key
// (Alg. 1, matching step), the one dense contraction of the method.
//
// bf16 caches, first event (thousands of evicted rows per head): the retained keys of a head are first
// gathered into a panel in list order; one workgroup of 8 wavefronts per compute unit then walks blocks of
// 512 evicted rows in passes.  Each wavefront keeps its 64 rows (two 32-row MFMA operands over the whole
// head dimension) in registers for a pass and the panel streams through LDS in 128-column stages.
// Every 32x32 f32 accumulator tile is reduced on the spot (scale by 1/|k_c|, running maxima); the
// similarity matrix is never written.  Steady state (one period's worth of evicted rows): a workgroup
// of 8 wavefronts per 64 rows, the columns split over the wavefronts (and, with few heads, over up to
// four such workgroups that join their results through a ticket).
//
// Exactness: the f32 result decides a row only when the best value leads the second by more than
// the rounding envelope and is away from the threshold by as much; all other rows (a fraction of a
// percent) are queued and re-evaluated in f64, where products of bf16 or f32 values are exact and
// the sum is taken in channel order.  f32 caches go through the f64 kernel entirely.
#include "kk_common.hpp"

namespace kk {
// Phase timestamps for kernel tuning; compiled in only with -DKEEPKV_TRACE (never in the product build).
#ifdef KEEPKV_TRACE
// per workgroup: [0] start, [1] first loop start, [2] first loop end, [3] first loop's shader cycles,
// [4..7] end of pass 0..3 (100 MHz wall clock except [3])
__device__ long long kk_trace_match[8 * 2048];
#define KX_TS(i) do { const int b_ = blockIdx.x; if (threadIdx.x == 0 && b_ < 2048) \
  kk_trace_match[b_ * 8 + (i)] = wall_clock64(); } while (0)
#define KX_CYC(i, v) do { const int b_ = blockIdx.x; if (threadIdx.x == 0 && b_ < 2048) \
  kk_trace_match[b_ * 8 + (i)] = (v); } while (0)
// the steady-state kernel: indexed by head
#define KS_TS(i) do { if (threadIdx.x == 0 && blockIdx.y < 256) kk_trace_match[blockIdx.y * 8 + (i)] = wall_clock64(); } while (0)
#else
#define KX_TS(i) do { } while (0)
#define KX_CYC(i, v) do { } while (0)
#define KS_TS(i) do { } while (0)
#endif
namespace {

constexpr int kRowsPerWave = 64;
constexpr int kMWaves = 8;                              // wavefronts per workgroup of the first event's kernel
constexpr int kStageCols = 128;                         // retained keys per LDS stage
constexpr unsigned kResidentWorkgroups = 256;           // of the first event's kernel: one on each of 256 compute units
constexpr int kXcds = 8;                                // accelerator dies, each with its own L2

// ---------------------------------------------------------------------------------------------------
// The f32 similarities are good to their margin while both |k|^2 lie in this range: above it sums of squares and
// products come near the end of the f32 range, below it a product's terms may fall under 2^-126 (at most 128 of them,
// 2^-119 against |k_e||k_c| >= 2^-80, a relative 2^-39).  A row outside it is evaluated in f64 against every column, a
// column outside it makes every row that sees it do so (1/|k_c| is NaN then; zero keys match nothing and have 0).
constexpr float kNormLeast = 0x1p-80f, kNormMost = 0x1p100f;
__device__ __forceinline__ bool norm_in_range(float ss) { return ss >= kNormLeast && ss <= kNormMost; }   // (NaN: no)
// 1/|k_c| of a column from |k_c|^2; nonzero: some element of the key is not 0
__device__ __forceinline__ float column_rnorm(float ss, bool nonzero) {
  return norm_in_range(ss) ? 1.0f / sqrtf(ss) : (nonzero ? __builtin_nanf("") : 0.f);
}
// Whether some element of the row of LPS lanes is not 0; x: this lane's 16 bytes.
template <typename T, int LPS>
__device__ __forceinline__ bool row_nonzero(const uint4& x) {
  const uint32_t magnitudes = sizeof(T) == 2 ? 0x7FFF7FFFu : 0x7FFFFFFFu;
  return group_sum<LPS>(((x.x | x.y | x.z | x.w) & magnitudes) != 0 ? 1.f : 0.f) > 0.f;
}

// 1/|k_c| (f32) of every retained key; 0 for padding and for zero keys, NaN where f32 cannot hold the norm.  With `panel`, the retained keys are
// also copied there in list order, rn_pitch rows per head (padding rows zero), each row with its 16-byte
// chunk c stored at position c ^ (row mod chunks): the LDS image that the first event's kernel wants, so
// that its stage loads are straight copies that need no slot index.
constexpr int kRnormRows = 4;
template <typename T, int D>
__global__ __launch_bounds__(256) void rnorm_kernel(const T* __restrict__ k, const int32_t* __restrict__ keep_idx,
                                                    const int32_t* __restrict__ n_evict, float* __restrict__ rnorm,
                                                    int capacity, int budget, int rn_pitch, uint4* __restrict__ panel) {
  constexpr int EPL = 16 / (int)sizeof(T), LPS = D / EPL, RPB = 256 / LPS;
  const int unit = blockIdx.y;
  const int sub = threadIdx.x % LPS;
  // kRnormRows rows per lane group, all requested before the first wait (slot numbers beside the head's
  // eviction count, then the rows)
  int r[kRnormRows], slot[kRnormRows];
#pragma unroll
  for (int i = 0; i < kRnormRows; ++i) {
    r[i] = (blockIdx.x * kRnormRows + i) * RPB + threadIdx.x / LPS;
    slot[i] = r[i] < budget ? keep_idx[(size_t)unit * budget + r[i]] : -1;
  }
  if (n_evict[unit] <= 0) return;
  uint4 x[kRnormRows];
#pragma unroll
  for (int i = 0; i < kRnormRows; ++i) {
    x[i] = make_uint4(0, 0, 0, 0);
    if (slot[i] >= 0) x[i] = reinterpret_cast<const uint4*>(k)[((size_t)unit * capacity + slot[i]) * LPS + sub];
  }
#pragma unroll
  for (int i = 0; i < kRnormRows; ++i) {
    if (r[i] >= rn_pitch) continue;              // whole lane groups
    float ss = 0.f;
    if constexpr (sizeof(T) == 2) {
      const uint32_t w[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = bf16_lo(w[e]), b = bf16_hi(w[e]);
        ss = fmaf(a, a, ss);
        ss = fmaf(b, b, ss);
      }
    } else {
      const float w[4] = {__builtin_bit_cast(float, x[i].x), __builtin_bit_cast(float, x[i].y),
                          __builtin_bit_cast(float, x[i].z), __builtin_bit_cast(float, x[i].w)};
#pragma unroll
      for (int e = 0; e < 4; ++e) ss = fmaf(w[e], w[e], ss);
    }
    if (panel != nullptr) panel[((size_t)unit * rn_pitch + r[i]) * LPS + (sub ^ (r[i] & (LPS - 1)))] = x[i];
    ss = group_sum<LPS>(ss);
    // positions budget .. rn_pitch - 1 are padding: zero, so padded columns score 0; so do zero keys and
    // negative slot numbers
    const bool nonzero = norm_in_range(ss) || row_nonzero<T, LPS>(x[i]);   // (whole lane groups)
    if (sub == 0) rnorm[(size_t)unit * rn_pitch + r[i]] = column_rnorm(ss, nonzero);
  }
}

// ---------------------------------------------------------------------------------------------------
struct ExactPartial;
struct MatchParams {
  const void* k;
  const int32_t* keep_idx;
  const int32_t* evict_idx;
  const int32_t* n_evict;
  const float* rnorm;
  const unsigned char* panel;   // retained keys in list order, rows pre-swizzled (first event's kernel only)
  int32_t* match;
  float* sim_out;
  struct ExactPartial* exact_partial;   // [kExactResident] per-share results of the f64 kernel
  int32_t* exact_ticket;                // control words at the head of the workspace
  int32_t* flag_count;   // [1] rows queued for the f64 kernel; zero between calls (the f64 kernel clears it)
  int32_t* exact_done;   // [1] queued rows that the f64 kernel has finished; zero between calls
  int32_t* flag_rows;    // [units * max_evict]: unit * max_evict + j
  uint32_t* flag_cols;   // [units * max_evict]: the queued row's candidate columns, bit o for the columns 32 b + o
                         // (first event and prefill pass; the steady-state kernel's rows are re-checked against all columns)
  int capacity, budget, max_evict, rn_pitch;
  float threshold, delta;
  int per_unit, n_units;   // first event's kernel: workgroups per head, heads
  int causal;              // prefill pass: row j is slot j and its columns are the slots before it (no lists)
  const int32_t* len;      // prefill pass: live slots per head
  int small_parts;         // steady-state kernel: workgroups that share the retained list of one 64-row block
  int32_t* small_partial;  // [row blocks * small_parts][64][3] their per-row results
};

__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }
// median of three; the backend folds this into v_med3_i32
__device__ __forceinline__ int imed3(int a, int b, int c) { return imax(imin(a, b), imin(imax(a, b), c)); }

// A row whose best cosine lies below the threshold by more than the f32 arithmetic's error has no target
// whichever column holds that best value, so neither a small margin to the runner-up nor a best value that
// is not positive (`upper` is then 0: every value of the row is at most 0) makes it undecided, as long as
// the caller does not ask for the similarity itself.  A NaN in `upper` compares false and keeps the row queued.
__device__ __forceinline__ bool surely_below(const MatchParams& p, float upper, float ss, float rn_e) {
  return p.sim_out == nullptr && ss > 0.f && rn_e < INFINITY && upper + p.delta < p.threshold;
}

// Decision of one row from the integer images of its best value v1 (column c1) and of an upper bound v2 of
// every other column's value, both still lacking the factor 1/|k_e| (ss = |k_e|^2); a row that the f32
// arithmetic cannot decide is queued for the f64 kernel.
__device__ __forceinline__ void decide_row(const MatchParams& p, int unit, int j, int v1, int c1, int v2, float ss) {
  const float rn_e = 1.0f / sqrtf(ss);
  const float y1 = __builtin_bit_cast(float, v1), y2 = (v2 > 0) ? __builtin_bit_cast(float, v2) : 0.f;
  const float cos1 = y1 * rn_e;
  bool fragile = !(v1 > 0) || !((y1 - y2) * rn_e > p.delta) || !(fabsf(cos1 - p.threshold) > p.delta) || c1 >= p.budget;
  if (surely_below(p, (v1 > 0) ? cos1 : 0.f, ss, rn_e)) fragile = false;
  if (!norm_in_range(ss)) fragile = true;
  const size_t o = (size_t)unit * p.max_evict + j;
  p.match[o] = (cos1 > p.threshold) ? c1 : -1;
  if (p.sim_out != nullptr) p.sim_out[o] = cos1;
  if (fragile) {
    const int at = atomicAdd(p.flag_count, 1);
    p.flag_rows[at] = (int)o;
  }
}

// f32 decision of one row from its best value y1 (column c1) and an upper bound y2 of every other column's
// value, both still lacking the factor 1/|k_e|.  Returns whether the f32 arithmetic cannot decide the row, which the
// caller then queues.
__device__ __forceinline__ bool decide_row_f32(const MatchParams& p, size_t o, float y1, int c1, float y2, float ss, int n_cols) {
  const float rn_e = 1.0f / sqrtf(ss);
  const float cos1 = y1 * rn_e;
  bool fragile = !(y1 > 0.f) || !((y1 - y2) * rn_e > p.delta) || !(fabsf(cos1 - p.threshold) > p.delta) || c1 >= n_cols;
  if (surely_below(p, (y1 <= 0.f) ? 0.f : cos1, ss, rn_e)) fragile = false;
  if (!norm_in_range(ss)) fragile = true;
  p.match[o] = (cos1 > p.threshold) ? c1 : -1;
  if (p.sim_out != nullptr) p.sim_out[o] = cos1;
  return fragile;
}

// The columns that can hold a row's true best value, as a mask over the column number modulo 32: those whose column
// class has an f32 best within the margin of the row's best (the rule by which a row without a close runner-up is
// decided, a little wider for the rounding of `lim`).  cls: this lane's 16 classes, columns 8 (i / 4) + 4 half + i % 4
// of every block; the lanes l and l ^ 32 hold the two halves.  A row of a few hundred columns has two or three candidate
// classes as a rule, so the f64 kernel has a tenth of its columns or less to look at.  A norm out of range or a NaN: all
// columns.
__device__ __forceinline__ uint32_t candidate_columns(const MatchParams& p, const int (&cls)[16], float y1, float ss, int half) {
  const float lim = norm_in_range(ss) ? y1 - 1.01f * p.delta * sqrtf(ss) : -INFINITY;
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    m |= (!(__builtin_bit_cast(float, cls[i]) < lim) ? 1u : 0u) << (8 * (i / 4) + (i % 4));
  m <<= 4 * half;
  return m | (uint32_t)__shfl_xor((int)m, 32);
}

// The first event's kernel.  The product is taken transposed, retained keys as the A operand and the
// wavefront's evicted rows as B, so that lane (l32, half) holds, for ITS evicted row, the 16 retained columns
// 8 (i / 4) + 4 half + i % 4 of each 32-column block: all values in a lane belong to one row.  Per value the
// fold then costs a multiply by 1/|k_c| and a maximum into the running best of its column class i, plus a
// share of a max3 tree that gives the block's best, which goes into a running (best, second best, block)
// triple.  No column number travels with the values: at the end the winning class is the one whose running
// best equals the overall best, and the winning block is the triple's.  Every other column's value is
// bounded by the second best block value or by the best of the other classes, which is all that the
// exactness test needs.
//
// CAUSAL: the search of the prefill pass (App. B.4), every live slot against the slots before it.  A workgroup takes one
// block of 64 NW consecutive slots as rows.  The slots before the block are plain columns of the loop above, copied from
// the cache itself with the row swizzle applied on the address side; the stages that hold the block's own slots follow,
// with the columns at or behind a row masked and the tiles wholly before the columns skipped.  Long blocks start first
// (the launch order), which evens out the triangle over the compute units.  Bound by the matrix
// pipes and the clock they leave (64 heads x 8192 slots, 550 GFLOP: 990 us with one 32-row operand per wavefront, where
// every fragment read from LDS fed a single MFMA; now 500 us, 1.1 PFLOP/s, which is what a large bf16 matrix product
// of random operands reaches on this part).
template <int D, bool CAUSAL, int NW>
__global__ __launch_bounds__(NW* kWave, 2) void match_mfma_kernel(MatchParams p) {
  constexpr int kRowsPerBlock = kRowsPerWave * NW;   // rows per workgroup and pass
  constexpr int KS = D / 16;                 // MFMA k-steps over the head dimension
  constexpr int ROWB = D * 2;                // bytes per key
  constexpr int CHUNKS = ROWB / 16;          // 16-byte chunks per key
  constexpr int STAGE_BYTES = kStageCols * ROWB;
  constexpr int LOADS = kStageCols * CHUNKS / (NW * kWave);   // async 16-byte loads per lane per stage

  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* s_stage = smem;                                        // 2 stages, swizzled rows
  float* s_rn = reinterpret_cast<float*>(smem + 2 * STAGE_BYTES);       // [2][kStageCols]

  // Workgroups are dealt to the 8 XCDs in turn, each with an L2 of its own.  All workgroups of a head are
  // placed on one XCD (when the heads divide evenly), so that the head's retained keys, which every pass of
  // every one of them streams again, stay in that L2.
  int unit, first_rb;
  {
    const bool even = p.n_units % kXcds == 0;
    const int xcd = even ? blockIdx.x % kXcds : 0, slot = even ? blockIdx.x / kXcds : blockIdx.x;
    const int units = even ? p.n_units / kXcds : p.n_units;          // heads of this die
    if constexpr (CAUSAL) {
      unit = xcd * units + slot % units;
      first_rb = p.per_unit - 1 - slot / units;
    } else {
      unit = xcd * units + slot / p.per_unit;
      first_rb = slot % p.per_unit;
    }
  }
  const int n_ev = CAUSAL ? p.len[unit] : p.n_evict[unit];           // rows
  const int n_rb = (n_ev + kRowsPerBlock - 1) / kRowsPerBlock;
  int rb = first_rb;                         // this pass's block of rows; later passes: rb + per_unit, ...
  if (rb >= n_rb) return;
  KX_TS(0);
  // columns that every row sees (n_evict > 0 implies the retained list is full)
  const int n_keep = CAUSAL ? first_rb * kRowsPerBlock : p.budget;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;

  const unsigned char* kbytes = reinterpret_cast<const unsigned char*>(p.k) + (size_t)unit * p.capacity * ROWB;
  const int32_t* evict = CAUSAL ? nullptr : p.evict_idx + (size_t)unit * p.max_evict;
  const float* rn_c = p.rnorm + (size_t)unit * p.rn_pitch;

  // ---- stage loader: global -> LDS without passing through registers.  The panel holds the head's retained
  // keys in list order with chunk c of key `col` at position c ^ (col mod CHUNKS) of its row, which keeps the
  // MFMA operand reads below free of bank conflicts; a stage is one contiguous piece of it, copied as is.
  // (CAUSAL: the chunk numbers are exchanged within the row; a lane's rows of a stage are a multiple of CHUNKS apart, so
  // its exchanged chunk is the same in all of them.  The last stage may reach beyond the cache and stops at len.)
  const unsigned char* panel = CAUSAL ? kbytes : p.panel + (size_t)unit * p.rn_pitch * ROWB;
  static_assert(!CAUSAL || (NW * kWave / CHUNKS) % CHUNKS == 0, "rows of a lane in a stage");
  const int stage_row = tid / CHUNKS;
  const uint32_t stage_off = CAUSAL ? stage_row * ROWB + ((tid % CHUNKS) ^ (stage_row & (CHUNKS - 1))) * 16 : tid * 16;
  auto issue_stage = [&](int s, int buf) {
    const unsigned char* src = panel + (size_t)s * STAGE_BYTES + stage_off;
    unsigned char* dst = s_stage + buf * STAGE_BYTES + wave * 64 * 16;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const unsigned char* at = src + i * (NW * kWave) * 16;
      if constexpr (CAUSAL) {
        const int beyond = s * kStageCols + stage_row + i * (NW * kWave / CHUNKS) - (n_ev - 1);
        if (beyond > 0) at -= (size_t)beyond * ROWB;
      }
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)at,
                                       (__attribute__((address_space(3))) void*)(dst + i * (NW * kWave) * 16), 16, 0, 0);
    }
    if (wave < kStageCols / 64) {            // 1/|k_c| of the stage's keys (padded with zeros by rnorm_kernel)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(rn_c + (CAUSAL ? min(s * kStageCols + tid, n_ev - 1) : s * kStageCols + tid)),
                                       (__attribute__((address_space(3))) void*)(s_rn + buf * kStageCols + wave * 64),
                                       4, 0, 0);
    }
  };
  int par = 0;                               // LDS buffer of the stage being consumed
  issue_stage(0, 0);

  // ---- B operands: this wavefront's 64 evicted rows of the pass, resident in registers.  The byte offsets
  // of a pass's rows are fetched one pass ahead, the rows themselves as soon as the previous pass has
  // issued its last MFMA, so that their latency overlaps that pass's epilogue.
  // (the slot numbers as loaded: any arithmetic on them would be a first use, and the compiler waits for a
  // load at its first use -- here that is request_rows(), a whole pass later)
  auto row_offset = [&](int rb_, int t) {
    const int j = min(rb_ * kRowsPerBlock + wave * kRowsPerWave + t * 32 + l32, n_ev - 1);
    return CAUSAL ? j : evict[j];
  };
  int row_off[2] = {row_offset(rb, 0), row_offset(rb, 1)};
  bf16x8_t e[2][KS];
  auto request_rows = [&]() {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        e[t][ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(
            kbytes + (uint32_t)row_off[t] * (uint32_t)ROWB + ks * 32 + half * 16));
  };
  request_rows();

  const int n_stage = (n_keep + kStageCols - 1) / kStageCols;
  // CAUSAL: the stages that hold the block's own slots (but not the last one)
  const int n_diag = CAUSAL ? (min(n_ev - n_keep, kRowsPerBlock) + kStageCols - 1) / kStageCols : 0;
  const uint32_t frag0 = l32 * ROWB + (((l32 & (CHUNKS - 1)) ^ half) * 16);
  for (;;) {                                 // one pass per iteration
  float ss_row[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    float ss = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 x = __builtin_bit_cast(uint4, e[t][ks]);
      const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = bf16_lo(w[i]), hi = bf16_hi(w[i]);
        ss = fmaf(lo, lo, ss);
        ss = fmaf(hi, hi, ss);
      }
    }
    ss_row[t] = ss + __shfl_xor(ss, 32);
  }
  // wavefronts whose rows all lie beyond the last one only copy stages
  // (they repeated the last row: with 1024 heads of 7372 rows, 14.4 blocks, the first event took 1 % longer)
  const bool has_rows = rb * kRowsPerBlock + wave * kRowsPerWave < n_ev;
  const int rb_next = rb + p.per_unit;
  const bool more = !CAUSAL && rb_next < n_rb;   // uniform over the workgroup

  // running state per tile: best of each column class, and (best, second best, block) over block maxima.
  // Values are compared through their integer images (for positive floats the order is the same, and a
  // negative one loses to the initial 0): a row without a positive similarity is queued for the f64 kernel
  // anyway, and so is one whose best image is a NaN's.
  int cls[2][16];
  int b1[2] = {0, 0}, b2[2] = {0, 0};
  int g1[2] = {0, 0};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) cls[t][i] = 0;
  // software pipeline: the MFMAs of column block cb are issued together with the fold of block
  // cb - 1.  Two accumulator sets alternate (even blocks write A and fold B, odd blocks the reverse), so
  // no accumulator is ever copied.  The first fold sees zeros and is harmless.
  // rn[g]: 1/|k_c| of the columns of accumulator registers 4g .. 4g+3, for the block being folded; each
  // group is replaced by the next block's as soon as its last value is folded.
  f32x16_t accA0 = {0}, accA1 = {0}, accB0 = {0}, accB1 = {0};
  f32x4_t rn[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) rn[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int cb_prev = 0;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (rb == first_rb) KX_TS(1);
#ifdef KEEPKV_TRACE
  const long long cyc0 = clock64();
#endif
  if (more) {                                // next pass's row offsets: in flight during this pass's first stage
    row_off[0] = row_offset(rb_next, 0);
    row_off[1] = row_offset(rb_next, 1);
  }

  constexpr int VPK = 16 / KS;               // accumulator values folded per k-step and tile
  constexpr int BPS = kStageCols / 32;       // column blocks per stage (even)
  static_assert(BPS % 2 == 0, "the accumulator sets alternate by column block");
  static_assert(VPK == 2 || VPK == 4, "fold_vals handles two or four values per k-step");
  const int n_blk = (n_keep + 31) / 32;

  // values [ks * VPK, (ks + 1) * VPK) of one finished accumulator tile: scale, class maxima, block maximum.  The scaled values of
  // an even block wait in `held` for those of the odd one behind it, and both enter their classes with one instruction.
  // (Not in the first event's kernel of D 128, whose 256 registers do not hold them: with 56 bytes of spills it took 193 us
  // instead of 186 for the batch-8 first event.  The prefill search of 64 heads x 8192 slots gains 6 us of 495, 24 heads x 4500 rows of D 64 0.7 of 16.)
  constexpr bool kHold = CAUSAL || D == 64;
  int held[2][16];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) held[t][i] = 0;
  auto fold_vals = [&](int ks, bool hold, const f32x16_t& od, int (&c)[16], int (&h)[16], int& gm) {
#pragma unroll
    for (int i = ks * VPK; i < (ks + 1) * VPK; i += 2) {
      const int k0 = __builtin_bit_cast(int, od[i] * rn[i / 4][i % 4]);
      const int k1 = __builtin_bit_cast(int, od[i + 1] * rn[(i + 1) / 4][(i + 1) % 4]);
      if (!kHold) {
        c[i] = imax(c[i], k0);
        c[i + 1] = imax(c[i + 1], k1);
      } else if (hold) {
        h[i] = k0;
        h[i + 1] = k1;
      } else {
        asm("v_max3_i32 %0, %1, %2, %3" : "=v"(c[i]) : "v"(c[i]), "v"(h[i]), "v"(k0));
        asm("v_max3_i32 %0, %1, %2, %3" : "=v"(c[i + 1]) : "v"(c[i + 1]), "v"(h[i + 1]), "v"(k1));
      }
      if (i == 0) gm = imax(k0, k1);
      else asm("v_max3_i32 %0, %1, %2, %3" : "=v"(gm) : "v"(gm), "v"(k0), "v"(k1));   // kept in this order
    }
  };
  auto fold_group = [&](int gm, int ocb, int& v1, int& v2, int& blk) {
    blk = (gm > v1) ? ocb : blk;
    v2 = imed3(v1, v2, gm);
    v1 = imax(v1, gm);
  };

  for (int s = 0; s < n_stage; ++s) {
    if (CAUSAL || s + 1 < n_stage) issue_stage(s + 1, par ^ 1);
    else if (more) issue_stage(0, par ^ 1);                   // the next pass starts over at the first columns
    // operand fragment of key 32 cbl + l32: chunk (2 ks + half) ^ (l32 mod CHUNKS) of its row, which is the
    // lane's chunk of k-step 0 with 32 ks XORed into the byte offset
    const uint32_t frag_cur = frag0 + par * STAGE_BYTES;
    auto frag = [&](int cbl, int ks) {
      return *reinterpret_cast<const bf16x8_t*>(s_stage + ((frag_cur ^ (uint32_t)(ks * 32)) + cbl * 32 * ROWB));
    };
    bf16x8_t bq = frag(0, 0);
    // Explicit interleave: each MFMA is followed by the fold of VPK values of the previous column
    // block, and nothing may be scheduled across the fences, so the matrix pipe and the vector ALU of
    // this wavefront run side by side.
    auto block = [&](int cbl, bool hold, f32x16_t& nw0, f32x16_t& nw1, const f32x16_t& od0, const f32x16_t& od1) {
      const f32x16_t zero = {0};
      // 1/|k_c| of the 16 columns that this lane's accumulator registers hold in block cbl
      const f32x4_t* rn_src = reinterpret_cast<const f32x4_t*>(s_rn + par * kStageCols + cbl * 32 + 4 * half);
      int gm0 = 0, gm1 = 0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        // (requested ahead of the operand fragment: the wait for that one then does not wait for a younger request too;
        // 1024 heads x 7372 x 820 1.2 % faster, as are the other shapes)
        if (ks > 0 && (ks * VPK) % 4 == 0) rn[(ks * VPK) / 4 - 1] = rn_src[2 * ((ks * VPK) / 4 - 1)];
        const bf16x8_t bnext = (ks + 1 < KS) ? frag(cbl, ks + 1) : frag((cbl + 1) % BPS, 0);
        nw0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq, e[0][ks], ks == 0 ? zero : nw0, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fold_vals(ks, hold, od0, cls[0], held[0], gm0);
        __builtin_amdgcn_sched_barrier(0);
        nw1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq, e[1][ks], ks == 0 ? zero : nw1, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fold_vals(ks, hold, od1, cls[1], held[1], gm1);
        __builtin_amdgcn_sched_barrier(0);
        bq = bnext;
      }
      rn[3] = rn_src[6];
      fold_group(gm0, cb_prev, b1[0], b2[0], g1[0]);
      fold_group(gm1, cb_prev, b1[1], b2[1], g1[1]);
    };
#pragma unroll
    for (int cbl = 0; cbl < BPS; ++cbl) {
      const int cb = s * BPS + cbl;                           // global column block
      if (cb < n_blk && has_rows) {                           // uniform over the wavefront
        if (cbl % 2 == 0) block(cbl, false, accA0, accA1, accB0, accB1);
        else block(cbl, true, accB0, accB1, accA0, accA1);
        cb_prev = cb;
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    par ^= 1;
  }
  if (rb == first_rb) { KX_TS(2); KX_CYC(3, clock64() - cyc0); }
  if (more) request_rows();                                   // the operand registers are free: next pass's rows
  {                                                           // the last block is still unfolded
    const bool even_last = (n_blk & 1) != 0;
    int gm0 = 0, gm1 = 0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (even_last) {
        fold_vals(ks, false, accA0, cls[0], held[0], gm0);
        fold_vals(ks, false, accA1, cls[1], held[1], gm1);
      } else {
        fold_vals(ks, false, accB0, cls[0], held[0], gm0);
        fold_vals(ks, false, accB1, cls[1], held[1], gm1);
      }
    }
    fold_group(gm0, cb_prev, b1[0], b2[0], g1[0]);
    fold_group(gm1, cb_prev, b1[1], b2[1], g1[1]);
  }

  if constexpr (CAUSAL) {                                     // the block's own slots as columns
    for (int sd = 0; sd < n_diag; ++sd) {
      if (sd + 1 < n_diag) issue_stage(n_stage + sd + 1, par ^ 1);
#pragma unroll
      for (int cbl = 0; cbl < BPS; ++cbl) {
        const int col0 = sd * kStageCols + 32 * cbl;          // block of columns and tile of rows, within the block of slots
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int row0 = wave * kRowsPerWave + t * 32;
          if (col0 > row0) continue;                          // uniform over the wavefront: nothing before a row
          f32x16_t acc = {0};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(
                s_stage + (((frag0 + par * STAGE_BYTES) ^ (uint32_t)(ks * 32)) + cbl * 32 * ROWB));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, e[t][ks], acc, 0, 0, 0);
          }
          int gm = 0;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4_t rn4 = *reinterpret_cast<const f32x4_t*>(s_rn + par * kStageCols + cbl * 32 + 4 * half + 8 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              int k = __builtin_bit_cast(int, (float)(acc[4 * g + i] * rn4[i]));
              if (col0 == row0) k = 8 * g + 4 * half + i < l32 ? k : 0;   // the tile on the diagonal: earlier columns only
              cls[t][4 * g + i] = imax(cls[t][4 * g + i], k);
              gm = imax(gm, k);
            }
          }
          fold_group(gm, (n_keep + col0) >> 5, b1[t], b2[t], g1[t]);
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      par ^= 1;
    }
  }

  // ---- finish: winning class per tile, then the two lanes of a row (the halves) meet ----------------
  float y1[2], y2[2];
  int c1[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int s1 = cls[t][0], s2 = 0, ci = 0;
#pragma unroll
    for (int i = 1; i < 16; ++i) {
      const int x = cls[t][i];
      const bool up = x > s1;
      s2 = up ? s1 : imax(s2, x);
      ci = up ? i : ci;
      s1 = up ? x : s1;
    }
    // s1 equals b1[t]: both are the largest value of this lane's half of the row
    const int col = 32 * g1[t] + 8 * (ci / 4) + 4 * half + (ci % 4);
    const int rest = imax(b2[t], s2);                         // bounds every other column of this half
    const int o1 = __shfl_xor(s1, 32), orest = __shfl_xor(rest, 32), ocol = __shfl_xor(col, 32);
    y1[t] = __builtin_bit_cast(float, imax(s1, o1));
    c1[t] = (s1 > o1) ? col : ((o1 > s1) ? ocol : min(col, ocol));
    y2[t] = __builtin_bit_cast(float, imax(imax(rest, orest), imin(s1, o1)));
  }
  const int j = rb * kRowsPerBlock + wave * kRowsPerWave + lane;   // lane = 32 half + l32 finishes row l32 of tile `half`
  const size_t o = (size_t)unit * p.max_evict + j;
  bool fragile = false;
  if (CAUSAL && j == 0) {                    // no earlier key
    p.match[o] = -1;
    if (p.sim_out != nullptr) p.sim_out[o] = -INFINITY;
  } else if (j < n_ev)
    fragile = decide_row_f32(p, o, half ? y1[1] : y1[0], half ? c1[1] : c1[0], half ? y2[1] : y2[0],
                             half ? ss_row[1] : ss_row[0], CAUSAL ? j : n_keep);
  if (__any(fragile)) {                      // uniform over the wavefront
    const uint32_t m0 = candidate_columns(p, cls[0], y1[0], ss_row[0], half);
    const uint32_t m1 = candidate_columns(p, cls[1], y1[1], ss_row[1], half);
    if (fragile) {
      const int at = atomicAdd(p.flag_count, 1);
      p.flag_rows[at] = (int)o;
      p.flag_cols[at] = half ? m1 : m0;
    }
  }
  { const int pass = (rb - first_rb) / p.per_unit; if (pass < 4) KX_TS(4 + pass); }
  if (!more) break;
  rb = rb_next;
  }
}

// Few evicted rows per head (the steady state: one period's worth).  One workgroup of 8 wavefronts per
// 64-row block, so the work of one head spreads over a whole compute unit instead of a single
// wavefront.  The 64 evicted rows are copied once into LDS (swizzled like the stages above) and serve as
// the B operand of every wavefront; a wavefront takes every 8th block of 32 retained columns and requests
// the keys of four of its blocks at once, straight into registers as A operands, because the kernel is
// all memory latency: nothing is reused and little is computed.  1/|k_c| is formed here from the operand
// registers (the two lanes of a column hold one half of its channels each).  The fold is the transposed one
// of the first event's kernel (a lane holds one evicted row; class maxima and a (best, second, block) triple).
constexpr int kSmallWaves = 8;
constexpr int kSmallBatch = 4;        // column blocks in flight per wavefront
constexpr int kSmallMaxParts = 4;     // workgroups that may share one 64-row block
template <int D>
__global__ __launch_bounds__(kSmallWaves* kWave, 2) void match_small_kernel(MatchParams p) {
  constexpr int KS = D / 16, ROWB = D * 2, CHUNKS = ROWB / 16;
  constexpr int ROW_LOADS = 64 * CHUNKS / (kSmallWaves * kWave);       // 16-byte copies per thread for the 64 rows
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* s_rows = smem;                                         // [64][ROWB], chunk c at c ^ (row mod CHUNKS)
  int* s_top = reinterpret_cast<int*>(smem + 64 * ROWB);                // [kSmallWaves][64][3]
  float* s_rn = reinterpret_cast<float*>(s_top + kSmallWaves * 64 * 3); // [kSmallWaves][32]: a wavefront's current block

  const int unit = blockIdx.y;
  const int part = blockIdx.z, parts = p.small_parts;
  KS_TS(0);
  const int n_ev = p.n_evict[unit];
  const int row_blk = blockIdx.x * 64;
  if (row_blk >= n_ev) return;                 // all parts of the block alike
  KS_TS(1);
  const int n_keep = p.budget;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const unsigned char* kbytes = reinterpret_cast<const unsigned char*>(p.k) + (size_t)unit * p.capacity * ROWB;
  const int32_t* keep = p.keep_idx + (size_t)unit * p.budget;
  const int32_t* evict = p.evict_idx + (size_t)unit * p.max_evict;
  const int ncb = (n_keep + 31) / 32;

  // ---- requests, all issued before the first wait ---------------------------------------------------
  // (1) slot numbers of the evicted rows this thread copies, and of the first batch's retained keys
  int ev_slot[ROW_LOADS];
#pragma unroll
  for (int i = 0; i < ROW_LOADS; ++i) {
    const int q = tid + i * (kSmallWaves * kWave);
    ev_slot[i] = evict[min(row_blk + q / CHUNKS, n_ev - 1)];
  }
  auto col_slot = [&](int cb) { return keep[min(cb * 32 + l32, n_keep - 1)]; };
  // column blocks of this wavefront: first_cb, first_cb + stride, ...; kSmallBatch of them in flight
  const int first_cb = part * kSmallWaves + wave, stride = parts * kSmallWaves;
  int slot[kSmallBatch];
  bool slot_ok[kSmallBatch];
#pragma unroll
  for (int i = 0; i < kSmallBatch; ++i) slot[i] = col_slot(min(first_cb + i * stride, ncb - 1));
  // (2) the first batch of retained keys, as A operands: lane (l32, half) holds chunks 2 ks + half of column l32.
  // They are requested BEFORE the evicted rows' asynchronous copies: the compiler waits for a load into
  // registers (here the slot numbers) behind every outstanding asynchronous copy, so the other order put the
  // rows' whole round trip in front of these requests, and each block's requests behind the previous block's.
  uint4 akey[kSmallBatch][KS];
  auto request_keys = [&](int cb_first) {
    // one wait for all slot numbers, then all requests: a wait placed behind a conditional batch of requests
    // would cover that batch as well
    static_assert(kSmallBatch == 4, "the statement below names four slot numbers");
    asm volatile("" : "+v"(slot[0]), "+v"(slot[1]), "+v"(slot[2]), "+v"(slot[3]));   // first use of all four: here
#pragma unroll
    for (int i = 0; i < kSmallBatch; ++i) {
      slot_ok[i] = slot[i] >= 0;             // (a negative slot number: slot 0 stands in, its column scores 0)
      if (cb_first + i * stride < ncb) {     // uniform over the wavefront; blocks beyond the list are not fetched
        const unsigned char* row = kbytes + ((uint32_t)max(slot[i], 0) * ROWB + half * 16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) akey[i][ks] = *reinterpret_cast<const uint4*>(row + ks * 32);
      }
    }
  };
  // (the evicted rows' slot numbers too have their first use here, ahead of the key requests: their wait
  // would otherwise come behind those requests and cover them)
#pragma unroll
  for (int i = 0; i < ROW_LOADS; ++i) asm volatile("" : "+v"(ev_slot[i]));
  request_keys(first_cb);
  // (3) the evicted rows -> LDS; a wavefront instruction deposits 64 consecutive 16-byte chunks
#pragma unroll
  for (int i = 0; i < ROW_LOADS; ++i) {
    const int q = tid + i * (kSmallWaves * kWave);
    const int r = q / CHUNKS, phys = q % CHUNKS;
    const unsigned char* src = kbytes + ((uint32_t)ev_slot[i] * ROWB + ((phys ^ (r & (CHUNKS - 1))) * 16));
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(s_rows + (q - lane) * 16), 16, 0, 0);
  }

  int cls[2][16];
  int b1[2] = {0, 0}, b2[2] = {0, 0}, g1[2] = {0, 0};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) cls[t][i] = 0;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();                           // the rows are in LDS
  KS_TS(2);

  const uint32_t frag0 = l32 * ROWB + (((l32 & (CHUNKS - 1)) ^ half) * 16);
  auto efrag = [&](int t, int ks) {          // B operand: evicted row 32 t + l32, chunk (2 ks + half) ^ (row mod CHUNKS)
    return *reinterpret_cast<const bf16x8_t*>(s_rows + ((frag0 ^ (uint32_t)(ks * 32)) + t * 32 * ROWB));
  };
  for (int cb0 = first_cb; cb0 < ncb; cb0 += kSmallBatch * stride) {
#pragma unroll
    for (int i = 0; i < kSmallBatch; ++i) {
      const int cb = cb0 + i * stride;
      if (cb < ncb) {                        // uniform over the wavefront
        asm volatile("" ::: "memory");       // the evicted rows are read from LDS again for every block: kept
                                             // in registers beside four blocks of keys they would spill
        // 1/|k_c| of this block's columns: each lane squares its half of column l32's channels, the halves
        // meet, and the 32 values pass through this wavefront's corner of LDS to reach the lanes that hold
        // the columns' products (registers 4 g + e of a lane: columns 8 g + 4 half + e).  Zero for a column
        // beyond the list, a negative slot number or a zero key: such a column scores 0.
        {
          float ssq = 0.f;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const uint32_t w4[4] = {akey[i][ks].x, akey[i][ks].y, akey[i][ks].z, akey[i][ks].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float lo = bf16_lo(w4[e]), hi = bf16_hi(w4[e]);
              ssq = fmaf(lo, lo, ssq);
              ssq = fmaf(hi, hi, ssq);
            }
          }
          ssq += __shfl_xor(ssq, 32);
          uint32_t bits = 0;
          if (__any(!norm_in_range(ssq))) {   // (rare: a zero key, or a norm that f32 cannot hold)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) bits |= akey[i][ks].x | akey[i][ks].y | akey[i][ks].z | akey[i][ks].w;
            bits |= (uint32_t)__shfl_xor((int)bits, 32);
          }
          const bool real = cb * 32 + l32 < n_keep && slot_ok[i];
          if (half == 0) s_rn[wave * 32 + l32] = real ? column_rnorm(ssq, (bits & 0x7FFF7FFFu) != 0) : 0.f;
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        const f32x4_t* rn_src = reinterpret_cast<const f32x4_t*>(s_rn + wave * 32 + 4 * half);
#pragma unroll
        for (int t = 0; t < 2; ++t) {        // one 32-row tile after the other: 16 accumulator registers
          f32x16_t acc = {0};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, akey[i][ks]), efrag(t, ks), acc, 0, 0, 0);
          int gm = 0;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4_t rn = rn_src[2 * g];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int k = __builtin_bit_cast(int, acc[4 * g + e] * rn[e]);
              cls[t][4 * g + e] = imax(cls[t][4 * g + e], k);
              gm = imax(gm, k);
            }
          }
          g1[t] = (gm > b1[t]) ? cb : g1[t];
          b2[t] = imed3(b1[t], b2[t], gm);
          b1[t] = imax(b1[t], gm);
        }
      }
    }
    if (cb0 + kSmallBatch * stride < ncb) {   // a long retained list: the next batch (its latency is exposed)
#pragma unroll
      for (int i = 0; i < kSmallBatch; ++i)
        slot[i] = col_slot(min(cb0 + (kSmallBatch + i) * stride, ncb - 1));
      request_keys(cb0 + kSmallBatch * stride);
    }
  }

  KS_TS(3);
  // ---- this wavefront's result per row: winning class per tile, then the two halves of a row meet ----
  int y1[2], y2[2], c1[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int s1 = cls[t][0], s2 = 0, ci = 0;
#pragma unroll
    for (int i = 1; i < 16; ++i) {
      const int x = cls[t][i];
      const bool up = x > s1;
      s2 = up ? s1 : imax(s2, x);
      ci = up ? i : ci;
      s1 = up ? x : s1;
    }
    const int col = 32 * g1[t] + 8 * (ci / 4) + 4 * half + (ci % 4);
    const int rest = imax(b2[t], s2);                         // bounds every other column of this half
    const int o1 = __shfl_xor(s1, 32), orest = __shfl_xor(rest, 32), ocol = __shfl_xor(col, 32);
    y1[t] = imax(s1, o1);
    c1[t] = (s1 > o1) ? col : ((o1 > s1) ? ocol : min(col, ocol));
    y2[t] = imax(imax(rest, orest), imin(s1, o1));
  }
  {                                                           // lane = 32 half + l32 speaks for row l32 of tile `half`
    int* t3 = s_top + (wave * 64 + lane) * 3;
    t3[0] = half ? y1[1] : y1[0];
    t3[1] = half ? c1[1] : c1[0];
    t3[2] = half ? y2[1] : y2[0];
  }
  __syncthreads();
  KS_TS(4);
  if (wave != 0) return;
  const int j = row_blk + lane;
  int v1 = (int)0x80000000, v2 = (int)0x80000000, cc = 0;
  auto join = [&](int val, int col, int val2) {      // another share's (best, column, runner-up) for this row
    if (val > v1 || (val == v1 && col < cc)) {
      v2 = imax(v1, val2);
      v1 = val;
      cc = col;
    } else {
      v2 = imax(v2, val);
    }
  };
  for (int w = 0; w < kSmallWaves; ++w) {
    const int* t3 = s_top + (w * 64 + lane) * 3;
    join(t3[0], t3[1], t3[2]);
  }
  if (parts > 1) {
    // The workgroups that share this row block meet the way the decode splits do: device-scope stores of the
    // per-row results, a ticket (a control word at the head of the workspace, zero between calls), and the
    // last one to arrive joins all shares, in list order, and clears the ticket.
    const int blk = unit * (int)gridDim.x + (int)blockIdx.x;
    int32_t* mine = p.small_partial + ((size_t)(blk * parts + part) * 64 + lane) * 3;
    __hip_atomic_store(mine + 0, v1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(mine + 1, cc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(mine + 2, v2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the wavefront's write-through stores have completed
    int ticket = 0;
    if (lane == 0) ticket = __hip_atomic_fetch_add(&p.exact_ticket[blk], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ticket = __builtin_amdgcn_readfirstlane(ticket);
    if (ticket != parts - 1) return;
    v1 = (int)0x80000000; v2 = (int)0x80000000; cc = 0;
    int val[kSmallMaxParts], col[kSmallMaxParts], val2[kSmallMaxParts];
#pragma unroll
    for (int q = 0; q < kSmallMaxParts; ++q) {       // one round trip for all shares
      const int32_t* r = p.small_partial + ((size_t)(blk * parts + min(q, parts - 1)) * 64 + lane) * 3;
      val[q] = __hip_atomic_load(r + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      col[q] = __hip_atomic_load(r + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      val2[q] = __hip_atomic_load(r + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int q = 0; q < kSmallMaxParts; ++q)
      if (q < parts) join(val[q], col[q], val2[q]);
    if (lane == 0) __hip_atomic_store(&p.exact_ticket[blk], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (j >= n_ev) return;
  // |k_e|^2 of this lane's row, from the LDS copy
  float ss = 0.f;
  {
    const unsigned char* row = s_rows + lane * ROWB;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      const uint4 x = *reinterpret_cast<const uint4*>(row + c * 16);   // the order of the chunks does not matter here
      const uint32_t w4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = bf16_lo(w4[i]), hi = bf16_hi(w4[i]);
        ss = fmaf(lo, lo, ss);
        ss = fmaf(hi, hi, ss);
      }
    }
  }
  decide_row(p, unit, j, v1, cc, v2, ss);
  KS_TS(5);
}

// ---------------------------------------------------------------------------------------------------
// f64 evaluation, of all rows (f32 caches, the kernel below) or of the queued ones (bf16 caches, further down).  f32 caches: threads
// stride over the retained keys (each thread evaluates whole keys,
// channels in index order, so the sums match an index-order f64 sum).  One workgroup per row; when the
// live rows are so few that the compute units would mostly idle (the steady state), up to
// kExactMaxParts workgroups per row, each over a contiguous share of the retained list, as long as a thread of an undivided list
// would have a second key to go through (exact_shares).  Their results
// meet the way the decode splits do: device-scope stores, a ticket, the last one to arrive combines and
// clears the ticket (the tickets are control words at the head of the workspace, zero between calls).
constexpr int kExactMaxParts = 8;
constexpr int kExactResident = 512;     // workgroups of the bf16 f64 kernel that run at once (two per compute unit); size of the partial array
constexpr int kExactResidentGeneric = 256;   // f32 rows are shared while every share finds a compute unit of its own
// most shares that a row of `cols` columns is worth
__host__ __device__ constexpr int exact_shares(int cols) {
  int n = 1;
  while (n < kExactMaxParts && cols > n * 256) n *= 2;
  return n;
}
struct ExactPartial {
  unsigned long long best_bits;
  int best_c, pad;
};

// The queue counter is a control word that must be zero when the next call starts.  A workgroup adds the
// number of queued rows it has finished to the exit counter (nothing if it finished none: with an empty queue
// no workgroup touches either word), and the workgroup whose addition completes the queue clears both.
// Every workgroup that had work read the queue counter before it started, and the others do nothing whatever
// value they read, so clearing it then is safe.
__device__ __forceinline__ void exact_exit(const MatchParams& p, int n_flag, int rows_finished) {
  if (threadIdx.x == 0 && rows_finished > 0 &&
      __hip_atomic_fetch_add(p.exact_done, rows_finished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + rows_finished == n_flag) {
    __hip_atomic_store(p.flag_count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p.exact_done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ int wave_prefix_sum(int n, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(n, off);
    if (lane >= off) n += o;
  }
  return n;
}

template <typename T, int D>
__global__ __launch_bounds__(256) void match_exact_kernel(MatchParams p) {
  __shared__ double s_e[D];
  __shared__ double s_best[4];
  __shared__ int s_bestc[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const T* kall = reinterpret_cast<const T*>(p.k);
  constexpr int EPV = 16 / (int)sizeof(T), NV = D / EPV;
  // The live rows are counted and not queued, which took a launch of its own.  Where the heads differ, thread t adds up those of `per`
  // heads, and s_first[t] is how many come before them; the usual case of equally many in every head needs neither that nor a search.
  // Measured, D 64, queued / stepping over every row that the caches have room for / this way: 4 heads of 32 live rows x 820 keys in caches of
  // 16384 slots 12.9 / 26.5 / 10.6 us, 4 heads of 32 rows x 52 keys in caches of 84 10.2 / 7.6 / 5.7.
  __shared__ int s_first[257], s_wave[4];
  __shared__ int s_group;
  auto live = [&](int u) {
    return u >= p.n_units ? 0 : imax(p.causal ? imin(p.len[u], p.capacity) : imin(p.n_evict[u], p.max_evict), 0);
  };
  const int per = (p.n_units + 255) / 256, n_first = __builtin_amdgcn_readfirstlane(live(0));
  bool same = true;
  for (int u = lane; u < p.n_units; u += 64) same = same && live(u) == n_first;
  same = __all(same);
  int n_rows = p.n_units * n_first;
  if (!same) {
    int n = 0;
    for (int u = tid * per; u < (tid + 1) * per; ++u) n += live(u);
    int upto = wave_prefix_sum(n, lane);
    if (lane == 63) s_wave[wave] = upto;
    __syncthreads();
    for (int w = 0; w < wave; ++w) upto += s_wave[w];
    s_first[tid + 1] = upto;
    if (tid == 0) s_first[0] = 0;
    __syncthreads();
    n_rows = __builtin_amdgcn_readfirstlane(s_first[256]);
  }
  int parts = exact_shares(p.causal ? p.capacity : p.budget);
  while (parts > 1 && (long)n_rows * parts > (long)imin((int)gridDim.x, kExactResidentGeneric)) parts /= 2;
  const unsigned n_work = (unsigned)n_rows * parts;        // (below 2^31: shared only if at most kExactResidentGeneric)
  for (unsigned w = blockIdx.x; w < n_work; w += gridDim.x) {
    const int f = (int)(w / (unsigned)parts), part = (int)(w % (unsigned)parts);
    __syncthreads();                      // previous row's shared values are no longer read
    int unit, j;
    if (same) {
      unit = f / n_first;
      j = f % n_first;
    } else {
      if (s_first[tid] <= f && f < s_first[tid + 1]) s_group = tid;      // one thread
      __syncthreads();
      // The row's head among those `per`, a head a lane (16384 heads of 2 to 4 rows x 36 keys, D 64: 521 us when one
      // thread walked over them, 280).
      unit = s_group * per;
      j = f - s_first[s_group];
      if (per > 1) {
        static_assert(kMaxUnits <= 256 * 64);
        const int n = lane < per ? live(unit + lane) : 0;
        const int end = wave_prefix_sum(n, lane);
        const int at = __builtin_ctzll(__ballot(j < end) | 1ull << 63);
        j -= __shfl(end - n, at);
        unit += at;
      }
    }
    unit = __builtin_amdgcn_readfirstlane(unit);
    j = __builtin_amdgcn_readfirstlane(j);
    const int o = unit * p.max_evict + j;
    if (p.causal && j == 0) {              // no earlier key
      if (tid == 0 && part == 0) {
        p.match[o] = -1;
        if (p.sim_out != nullptr) p.sim_out[o] = -INFINITY;
      }
      continue;
    }
    const T* kunit = kall + (size_t)unit * p.capacity * D;
    // causal (the prefill pass): the row is slot j itself and its columns are the slots 0 .. j - 1
    const int32_t* keep = p.causal ? nullptr : p.keep_idx + (size_t)unit * p.budget;
    const int e = p.causal ? j : p.evict_idx[(size_t)unit * p.max_evict + j];
    const int n_cols = p.causal ? j : p.budget;
    const int share = (n_cols + parts - 1) / parts;
    const int c_lo = part * share, c_hi = imin(n_cols, c_lo + share);
    for (int d = tid; d < D; d += 256) {
      if constexpr (sizeof(T) == 2) s_e[d] = (double)bf16_to_f32(reinterpret_cast<const uint16_t*>(kunit)[(size_t)e * D + d]);
      else s_e[d] = (double)kunit[(size_t)e * D + d];
    }
    __syncthreads();
    double ss_e = 0.0;
    for (int d = 0; d < D; ++d) ss_e = fma(s_e[d], s_e[d], ss_e);
    const double rn_e = 1.0 / sqrt(ss_e);
    double best = -INFINITY;
    int best_c = 0x7FFFFFFF;
    for (int c = c_lo + tid; c < c_hi; c += 256) {
      const int slot = p.causal ? c : keep[c];
      if (slot < 0) continue;
      const T* kc = kunit + (size_t)slot * D;
      uint4 rowv[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) rowv[v] = reinterpret_cast<const uint4*>(kc)[v];   // one round trip per key
      // Left to itself the compiler either loaded a vector when the one before was used up or held the row s_e in registers, two
      // workgroups per compute unit at D 64 and one at 128; with the loads kept ahead it is four and two (24 heads of 616 rows x 52 keys, D 64,
      // 80 us, now 52; 8 heads of 512 x 512, D 128, 164, now 142).
      __builtin_amdgcn_sched_barrier(0);
      double dot = 0.0, ss_c = 0.0;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int d0 = v * EPV;
        const uint4 x = rowv[v];
        if constexpr (sizeof(T) == 2) {
          const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double lo = (double)bf16_lo(w[i]), hi = (double)bf16_hi(w[i]);
            dot = fma(s_e[d0 + 2 * i], lo, dot);
            ss_c = fma(lo, lo, ss_c);
            dot = fma(s_e[d0 + 2 * i + 1], hi, dot);
            ss_c = fma(hi, hi, ss_c);
          }
        } else {
          const float w[4] = {__builtin_bit_cast(float, x.x), __builtin_bit_cast(float, x.y),
                              __builtin_bit_cast(float, x.z), __builtin_bit_cast(float, x.w)};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            dot = fma(s_e[d0 + i], (double)w[i], dot);
            ss_c = fma((double)w[i], (double)w[i], ss_c);
          }
        }
      }
      const double rn_c = 1.0 / sqrt(ss_c);
      double u = (dot * rn_e) * rn_c;
      if (!(fabs(u) <= 1.79e308)) u = -INFINITY;   // zero-norm keys (nan / inf) match nothing
      if (u > best) {
        best = u;
        best_c = c;
      }
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double ob = __shfl_xor(best, off);
      const int oc = __shfl_xor(best_c, off);
      if (ob > best || (ob == best && oc < best_c)) {
        best = ob;
        best_c = oc;
      }
    }
    if (lane == 0) {
      s_best[wave] = best;
      s_bestc[wave] = best_c;
    }
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < 4; ++w)
        if (s_best[w] > best || (s_best[w] == best && s_bestc[w] < best_c)) {
          best = s_best[w];
          best_c = s_bestc[w];
        }
      bool finish = parts == 1;
      if (!finish) {
        // with parts > 1 every workgroup has at most one work item, w < gridDim.x
        ExactPartial* mine = p.exact_partial + w;
        __hip_atomic_store(&mine->best_bits, __builtin_bit_cast(unsigned long long, best), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&mine->best_c, best_c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the two write-through stores have completed
        finish = __hip_atomic_fetch_add(&p.exact_ticket[f], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
        if (finish) {                     // the last share of this row: join them, in list order
          best = -INFINITY;
          best_c = 0x7FFFFFFF;
          for (int q = 0; q < parts; ++q) {
            const ExactPartial* r = p.exact_partial + f * parts + q;
            const double rb = __builtin_bit_cast(double, __hip_atomic_load(&r->best_bits, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT));
            const int rc = __hip_atomic_load(&r->best_c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (rb > best) {
              best = rb;
              best_c = rc;
            }
          }
          __hip_atomic_store(&p.exact_ticket[f], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
        }
      }
      if (finish) {
        p.match[o] = (best > (double)p.threshold) ? best_c : -1;
        if (p.sim_out != nullptr) p.sim_out[o] = (float)best;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Merge-first prefill pass (App. B.4): for every live slot its most similar EARLIER key, by the first event's kernel in
// its causal mode.
// 1/|k_i| (f32) of every live slot; 0 for zero keys and beyond len, NaN where f32 cannot hold the norm
template <typename T, int D>
__global__ __launch_bounds__(256) void slot_rnorm_kernel(const T* __restrict__ k, const int32_t* __restrict__ len,
                                                         float* __restrict__ rn, int capacity) {
  constexpr int EPL = 16 / (int)sizeof(T), LPS = D / EPL, RPB = 256 / LPS;
  const int unit = blockIdx.y, sub = threadIdx.x % LPS;
  const int r = blockIdx.x * RPB + threadIdx.x / LPS;
  const int n = len[unit];
  if (r >= capacity) return;
  float ss = 0.f;
  uint4 x = make_uint4(0, 0, 0, 0);
  if (r < n) {
    x = reinterpret_cast<const uint4*>(k)[((size_t)unit * capacity + r) * LPS + sub];
    if constexpr (sizeof(T) == 2) {
      const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = bf16_lo(w[e]), b = bf16_hi(w[e]);
        ss = fmaf(a, a, ss);
        ss = fmaf(b, b, ss);
      }
    } else {
      const float w[4] = {__builtin_bit_cast(float, x.x), __builtin_bit_cast(float, x.y),
                          __builtin_bit_cast(float, x.z), __builtin_bit_cast(float, x.w)};
#pragma unroll
      for (int e = 0; e < 4; ++e) ss = fmaf(w[e], w[e], ss);
    }
  }
  ss = group_sum<LPS>(ss);
  const bool nonzero = norm_in_range(ss) || row_nonzero<T, LPS>(x);   // (whole lane groups)
  if (sub == 0) rn[(size_t)unit * capacity + r] = column_rnorm(ss, nonzero);
}


// The f64 kernels for bf16 caches.  Products of bf16 values are exact in f64 and so are their sums over the head
// dimension (for any ordinary exponent spread), whatever the order, so a key's channels may be split over lanes:
// four lanes share a key, each holding a quarter of the channels of the evicted row in registers (as f64) and
// loading the same quarter of the key.
template <int D>
struct ExactQuarter {
  static constexpr int CPL = D / 32, EPL = CPL * 8;          // 16-byte chunks / channels per lane
  double ed[EPL];
  double rn_e;
  __device__ __forceinline__ void load(const unsigned char* row, int sub) {
    uint4 ev[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) ev[q] = *reinterpret_cast<const uint4*>(row + (sub * CPL + q) * 16);
    double ss_e = 0.0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const uint32_t wv[4] = {ev[q].x, ev[q].y, ev[q].z, ev[q].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ed[q * 8 + 2 * i] = (double)bf16_lo(wv[i]);
        ed[q * 8 + 2 * i + 1] = (double)bf16_hi(wv[i]);
        ss_e = fma(ed[q * 8 + 2 * i], ed[q * 8 + 2 * i], ss_e);
        ss_e = fma(ed[q * 8 + 2 * i + 1], ed[q * 8 + 2 * i + 1], ss_e);
      }
    }
    ss_e += __shfl_xor(ss_e, 1);
    ss_e += __shfl_xor(ss_e, 2);
    rn_e = 1.0 / sqrt(ss_e);
  }
  // the cosine with the key whose quarter is in x (the same value in the four lanes); -inf for a zero-norm key
  __device__ __forceinline__ double cosine(const uint4 (&x)[CPL]) const {
    double dot = 0.0, ss_c = 0.0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const uint32_t wv[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double lo = (double)bf16_lo(wv[i]), hi = (double)bf16_hi(wv[i]);
        dot = fma(ed[q * 8 + 2 * i], lo, dot);
        ss_c = fma(lo, lo, ss_c);
        dot = fma(ed[q * 8 + 2 * i + 1], hi, dot);
        ss_c = fma(hi, hi, ss_c);
      }
    }
    dot += __shfl_xor(dot, 1);
    ss_c += __shfl_xor(ss_c, 1);
    dot += __shfl_xor(dot, 2);
    ss_c += __shfl_xor(ss_c, 2);
    const double u = (dot * rn_e) * (1.0 / sqrt(ss_c));
    return fabs(u) <= 1.79e308 ? u : -INFINITY;               // zero-norm keys (nan / inf) match nothing
  }
};
// best value and lowest column of the 16 quads of a wavefront (the four lanes of a quad hold the same pair)
__device__ __forceinline__ void best_of_quads(double& best, int& best_c) {
#pragma unroll
  for (int off = 4; off < 64; off <<= 1) {
    const double ob = __shfl_xor(best, off);
    const int oc = __shfl_xor(best_c, off);
    if (ob > best || (ob == best && oc < best_c)) {
      best = ob;
      best_c = oc;
    }
  }
}

// First event and prefill pass: every queued row comes with the mask of its candidate columns (candidate_columns above),
// and one wavefront re-evaluates them, 16 at a time and kRecheckBatch such rounds in flight.  The first event reads the
// retained keys from the gathered panel; the prefill pass (causal) the slots before the row.
// What bounds it: a chain of four dependent round trips per row (queue, evicted slot, its row, keys).  Evaluating every
// column of a row with a whole workgroup took (MI355X) 218 us for the long-context first event and 450 us for the
// batch-128 one; the candidates alone take 21 and 32 us.
constexpr int kRecheckBatch = 4;
template <int D>
__global__ __launch_bounds__(256) void match_recheck_kernel(MatchParams p) {
  constexpr int ROWB = D * 2, CHUNKS = ROWB / 16, CPL = ExactQuarter<D>::CPL;
  __shared__ int s_done;
  __shared__ unsigned char s_off[4][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, quad = lane >> 2, sub = lane & 3;
  const int n_flag = *p.flag_count;
  if (tid == 0) s_done = 0;
  __syncthreads();
  int finished = 0;                          // rows whose result this wavefront has written
  for (int f = blockIdx.x * 4 + wave; f < n_flag; f += gridDim.x * 4) {
    const int o = p.flag_rows[f];
    const uint32_t cols = p.flag_cols[f];
    const int unit = o / p.max_evict, j = o % p.max_evict;
    const unsigned char* kunit = reinterpret_cast<const unsigned char*>(p.k) + (size_t)unit * p.capacity * ROWB;
    const int e = p.causal ? j : p.evict_idx[(size_t)unit * p.max_evict + j];
    const int n_cols = p.causal ? j : p.budget;
    // the k-th candidate is column 32 (k / n_off) + s_off[k mod n_off]: ascending in k
    const int n_off = __popc(cols);
    if (lane < 32 && ((cols >> lane) & 1u)) s_off[wave][__popc(cols & ((1u << lane) - 1u))] = (unsigned char)lane;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int n_cand = n_off * ((n_cols + 31) / 32);
    const unsigned char* keys = p.causal ? kunit : p.panel + (size_t)unit * p.rn_pitch * ROWB;
    ExactQuarter<D> row;
    row.load(kunit + (size_t)e * ROWB, sub);
    double best = -INFINITY;
    int best_c = 0x7FFFFFFF;
    for (int k0 = 0; k0 < n_cand; k0 += 16 * kRecheckBatch) {
      int col[kRecheckBatch];
      uint4 x[kRecheckBatch][CPL];
#pragma unroll
      for (int b = 0; b < kRecheckBatch; ++b) {
        const int k = k0 + b * 16 + quad;
        const int blk = k / n_off;
        const int c = 32 * blk + s_off[wave][k - blk * n_off];
        col[b] = (k < n_cand && c < n_cols) ? c : -1;
        const int at = max(col[b], 0);                             // (n_cand > 0: column 0 exists)
        const unsigned char* rp = keys + (size_t)at * ROWB;
        const int swz = p.causal ? 0 : (at & (CHUNKS - 1));        // panel: chunk ch of key c at position ch ^ (c mod CHUNKS)
#pragma unroll
        for (int q = 0; q < CPL; ++q) x[b][q] = *reinterpret_cast<const uint4*>(rp + (((sub * CPL + q) ^ swz) * 16));
      }
#pragma unroll
      for (int b = 0; b < kRecheckBatch; ++b) {
        const double u = row.cosine(x[b]);
        if (col[b] >= 0 && (u > best || (u == best && col[b] < best_c))) {
          best = u;
          best_c = col[b];
        }
      }
    }
    best_of_quads(best, best_c);
    if (lane == 0) {
      p.match[o] = (best > (double)p.threshold) ? best_c : -1;
      if (p.sim_out != nullptr) p.sim_out[o] = (float)best;
    }
    ++finished;
  }
  if (lane == 0 && finished > 0) atomicAdd(&s_done, finished);
  __syncthreads();
  exact_exit(p, n_flag, s_done);
}

// Steady state: few queued rows, each against all retained keys.
// One workgroup per queued row, or per share of a row's columns when the queue is short (joined by a ticket, as
// in the generic kernel above).  The slot numbers of a whole batch are requested first, then their rows.
constexpr int kExactBatch = 4;
template <int D>
__global__ __launch_bounds__(256) void match_exact_bf16_kernel(MatchParams p) {
  constexpr int ROWB = D * 2, CPL = ExactQuarter<D>::CPL;
  __shared__ double s_best[4];
  __shared__ int s_bestc[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int quad = tid >> 2, sub = tid & 3;
  const int n_flag = *p.flag_count;
  int rows_finished = 0;                 // (thread 0) queued rows whose result this workgroup has written
  const unsigned char* kall = reinterpret_cast<const unsigned char*>(p.k);
  int parts = 1;
  {
    const int room = imin((int)gridDim.x, kExactResident);
    while (parts < kExactMaxParts && (long)n_flag * (parts * 2) <= (long)room) parts *= 2;
  }
  for (int w = blockIdx.x; w < n_flag * parts; w += gridDim.x) {
    const int f = w / parts, part = w % parts;
    const int o = p.flag_rows[f];
    const int unit = o / p.max_evict, j = o % p.max_evict;
    const unsigned char* kunit = kall + (size_t)unit * p.capacity * ROWB;
    const int32_t* keep = p.keep_idx + (size_t)unit * p.budget;
    const int share = (p.budget + parts - 1) / parts;
    const int c_lo = part * share, c_hi = imin(p.budget, c_lo + share);
    // this lane's quarter of the evicted row (its slot number is one more round trip; the keys below do not wait for it)
    ExactQuarter<D> row_e;
    row_e.load(kunit + (size_t)p.evict_idx[(size_t)unit * p.max_evict + j] * ROWB, sub);
    double best = -INFINITY;
    int best_c = 0x7FFFFFFF;
    for (int c0 = c_lo; c0 < c_hi; c0 += 64 * kExactBatch) {
      int slot[kExactBatch];
      uint4 row[kExactBatch][CPL];
#pragma unroll
      for (int b = 0; b < kExactBatch; ++b) {
        const int c = c0 + b * 64 + quad;
        slot[b] = (c < c_hi) ? keep[c] : -1;
      }
#pragma unroll
      for (int b = 0; b < kExactBatch; ++b) {
        const unsigned char* rp = kunit + (size_t)imax(slot[b], 0) * ROWB + sub * CPL * 16;
#pragma unroll
        for (int q = 0; q < CPL; ++q) row[b][q] = *reinterpret_cast<const uint4*>(rp + q * 16);
      }
#pragma unroll
      for (int b = 0; b < kExactBatch; ++b) {
        const double u = row_e.cosine(row[b]);
        if (slot[b] >= 0 && u > best) {              // ascending c per lane and strict: the first maximiser stays
          best = u;
          best_c = c0 + b * 64 + quad;
        }
      }
    }
    best_of_quads(best, best_c);
    __syncthreads();                                 // the previous row's shared values are no longer read
    if (lane == 0) {
      s_best[wave] = best;
      s_bestc[wave] = best_c;
    }
    __syncthreads();
    if (tid == 0) {
      for (int ww = 1; ww < 4; ++ww)
        if (s_best[ww] > best || (s_best[ww] == best && s_bestc[ww] < best_c)) {
          best = s_best[ww];
          best_c = s_bestc[ww];
        }
      bool finish = parts == 1;
      if (!finish) {
        ExactPartial* mine = p.exact_partial + w;    // with parts > 1 every workgroup has at most one work item
        __hip_atomic_store(&mine->best_bits, __builtin_bit_cast(unsigned long long, best), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&mine->best_c, best_c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the two write-through stores have completed
        finish = __hip_atomic_fetch_add(&p.exact_ticket[f], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
        if (finish) {                                // the last share of this row: join them, in list order
          best = -INFINITY;
          best_c = 0x7FFFFFFF;
          for (int q = 0; q < parts; ++q) {
            const ExactPartial* r = p.exact_partial + f * parts + q;
            const double rb = __builtin_bit_cast(double, __hip_atomic_load(&r->best_bits, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT));
            const int rc = __hip_atomic_load(&r->best_c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (rb > best) {
              best = rb;
              best_c = rc;
            }
          }
          __hip_atomic_store(&p.exact_ticket[f], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
        }
      }
      if (finish) {
        p.match[o] = (best > (double)p.threshold) ? best_c : -1;
        if (p.sim_out != nullptr) p.sim_out[o] = (float)best;
        ++rows_finished;
      }
    }
  }
  exact_exit(p, n_flag, rows_finished);
}

template <int D>
constexpr size_t mfma_smem_bytes() {
  return 2 * (size_t)kStageCols * (D * 2) + 2 * kStageCols * sizeof(float);
}
inline size_t small_smem_bytes(int head_dim) {   // evicted rows, per-wavefront results, 1/|k_c| of a block per wavefront
  return (size_t)64 * head_dim * 2 + (size_t)kSmallWaves * 64 * 3 * 4 + (size_t)kSmallWaves * 32 * 4;
}
constexpr int kSmallMaxEvict = 256;   // up to this many evictable slots per head the column-split kernel is used
constexpr int kSmallMaxShares = 256;  // workgroups of that kernel when row blocks are shared (one per compute unit)

inline int rn_pitch_of(int budget) { return (budget + kStageCols - 1) / kStageCols * kStageCols; }

// The causal search.  Workgroups of 4 wavefronts (256 rows, two on a compute unit) or of 8 (512 rows, one): the larger
// ones stream every column half as often but need many blocks to even out the triangle.  MI355X, D 128, whole call,
// 4 against 8 wavefronts: 8 heads x 2048 slots 38.9 / 52.7 us, 64 x 2048 52.6 / 62.7, 8 x 16384 (256 blocks of 512 rows)
// 295 / 346, 64 x 4096 (512 blocks) 144 / 144, 8 x 32768 (512 blocks) 958 / 903.
constexpr long kCausalWideBlocks = 512;
template <int D, int NW>
keepkv_status launch_causal_waves(MatchParams p, unsigned units, hipStream_t st) {
  static const hipError_t attr = hipFuncSetAttribute((const void*)match_mfma_kernel<D, true, NW>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)mfma_smem_bytes<D>());
  if (attr != hipSuccess) return KEEPKV_ERR_DEVICE;
  p.per_unit = (p.capacity + NW * kRowsPerWave - 1) / (NW * kRowsPerWave);
  p.n_units = (int)units;
  match_mfma_kernel<D, true, NW><<<units * p.per_unit, NW * kWave, mfma_smem_bytes<D>(), st>>>(p);
  return KEEPKV_OK;
}
template <int D>
keepkv_status launch_causal(const MatchParams& p, const void* k, unsigned units, int exact_blocks, hipStream_t st) {
  constexpr int rows = 256 / (D * 2 / 16);
  slot_rnorm_kernel<uint16_t, D><<<dim3((p.capacity + rows - 1) / rows, units), 256, 0, st>>>(
      (const uint16_t*)k, p.len, const_cast<float*>(p.rnorm), p.capacity);
  const bool wide = (long)units * ((p.capacity + 8 * kRowsPerWave - 1) / (8 * kRowsPerWave)) >= kCausalWideBlocks;
  const keepkv_status rc = wide ? launch_causal_waves<D, 8>(p, units, st) : launch_causal_waves<D, 4>(p, units, st);
  if (rc != KEEPKV_OK) return rc;
  match_recheck_kernel<D><<<exact_blocks, 256, 0, st>>>(p);
  return KEEPKV_OK;
}

template <int D>
keepkv_status launch_bf16(const MatchParams& p, const void* k, unsigned units, hipStream_t st) {
  constexpr int rows_per_block = 256 / (D * 2 / 16);
  const bool small = p.max_evict <= kSmallMaxEvict;
  if (!small)   // the steady-state kernel forms its own norms
    rnorm_kernel<uint16_t, D><<<dim3((p.rn_pitch + rows_per_block * kRnormRows - 1) / (rows_per_block * kRnormRows), units), 256, 0, st>>>(
        (const uint16_t*)k, p.keep_idx, p.n_evict, const_cast<float*>(p.rnorm), p.capacity, p.budget, p.rn_pitch,
        reinterpret_cast<uint4*>(const_cast<unsigned char*>(p.panel)));
  static const hipError_t a1 = hipFuncSetAttribute((const void*)match_mfma_kernel<D, false, kMWaves>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)mfma_smem_bytes<D>());
  static const hipError_t a2 = hipFuncSetAttribute((const void*)match_small_kernel<D>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   (int)small_smem_bytes(D));
  if (a1 != hipSuccess || a2 != hipSuccess) return KEEPKV_ERR_DEVICE;
  if (small) {
    // With few heads the row blocks alone leave most compute units idle, and one compute unit takes long to
    // pull a head's whole retained list: up to four workgroups share a row block, each over every fourth
    // batch of column blocks, as long as all of them are resident at once.
    const int row_blocks = (p.max_evict + 63) / 64, ncb = (p.budget + 31) / 32;
    int parts = 1;
    while (parts < kSmallMaxParts && (long)units * row_blocks * (parts * 2) <= kSmallMaxShares && parts * 2 * kSmallWaves < ncb + kSmallWaves)
      parts *= 2;
    MatchParams q = p;
    q.small_parts = parts;
    match_small_kernel<D><<<dim3(row_blocks, units, parts), kSmallWaves * kWave, small_smem_bytes(D), st>>>(q);
  } else {
    // One workgroup fills a compute unit (8 wavefronts of 256 registers).  With fewer heads than compute
    // units each head gets an equal share of them, and a workgroup walks its head's row blocks in passes;
    // with more heads than that, one workgroup per head does all passes.
    constexpr unsigned rows_per_block = kMWaves * kRowsPerWave;
    const unsigned row_blocks = (p.max_evict + rows_per_block - 1) / rows_per_block;
    unsigned per_unit = kResidentWorkgroups / units;
    per_unit = per_unit < 1 ? 1 : (per_unit > row_blocks ? row_blocks : per_unit);
    MatchParams q = p;
    q.per_unit = (int)per_unit;
    q.n_units = (int)units;
    match_mfma_kernel<D, false, kMWaves><<<per_unit * units, kMWaves * kWave, mfma_smem_bytes<D>(), st>>>(q);
  }
  return KEEPKV_OK;
}

// f32 caches: a workgroup for every row and share that there can be, as many as run at once: four (D 64) or two (D 128) per compute unit.
// (The workgroups of a sixteenth of the rows, a rule for queues, walked the 128 rows of an event of 4 heads x 84 slots two by two.)
void launch_exact_f32(MatchParams p, size_t units, int head_dim, int cols, hipStream_t st) {
  const size_t work = units * (size_t)p.max_evict * (size_t)exact_shares(cols), resident = head_dim == 128 ? 512 : 1024;
  const int blocks = (int)(work < resident ? work : resident);
  p.n_units = (int)units;
  if (head_dim == 128) match_exact_kernel<float, 128><<<blocks, 256, 0, st>>>(p);
  else match_exact_kernel<float, 64><<<blocks, 256, 0, st>>>(p);
}

}  // namespace

MatchPlan plan_match(const keepkv_layout* L, int capacity, int budget) {
  MatchPlan pl;
  const size_t units = (size_t)L->batch * L->n_kv_heads;
  pl.rnorm_off = kWorkspaceHead;
  pl.flag_off = kWorkspaceHead + align_up(units * rn_pitch_of(budget) * sizeof(float), 256);
  pl.panel_off = pl.flag_off + align_up(2 * units * (size_t)(capacity - budget) * sizeof(int32_t), 256);
  // the panel is used by bf16 caches with more evictable slots than the column-split kernel takes
  const bool panel = L->dtype == KEEPKV_BF16 && capacity - budget > kSmallMaxEvict;
  pl.partial_off = pl.panel_off + (panel ? align_up(units * rn_pitch_of(budget) * (size_t)L->head_dim * 2, 256) : 0);
  pl.small_partial_off = pl.partial_off + (size_t)kExactResident * 16;
  pl.bytes = pl.small_partial_off + (size_t)kSmallMaxShares * 64 * 3 * sizeof(int32_t);
  return pl;
}

PrefillMatchPlan plan_prefill_match(const keepkv_layout* L, int capacity) {
  PrefillMatchPlan pl;
  const size_t units = (size_t)L->batch * L->n_kv_heads;
  pl.rnorm_off = kWorkspaceHead;
  pl.flag_off = pl.rnorm_off + align_up(units * capacity * sizeof(float), 256);
  pl.partial_off = pl.flag_off + align_up(2 * units * (size_t)capacity * sizeof(int32_t), 256);
  pl.bytes = pl.partial_off + (size_t)kExactResident * 16;
  return pl;
}

}  // namespace kk

extern "C" keepkv_status keepkv_prefill_match(const keepkv_layout* layout, const keepkv_cache* cache, float threshold,
                                              int32_t* near, float* sim_out, void* workspace, size_t workspace_bytes,
                                              void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(cache) || !near) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (!(threshold == threshold) || !aligned16(cache->k)) return KEEPKV_ERR_INVALID_ARG;
  if (layout->head_dim != 64 && layout->head_dim != 128) return KEEPKV_ERR_UNSUPPORTED;
  const size_t units = (size_t)layout->batch * layout->n_kv_heads;
  const int cap = cache->capacity;
  if (units * (size_t)cap >= (size_t)1 << 31) return KEEPKV_ERR_UNSUPPORTED;
  const PrefillMatchPlan pl = plan_prefill_match(layout, cap);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);

  MatchParams p;
  p.k = cache->k; p.keep_idx = nullptr; p.evict_idx = nullptr; p.n_evict = nullptr;
  p.rnorm = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + pl.rnorm_off);
  p.panel = nullptr;
  p.flag_count = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + kMatchCountersOff);
  p.exact_done = p.flag_count + 1;
  p.flag_rows = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.flag_off);
  p.flag_cols = reinterpret_cast<uint32_t*>(p.flag_rows + units * cap);
  p.exact_partial = reinterpret_cast<ExactPartial*>(reinterpret_cast<char*>(workspace) + pl.partial_off);
  p.exact_ticket = reinterpret_cast<int32_t*>(workspace);
  p.match = near; p.sim_out = sim_out;
  p.capacity = cap; p.budget = 0; p.max_evict = cap; p.rn_pitch = cap;
  p.threshold = threshold; p.delta = 1.6e-5f;
  p.per_unit = 0; p.n_units = 0; p.small_parts = 1; p.small_partial = nullptr;
  p.causal = 1; p.len = cache->len;

  long eb = (long)units * cap / 16;
  const int exact_blocks = (int)(eb < 64 ? 64 : (eb > 512 ? 512 : eb));
  if (layout->dtype == KEEPKV_BF16) {
    const keepkv_status rc = layout->head_dim == 128 ? launch_causal<128>(p, cache->k, (unsigned)units, exact_blocks, st)
                                                     : launch_causal<64>(p, cache->k, (unsigned)units, exact_blocks, st);
    if (rc != KEEPKV_OK) return rc;
  } else {
    launch_exact_f32(p, units, layout->head_dim, cap, st);
  }
  return launch_status();
}

extern "C" keepkv_status keepkv_match(const keepkv_layout* layout, const keepkv_cache* cache, int32_t budget,
                                      const int32_t* keep_idx, const int32_t* evict_idx, const int32_t* n_evict,
                                      float threshold, int32_t* match, float* sim_out, void* workspace,
                                      size_t workspace_bytes, void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(cache) || !keep_idx || !n_evict) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (budget < 1 || budget > cache->capacity) return KEEPKV_ERR_INVALID_ARG;
  const int max_evict = cache->capacity - budget;
  if (max_evict == 0) return KEEPKV_OK;   // nothing can be evicted
  if (!evict_idx || !match) return KEEPKV_ERR_INVALID_ARG;
  if (!(threshold == threshold)) return KEEPKV_ERR_INVALID_ARG;
  if (!aligned16(cache->k)) return KEEPKV_ERR_INVALID_ARG;
  if (layout->head_dim != 64 && layout->head_dim != 128) return KEEPKV_ERR_UNSUPPORTED;
  if (budget > 4096) return KEEPKV_ERR_UNSUPPORTED;
  const size_t units = (size_t)layout->batch * layout->n_kv_heads;
  if (units * (size_t)max_evict >= (size_t)1 << 31) return KEEPKV_ERR_UNSUPPORTED;
  const MatchPlan pl = plan_match(layout, cache->capacity, budget);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);

  MatchParams p;
  p.k = cache->k; p.keep_idx = keep_idx; p.evict_idx = evict_idx; p.n_evict = n_evict;
  p.rnorm = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + pl.rnorm_off);
  // queue counter and the f64 kernel's exit counter: control words, zero between calls
  p.flag_count = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + kMatchCountersOff);
  p.exact_done = p.flag_count + 1;
  p.flag_rows = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.flag_off);
  p.flag_cols = reinterpret_cast<uint32_t*>(p.flag_rows + units * max_evict);
  p.panel = reinterpret_cast<const unsigned char*>(workspace) + pl.panel_off;
  p.exact_partial = reinterpret_cast<ExactPartial*>(reinterpret_cast<char*>(workspace) + pl.partial_off);
  p.exact_ticket = reinterpret_cast<int32_t*>(workspace);
  p.causal = 0; p.len = cache->len;
  p.small_parts = 1;
  p.small_partial = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.small_partial_off);
  p.match = match; p.sim_out = sim_out;
  p.capacity = cache->capacity; p.budget = budget; p.max_evict = max_evict;
  p.threshold = threshold;
  p.per_unit = 0; p.n_units = 0;   // set by the first event's launch
  // Margin below which the f32 result does not decide a row.  An f32 similarity carries the accumulation of
  // D exact products (at most D * 2^-24 relative to |k_e||k_c|, far less in practice) and the roundings of
  // the two norms; what is compared are two such values, or one and the threshold.
  p.delta = 1.6e-5f;

  p.rn_pitch = rn_pitch_of(budget);
  long eb = (long)units * max_evict / 16;      // queued rows are a small fraction of all rows
  const int exact_blocks = (int)(eb < 64 ? 64 : (eb > 512 ? 512 : eb));
  if (max_evict <= kSmallMaxEvict || layout->dtype != KEEPKV_BF16) p.panel = nullptr;   // only the first event's path gathers it
  if (layout->dtype == KEEPKV_BF16) {
    keepkv_status rc;
    if (layout->head_dim == 128) {
      rc = launch_bf16<128>(p, cache->k, (unsigned)units, st);
      if (rc != KEEPKV_OK) return rc;
      if (max_evict <= kSmallMaxEvict) match_exact_bf16_kernel<128><<<exact_blocks, 256, 0, st>>>(p);
      else match_recheck_kernel<128><<<exact_blocks, 256, 0, st>>>(p);
    } else {
      rc = launch_bf16<64>(p, cache->k, (unsigned)units, st);
      if (rc != KEEPKV_OK) return rc;
      if (max_evict <= kSmallMaxEvict) match_exact_bf16_kernel<64><<<exact_blocks, 256, 0, st>>>(p);
      else match_recheck_kernel<64><<<exact_blocks, 256, 0, st>>>(p);
    }
  } else {
    launch_exact_f32(p, units, layout->head_dim, budget, st);
  }
  return launch_status();
}

#ifdef KEEPKV_TRACE
extern "C" int keepkv_trace_read_match(long long* host, int n) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(kk::kk_trace_match), sizeof(long long) * n);
}
#endif
