// keepkv_select: per (batch, kv head) choose the retained set K_c and the to-be-evicted set K_e
// (Alg. 1, selection step) under the fixed-budget sink / recent / heavy-hitter policy (App. B.3).
//
// One 1024-thread workgroup per head; the (budget - n_sink - n_recent) slots with the largest ranking values
// ln p + ln s_hat (f64, equal values at lower indices first) are found and the slots compacted in index order.
//
// Up to 32768 slots (select_kernel) the values are formed in f32 and kept in registers, a wavefront a contiguous
// run of slots.  A histogram over kBins equal intervals of their range (a few outliers left out) gives the interval
// in which the threshold lies; slots more than the f32 arithmetic's error away from it are decided, the few others
// are evaluated in f64 and ranked exactly by counting.  The f64 value is some sixty instructions per slot, which
// bound the kernel when every slot was given one.  An interval with more than kRankSoon slots (skewed values, values
// spread over many orders of magnitude) is split again by the values' integer images, at most three times; a long run of
// equal values is kept in slot order.  Only when more than kMaxCand slots are so close that f32 cannot tell them apart
// though they differ, or a value is NaN, and for longer caches
// (select_long_kernel), the f64 values of all slots are mapped to order-preserving u64 keys in the workspace and the
// threshold is found by an 8-bit most-significant-digit radix select (LDS histograms, wavefront scan; digits in
// which no two keys differ are skipped).
// What bounds it: the latency of its steps (loads, block reduction, histogram, scan, ranking, two compaction sweeps).
// Measured (MI355X, graph replays), radix select over all f64 keys / now: 8 heads x 32768 slots 66 / 33.5 us, 64 x 8192
// 20.1 / 13.4, 64 x 884 8.1 / 7.0.  64 x 8192 by a caller's ranks: normal 16.3 / 10.1, exponential with three huge ones
// 16.2 / 10.1 (27.5 when all of a crowded interval went to the radix select), all equal 12.3 / 9.9 (25.0), log-normal with
// sigma 5 16.9 / 12.1 (29.5); 64 x 884: exponential 6.9 / 6.0, log-normal with sigma 5 6.4 / 7.8.
#include "kk_common.hpp"

namespace kk {
// Phase timestamps for kernel tuning; compiled in only with -DKEEPKV_TRACE (never in the product build).
#ifdef KEEPKV_TRACE
__device__ long long kk_trace_select[16 * 1024];
#define KS_TS(i) do { if (threadIdx.x == 0 && blockIdx.x < 1024) kk_trace_select[blockIdx.x * 16 + (i)] = wall_clock64(); } while (0)
#else
#define KS_TS(i) do { } while (0)
#endif
namespace {

constexpr int kSelThreads = 1024;
constexpr int kVotesTable = 256;       // ln p is tabulated for vote counts below this
constexpr int kTermTable = 2048;       // ln(1 - alpha^n) is tabulated for n below this (alpha up to 0.98 in full)

__device__ __attribute__((noinline)) double log_f64(double x) { return log(x); }
__device__ __attribute__((noinline)) double log_1m_exp_f64(double t) { return log(-expm1(t)); }

__device__ __forceinline__ uint64_t sortable_u64(double x) {
  x = x + 0.0;  // -0.0 -> +0.0
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// OR over the wavefront, delivered to every lane (quad swaps, mirrors within 8 and 16 lanes, then two exchanges)
__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
  x |= dpp_u32<0xB1>(x);
  x |= dpp_u32<0x4E>(x);
  x |= dpp_u32<0x141>(x);
  x |= dpp_u32<0x140>(x);
  x |= (uint32_t)__shfl_xor((int)x, 16);
  x |= (uint32_t)__shfl_xor((int)x, 32);
  return x;
}

// inclusive prefix sum over the wavefront in lane order: shifts within each row of 16 lanes (lanes without a
// source add zero), then lane 15 of rows 0 and 2 is added to rows 1 and 3, then lane 31 to rows 2 and 3
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int x) {
  return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, true);
}
__device__ __forceinline__ int wave_incl_scan(int x) {
  x = dpp_add<0x111, 0xF>(x);   // row_shr:1
  x = dpp_add<0x112, 0xF>(x);   // row_shr:2
  x = dpp_add<0x114, 0xF>(x);   // row_shr:4
  x = dpp_add<0x118, 0xF>(x);   // row_shr:8
  x = dpp_add<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
  x = dpp_add<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
  return x;
}

// number of set bits of `mask` below the calling lane
__device__ __forceinline__ int rank_in_wave(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// EXT: the ranking value is read from a caller-supplied array (passed as log_s; born, t_obs and votes
// unused) instead of being formed from the cache's votes and EMA scores.
// AGED: the live slots are not in age order.  `order` lists the slots below `budget` from oldest to newest and
// the slots from `budget` on follow in slot order (tokens appended since the last in-place event); the whole
// selection runs on the age rank i and reads and reports slot(i), so the lists come out in age order.
// Called by all threads of a head's workgroup; n = the head's length > budget.
struct SelectParams {
  const float* log_s;
  const int32_t *born, *t_obs, *votes, *len;
  uint64_t* keys;
  int32_t *keep_idx, *evict_idx, *n_evict;
  int capacity, budget, n_sink, n_recent;
  double ln_alpha;
  int n_table;               // counts below this have a tabulated ln(1 - alpha^n)
  const int32_t* order;
};
template <bool EXT, bool AGED>
__device__ __forceinline__ void select_radix(const SelectParams& p, int unit, int n) {
  const float* log_s = p.log_s;
  const int32_t *born = p.born, *votes = p.votes;
  const int capacity = p.capacity, budget = p.budget, n_sink = p.n_sink, n_recent = p.n_recent, n_table = p.n_table;
  const double ln_alpha = p.ln_alpha;
  constexpr int kWaves = kSelThreads / 64;
  __shared__ double s_lnterm[EXT ? 1 : kTermTable];
  __shared__ double s_lnvotes[EXT ? 1 : kVotesTable];
  __shared__ int s_hist[256];
  __shared__ int s_eq[kWaves], s_kept[kWaves];
  __shared__ uint64_t s_or[kWaves], s_nand[kWaves];
  __shared__ int s_digit, s_need, s_bucket;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t base = (size_t)unit * capacity;
  const int32_t* ord = AGED ? p.order + (size_t)unit * budget : nullptr;
  auto slot_of = [&](int i) -> int {              // age rank -> slot
    if constexpr (AGED) return i < budget ? min(max(ord[i], 0), capacity - 1) : i;   // (clamped: never out of bounds)
    else return i;
  };
  const int lo = n_sink;
  int nn[4], pv[4];
  float ls[4];
  uint64_t k_or = 0, k_nand = 0;              // OR of this thread's keys and of their complements
  auto request = [&](int i0) {
    int sl[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) sl[u] = slot_of(min(i0 + u * kSelThreads, capacity - 1));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = sl[u];
      nn[u] = EXT ? 0 : born[base + i];          // turned into the observation count t_obs - born at its use
      pv[u] = EXT ? 1 : votes[base + i];
      ls[u] = log_s[base + i];
    }
  };
  request(lo + tid);
  const int t_head = EXT ? 1 : p.t_obs[unit];
  int32_t* keep_out = p.keep_idx + (size_t)unit * budget;
  int32_t* evict_out = p.evict_idx + (size_t)unit * (capacity - budget);
  // ln(1 - alpha^n) depends on the observation count alone, and the f64 library routines behind it are some
  // hundreds of instructions: one evaluation per count (n_table of them: beyond, the term rounds to zero)
  // instead of one per slot
  if constexpr (!EXT) {
    for (int m = tid; m < n_table; m += kSelThreads) s_lnterm[m] = m > 0 ? log_1m_exp_f64((double)m * ln_alpha) : 0.0;
    // (the last wavefronts take the votes table: the first ones have the other one's entries)
    if (tid >= kSelThreads - kVotesTable) s_lnvotes[kSelThreads - 1 - tid] = log_f64((double)(kSelThreads - 1 - tid));
    __syncthreads();
  }
  uint64_t* key_g = p.keys + base;
  auto key = [&](int i) -> uint64_t& { return key_g[i]; };
  const int hi = n - n_recent;   // candidates are [lo, hi)
  const int n_heavy = budget - n_sink - n_recent;

  for (int i0 = lo + tid; i0 < hi; i0 += 4 * kSelThreads) {     // four slots per round trip
    double x[4];
    if (EXT) {
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = (ls[u] == ls[u]) ? (double)ls[u] : -INFINITY;     // NaN ranks lowest
    } else {
      // ln p + ln S - ln(1 - alpha^n), the two logarithms from the tables; a wavefront evaluates them itself
      // only where one of its lanes has a count beyond a table.
#pragma unroll
      for (int u = 0; u < 4; ++u) nn[u] = t_head - nn[u];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool valid = i0 + u * kSelThreads < hi;
        const double t = (double)nn[u] * ln_alpha;
        x[u] = (double)ls[u];
        const bool small_p = pv[u] >= 1 && pv[u] < kVotesTable;
        if (__any(valid && !small_p)) x[u] = (small_p ? s_lnvotes[pv[u]] : log_f64((double)pv[u])) + x[u];
        else x[u] = s_lnvotes[small_p ? pv[u] : 1] + x[u];
        const bool need = t > -40.0, listed = nn[u] > 0 && nn[u] < n_table;
        double term = (need && listed) ? s_lnterm[nn[u]] : 0.0;
        if (__any(valid && need && !listed)) term = (need && !listed) ? log_1m_exp_f64(t) : term;   // alpha close to 1
        x[u] -= term;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (nn[u] <= 0) x[u] = -INFINITY;
    }
    if (i0 + 4 * kSelThreads < hi) request(i0 + 4 * kSelThreads);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * kSelThreads;
      if (i < hi) {
        const uint64_t k = sortable_u64(x[u]);
        key(i) = k;
        k_or |= k;
        k_nand |= ~k;
      }
    }
  }
  // which bits differ between any two candidate keys of the head
  {
    const uint32_t o_lo = wave_or((uint32_t)k_or), o_hi = wave_or((uint32_t)(k_or >> 32));
    const uint32_t a_lo = wave_or((uint32_t)k_nand), a_hi = wave_or((uint32_t)(k_nand >> 32));
    if (lane == 0) {
      s_or[wave] = ((uint64_t)o_hi << 32) | o_lo;
      s_nand[wave] = ((uint64_t)a_hi << 32) | a_lo;
    }
  }
  if (tid < 256) s_hist[tid] = 0;
  __syncthreads();
  uint64_t all_or = 0, all_nand = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    all_or |= s_or[w];
    all_nand |= s_nand[w];
  }
  const uint64_t varying = all_or & all_nand;      // a bit that is 1 in some key and 0 in another

  // ---- radix select: tau = n_heavy-th largest key, need = how many keys equal to tau are kept.
  // A digit in which no two keys differ (the sign and exponent bits, as a rule) needs no histogram: it would
  // put every candidate into one bin, and same-address LDS atomics are served one lane at a time.
  uint64_t prefix = 0;
  int need = n_heavy;
  if (n_heavy > 0) {
    int n_cand = hi - lo;                             // keys that agree with the prefix so far
    bool first_hist = true;
    for (int pass = 7; pass >= 0; --pass) {
      const int shift = 8 * pass;
      int digit, bucket;
      if (((varying >> shift) & 255u) == 0) {
        digit = (int)((all_or >> shift) & 255u);
        bucket = n_cand;
      } else {
        // s_hist is zero here: cleared before the keys' barrier, and by the scan below after each use
        for (int i0 = lo + tid; i0 < hi; i0 += 4 * kSelThreads) {   // four keys per round trip
          uint64_t k4[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) k4[u] = key(min(i0 + u * kSelThreads, hi - 1));
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint64_t k = k4[u];
            const bool in = (i0 + u * kSelThreads < hi) && (first_hist || ((k >> (shift + 8)) == prefix));
            const int d = (int)((k >> shift) & 255u);
            // leading digits are shared by most keys: the lanes that agree with the first lane's digit add
            // their count once instead of queueing on one LDS word
            const uint64_t act = __ballot(in);
            if (act != 0) {
              const int first = __ffsll((long long)act) - 1;
              const int d0 = __builtin_amdgcn_readlane(d, first);
              const uint64_t same = __ballot(in && d == d0);
              if (in && d != d0) atomicAdd(&s_hist[d], 1);
              if (lane == first) atomicAdd(&s_hist[d0], __popcll(same));
            }
          }
        }
        first_hist = false;
        __syncthreads();
        if (tid < 64) {
          // lane covers digits 255-4*lane .. 252-4*lane, i.e. descending order over lanes
          int c[4], t = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            c[j] = s_hist[255 - 4 * tid - j];
            s_hist[255 - 4 * tid - j] = 0;
            t += c[j];
          }
          const int incl = wave_incl_scan(t);
          const uint64_t mask = __ballot(incl >= need);
          const int first = __ffsll((long long)mask) - 1;   // mask != 0: the candidates outnumber `need`
          if (tid == first) {
            int run = incl - t;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (run + c[j] >= need) {
                s_digit = 255 - 4 * tid - j;
                s_need = need - run;
                s_bucket = c[j];
                break;
              }
              run += c[j];
            }
          }
        }
        __syncthreads();          // s_digit is next written behind the next histogram's barrier
        digit = s_digit;
        need = s_need;
        bucket = s_bucket;
      }
      prefix = (prefix << 8) | (uint64_t)digit;
      n_cand = bucket;
      if (bucket == need && pass > 0 && prefix != 0) {
        // every key with this prefix is kept: stop refining and keep exactly the keys >= prefix << shift,
        // i.e. key > tau with no equal keys to count (prefix != 0: the candidates outnumber `need`)
        prefix = (prefix << shift) - 1;
        need = 0;
        break;
      }
    }
  }
  const uint64_t tau = prefix;
  const int need_eq = need;

  // ---- ordered compaction ------------------------------------------------------------------------
  // A wavefront owns a run of 64-slot chunks, lane = slot within the chunk; positions inside a chunk come
  // from a ballot, the wavefronts exchange their totals through LDS.  Equal keys are kept lowest index first.
  const int n_chunks = (n + 63) >> 6;
  const int cpw = (n_chunks + kWaves - 1) / kWaves;
  const int c0 = min(n_chunks, wave * cpw), c1 = min(n_chunks, c0 + cpw);
  const bool count_equal = n_heavy > 0 && need_eq > 0;          // uniform over the workgroup
  int eq_run = 0;
  if (count_equal) {
    int cnt = 0;
    for (int c = c0; c < c1; ++c) {
      const int i = c * 64 + lane;
      cnt += __popcll(__ballot(i >= lo && i < hi && key(i) == tau));
    }
    if (lane == 0) s_eq[wave] = cnt;
    __syncthreads();
    for (int w = 0; w < wave; ++w) eq_run += s_eq[w];          // equal keys at lower indices
  }
  // which slots of chunk c are kept; eq advances over the chunk's equal keys
  auto kept_mask = [&](int c, int& eq) -> uint64_t {
    const int i = c * 64 + lane;
    const bool cand = i >= lo && i < hi;
    const uint64_t k = (cand && n_heavy > 0) ? key(i) : 0;
    bool kept = i < n && (!cand || (n_heavy > 0 && k > tau));
    if (count_equal) {                                          // every lane takes part in the ballot
      const bool is_eq = cand && k == tau;
      const uint64_t m_eq = __ballot(is_eq);
      if (is_eq) kept = eq + rank_in_wave(m_eq) < need_eq;
      eq += __popcll(m_eq);
    }
    return __ballot(kept);
  };
  int nk = 0, eq = eq_run;
  for (int c = c0; c < c1; ++c) nk += __popcll(kept_mask(c, eq));
  if (lane == 0) s_kept[wave] = nk;
  __syncthreads();
  int kpos = 0;
  for (int w = 0; w < wave; ++w) kpos += s_kept[w];            // kept slots at lower indices
  eq = eq_run;
  for (int c = c0; c < c1; ++c) {
    const int i = c * 64 + lane;
    const uint64_t m = kept_mask(c, eq);
    const int at = kpos + rank_in_wave(m);
    if (i < n) {
      const int s = slot_of(i);
      if ((m >> lane) & 1) keep_out[at] = s;
      else evict_out[i - at] = s;
    }
    kpos += __popcll(m);
  }
  if (tid == 0) p.n_evict[unit] = n - budget;
}

// a head that evicts nothing
template <bool AGED>
__device__ __forceinline__ void select_nothing(const SelectParams& p, int unit, int n) {
  const int32_t* ord = AGED ? p.order + (size_t)unit * p.budget : nullptr;
  for (int i = threadIdx.x; i < p.budget; i += kSelThreads)
    p.keep_idx[(size_t)unit * p.budget + i] = (i < n) ? (AGED ? min(max(ord[i], 0), p.capacity - 1) : i) : -1;
  if (threadIdx.x == 0) p.n_evict[unit] = 0;
}

template <bool EXT, bool AGED>
__global__ __launch_bounds__(kSelThreads) void select_long_kernel(SelectParams p) {
  const int unit = blockIdx.x, n = p.len[unit];
  if (n <= p.budget) select_nothing<AGED>(p, unit, n);
  else select_radix<EXT, AGED>(p, unit, n);
}

// ---------------------------------------------------------------------------------------------------
constexpr int kBinBits = 11, kBins = 1 << kBinBits;
constexpr int kMaxCand = 256;          // undecided slots that are ranked by counting, at most
constexpr int kRankSoon = 128;         // up to this many rather than splitting their interval again

// over the 16 lanes of equal number modulo 4; over the four lanes of a quad
template <typename F>
__device__ __forceinline__ float class_reduce(float x, F f) {
  x = f(x, dpp_f32<0x124>(x));   // row_ror:4
  x = f(x, dpp_f32<0x128>(x));   // row_ror:8
  x = f(x, __shfl_xor(x, 16));
  return f(x, __shfl_xor(x, 32));
}
template <typename F>
__device__ __forceinline__ float quad_reduce(float x, F f) {
  x = f(x, dpp_f32<0xB1>(x));
  return f(x, dpp_f32<0x4E>(x));
}
template <typename F>
__device__ __forceinline__ float wave_reduce_f32(float x, F f) {
  x = f(x, dpp_f32<0xB1>(x));
  x = f(x, dpp_f32<0x4E>(x));
  x = f(x, dpp_f32<0x141>(x));
  x = f(x, dpp_f32<0x140>(x));
  x = f(x, __shfl_xor(x, 16));
  return f(x, __shfl_xor(x, 32));
}

template <typename F>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t x, F f) {
  return (uint32_t)__builtin_bit_cast(int, wave_reduce_f32(__builtin_bit_cast(float, x), [&](float a, float b) {
    return __builtin_bit_cast(float, f(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b)));
  }));
}
// order-preserving integer image of an f32 value (both zeros the same), and back
__device__ __forceinline__ uint32_t sortable_u32(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x == 0.f ? 0.f : x);
  return (u >> 31) != 0 ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float from_sortable_u32(uint32_t u) {
  return __builtin_bit_cast(float, (u >> 31) != 0 ? u & 0x7FFFFFFFu : ~u);
}

// ITEMS: chunks of 64 slots per wavefront that the registers hold; chunk c of wavefront w is the slots
// (w * cpw + c) * 64 + lane, cpw = ceil(capacity / 1024) <= ITEMS.
template <bool EXT, bool AGED, int ITEMS>
__global__ __launch_bounds__(kSelThreads, ITEMS <= 8 ? 8 : 4) void select_kernel(SelectParams p) {
  constexpr int kWaves = kSelThreads / 64;
  __shared__ float s_term[EXT ? 1 : kTermTable];
  __shared__ float s_lnp[EXT ? 1 : kVotesTable];
  __shared__ int s_hist[kBins];
  __shared__ double s_cand[kMaxCand];
  __shared__ int s_cand_i[kMaxCand];
  __shared__ unsigned long long s_bits[ITEMS * kWaves];    // undecided slots that are kept, by chunk
  __shared__ float s_min[kWaves * 4], s_max[kWaves * 4];
  __shared__ uint32_t s_umin[kWaves], s_umax[kWaves];
  __shared__ int s_wave[kWaves], s_above[kWaves];
  __shared__ int s_bin, s_count, s_need, s_n_cand, s_n_again, s_nan, s_ref;

  const int unit = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  KS_TS(0);
  const int capacity = p.capacity, budget = p.budget;
  const size_t base = (size_t)unit * capacity;
  const int32_t* ord = AGED ? p.order + (size_t)unit * budget : nullptr;
  const int cpw = (capacity + kSelThreads - 1) / kSelThreads;
  const int first = wave * cpw * 64 + lane;                          // this thread's slots: first + 64 c, c < cpw
  auto slot_of = [&](int i) -> int {              // age rank -> slot
    if constexpr (AGED) return i < budget ? min(max(ord[i], 0), capacity - 1) : i;   // (clamped: never out of bounds)
    else return i;
  };
  // the state of the first kLoad slots is requested together with the head's length
  constexpr int kLoad = ITEMS < 8 ? ITEMS : 8;
  int nn[kLoad], pv[kLoad];
  float ls[kLoad];
  auto request = [&](int c0) {
    int sl[kLoad];
#pragma unroll
    for (int u = 0; u < kLoad; ++u) sl[u] = slot_of(min(first + 64 * (c0 + u), capacity - 1));
#pragma unroll
    for (int u = 0; u < kLoad; ++u) {
      nn[u] = EXT ? 0 : p.born[base + sl[u]];     // turned into the observation count t_obs - born at its use
      pv[u] = EXT ? 1 : p.votes[base + sl[u]];
      ls[u] = p.log_s[base + sl[u]];
    }
  };
  request(0);
  const int t_head = EXT ? 1 : p.t_obs[unit];
  const int n = p.len[unit];
  // f32 tables of ln p and of ln(1 - alpha^n), which depends on the observation count alone
  if constexpr (!EXT) {
    for (int m = tid; m < p.n_table; m += kSelThreads) s_term[m] = m > 0 ? logf(-expm1f((float)((double)m * p.ln_alpha))) : 0.f;
    // (the last wavefronts take the votes table: the first ones have the other one's entries)
    if (tid >= kSelThreads - kVotesTable) s_lnp[kSelThreads - 1 - tid] = logf((float)(kSelThreads - 1 - tid));
  }
  for (int b = tid; b < kBins; b += kSelThreads) s_hist[b] = 0;
  for (int w = tid; w < ITEMS * kWaves; w += kSelThreads) s_bits[w] = 0;
  if (tid == 0) s_n_cand = s_n_again = s_nan = 0;
  if (n <= budget) {                              // uniform over the workgroup
    select_nothing<AGED>(p, unit, n);
    return;
  }
  __syncthreads();
  KS_TS(13);
  const int lo = p.n_sink, hi = n - p.n_recent;   // candidates are [lo, hi)
  const int n_heavy = budget - p.n_sink - p.n_recent;

  // ---- ranking values in f32, the least and the largest finite one
  float y[ITEMS] = {};
  float vmin = INFINITY, vmax = -INFINITY;
  bool nan = false;                               // a ranking value is NaN: where it ranks depends on its f64 image
#pragma unroll
  for (int c0 = 0; c0 < ITEMS; c0 += kLoad) {
    if (c0 < cpw) {                               // uniform over the workgroup
#pragma unroll
      for (int u = 0; u < kLoad; ++u) {
        const int i = first + 64 * (c0 + u);
        const bool cand = c0 + u < cpw && i >= lo && i < hi;
        float x = ls[u];
        if constexpr (EXT) {
          x = (x == x) ? x : -INFINITY;           // NaN ranks lowest
        } else {
          // a wavefront evaluates the logarithms itself only where one of its lanes has a count beyond a table
          const int cnt = t_head - nn[u];
          const bool small_p = (uint32_t)pv[u] < (uint32_t)kVotesTable;
          float lp = s_lnp[small_p ? pv[u] : 1];
          if (__any(cand && !small_p)) lp = small_p ? lp : logf((float)pv[u]);
          float term = (cnt > 0 && cnt < p.n_table) ? s_term[cnt] : 0.f;
          if (p.n_table == kTermTable && __any(cand && cnt >= kTermTable))     // alpha close to 1
            term = cnt >= kTermTable ? logf(-expm1f((float)((double)cnt * p.ln_alpha))) : term;
          x = (lp + x) - term;
          x = cnt <= 0 ? -INFINITY : x;
          nan |= cand && !(x == x);
        }
        y[c0 + u] = x;
        const bool finite = cand && fabsf(x) <= 3.0e38f;
        vmin = finite ? fminf(vmin, x) : vmin;
        vmax = finite ? fmaxf(vmax, x) : vmax;
      }
      if (c0 + kLoad < ITEMS && c0 + kLoad < cpw) request(c0 + kLoad);
    }
  }
  // by classes of equal slot number modulo 4
  auto least = [](float a, float b) { return fminf(a, b); };
  auto largest = [](float a, float b) { return fmaxf(a, b); };
  vmin = class_reduce(vmin, least);
  vmax = class_reduce(vmax, largest);
  if (lane < 4) {
    s_min[wave * 4 + lane] = vmin;
    s_max[wave * 4 + lane] = vmax;
  }
  if (!EXT && __any(nan)) s_nan = 1;              // (any lane)
  __syncthreads();
  KS_TS(1);

  // What is the same in all lanes goes through a scalar register: the branches below hold barriers and ballots, and are to be
  // branches of the whole wavefront in the compiler's eyes too (it moved register copies of an outer branch under the lane
  // mask of an inner one otherwise).
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  auto uniform_f = [&](float x) { return __builtin_bit_cast(float, uniform(__builtin_bit_cast(int, x))); };
  // bit c: slot first + 64 c is a candidate / is kept / is undecided
  uint32_t cand = 0, keep = 0, und = 0;
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int i = c < cpw ? first + 64 * c : n;
    if (i >= lo && i < hi) cand |= 1u << c;
    else if (i < n) keep |= 1u << c;
  }
  bool radix = !EXT && uniform(s_nan) != 0;       // left to the radix select
  const uint32_t keep_always = keep;
  // Adds the slots of `set` to the histogram.  Where many lanes of the wavefront's first chunk share an interval, the lanes
  // that agree with the first one add their count once in every chunk: adds to one LDS word are served a lane at a time.
  auto add_to_histogram = [&](uint32_t set, auto bin_of) {
    bool crowded = false;
#pragma unroll
    for (int c = 0; c < ITEMS; ++c) {
      if (c < cpw) {                              // uniform
        const bool in = (set >> c) & 1;
        const int b = bin_of(c);
        if (c == 0 || crowded) {                  // uniform
          const uint64_t act = __ballot(in);
          const int leader = act != 0 ? __ffsll((long long)act) - 1 : 0;
          const int b0 = __builtin_amdgcn_readlane(b, leader);
          const uint64_t same = __ballot(in && b == b0);
          if (c == 0) crowded = __popcll(same) >= 16;
          if (in && b != b0) atomicAdd(&s_hist[b], 1);
          if (act != 0 && lane == leader) atomicAdd(&s_hist[b0], __popcll(same));
        } else if (in) {
          atomicAdd(&s_hist[b], 1);
        }
      }
    }
  };
  // The boundary interval: the one in which the running count from the top reaches `need`; s_bin, its slots (s_count) and how many
  // of them are needed (s_need).
  auto find_boundary = [&](int need) {
    constexpr int kPer = kBins / kSelThreads;
    int cnt[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {              // thread 0 has the top intervals
      cnt[j] = s_hist[kBins - 1 - (tid * kPer + j)];
      s_hist[kBins - 1 - (tid * kPer + j)] = 0;   // for the next histogram
      sum += cnt[j];
    }
    const int incl = wave_incl_scan(sum);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = incl - sum;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) before += w < wave ? s_wave[w] : 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (before < need && before + cnt[j] >= need) {   // exactly one
        s_bin = kBins - 1 - (tid * kPer + j);
        s_count = cnt[j];
        s_need = need - before;
      }
      before += cnt[j];
    }
    __syncthreads();
  };
  auto list_undecided = [&](int& count) {
#pragma unroll
    for (int c = 0; c < ITEMS; ++c)
      if ((und >> c) & 1) {
        const int at = atomicAdd(&count, 1);
        if (at < kMaxCand) s_cand_i[at] = first + 64 * c;
      }
  };

  int m = 0;                                      // slots left to rank
  if (n_heavy > 0 && !radix) {                    // uniform
    // The histogram's range: from the largest of the four classes' least values to the least of their largest ones.  A few
    // outliers, which leave some class without one, do not stretch it; a handful of slots lies outside, in the end intervals.
    static_assert(kWaves * 4 == 64, "one value a lane");
    vmin = quad_reduce(class_reduce(s_min[lane], least), largest);
    vmax = quad_reduce(class_reduce(s_max[lane], largest), least);
    vmin = uniform_f(vmin);
    vmax = uniform_f(vmax);
    const float range = vmax - vmin;
    const float scale = range > 1e-30f && range < 3.0e38f ? (float)kBins / range : 0.f;   // 0: no such range
    auto coordinate = [&](float x) { return (x - vmin) * scale; };
    auto interval = [&](float x) {                // (the outermost ones also hold the values outside)
      const float t = coordinate(x);
      return t >= (float)kBins ? kBins - 1 : (t > 0.f ? (int)t : 0);
    };
    bool fine = scale == 0.f;                     // the equal intervals are too coarse
    if (!fine) {
      add_to_histogram(cand, [&](int c) { return interval(y[c]); });
      __syncthreads();
      KS_TS(2);
      find_boundary(n_heavy);
      KS_TS(3);
      fine = uniform(s_count) > kRankSoon;
    }
    if (!fine) {
      const int bin = uniform(s_bin);
      // The f32 values carry the roundings of two sums and of two logarithms whose magnitudes (at most 22 and 24) do not
      // show in the sum: within (magnitude + 64) * 2^-21 of the f64 values, and the coordinate its own two
      // roundings (below 1e-3 intervals).  With e that bound in intervals at the magnitude of the range's ends, the f64 threshold
      // lies within e of the boundary interval (counting the f32 values from either side), so a slot 2 e outside is decided
      // (one of larger magnitude too: its distance grows with it, the bound 2^21 times slower).
      const float mag = fmaxf(fabsf(vmin), fabsf(vmax));
      const float e2 = EXT ? 0.f : 2.f * ((mag + 64.f) * 4.8e-7f * scale + 1e-3f);
      const float t_lo = bin == 0 ? -INFINITY : (float)bin - e2;
      float t_hi = bin == kBins - 1 ? INFINITY : (float)(bin + 1) + e2;
      if (EXT && bin != kBins - 1) t_hi = __builtin_bit_cast(float, __builtin_bit_cast(int, t_hi) - 1);   // below bin + 1
#pragma unroll
      for (int c = 0; c < ITEMS; ++c) {
        const float t = coordinate(y[c]);
        const uint32_t bit = cand & (1u << c);
        keep |= t > t_hi ? bit : 0u;
        und |= t >= t_lo && t <= t_hi ? bit : 0u;
      }
      list_undecided(s_n_cand);
      const int n_above = wave_incl_scan(__popc(keep & cand));
      if (lane == 63) s_above[wave] = n_above;
      __syncthreads();
      m = uniform(s_n_cand);
      fine = m > kRankSoon;                       // (the f32 error reaches into crowded neighbours)
    }
    if (__builtin_expect(fine, 0)) {              // uniform
      // The boundary interval is split again, into equal intervals of the values' order-preserving integer images between
      // the least and the largest in it, until few slots or equal values are left: three times at most.
      int need = n_heavy, left = n;
      uint32_t u_lo = 0xFFFFFFFFu, u_hi = 0;
      const int bin0 = uniform(s_bin);
      if (scale != 0.f) {
        need = uniform(s_need);
        left = uniform(s_count);
      }
      uint32_t image[ITEMS];
#pragma unroll
      for (int c = 0; c < ITEMS; ++c) {
        image[c] = sortable_u32(y[c]);
        if (((cand >> c) & 1) && (scale == 0.f || interval(y[c]) == bin0)) {
          u_lo = min(u_lo, image[c]);
          u_hi = max(u_hi, image[c]);
        }
      }
      u_lo = wave_reduce_u32(u_lo, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
      u_hi = wave_reduce_u32(u_hi, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
      if (lane == 0) {
        s_umin[wave] = u_lo;
        s_umax[wave] = u_hi;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        u_lo = min(u_lo, s_umin[w]);
        u_hi = max(u_hi, s_umax[w]);
      }
      u_lo = (uint32_t)uniform((int)u_lo);
      u_hi = (uint32_t)uniform((int)u_hi);
      while (u_lo != u_hi && left > (EXT ? kRankSoon : kRankSoon / 2)) {   // uniform (not EXT: room for neighbours)
        const int bits = 32 - __clz((int)(u_hi - u_lo)), shift = bits > kBinBits ? bits - kBinBits : 0;
        uint32_t in = 0;
#pragma unroll
        for (int c = 0; c < ITEMS; ++c) in |= image[c] - u_lo <= u_hi - u_lo ? cand & (1u << c) : 0u;
        add_to_histogram(in, [&](int c) { return (int)((image[c] - u_lo) >> shift); });
        __syncthreads();
        find_boundary(need);
        need = uniform(s_need);
        left = uniform(s_count);
        u_lo += (uint32_t)uniform(s_bin) << shift;
        u_hi = min(u_hi, u_lo + ((1u << shift) - 1u));
      }
      // kept: above the interval; undecided: in it, or within the f32 error of it (as above, with the magnitude there)
      keep = keep_always;
      und = 0;
      const bool run = u_lo == u_hi;
      bool equal = run;                           // the undecided values are equal in f64 too
      if constexpr (!EXT) {
        float y_lo = from_sortable_u32(u_lo), y_hi = from_sortable_u32(u_hi);
        const bool fin_lo = fabsf(y_lo) < INFINITY, fin_hi = fabsf(y_hi) < INFINITY;
        const float mag = fmaxf(fin_lo ? fabsf(y_lo) : 0.f, fin_hi ? fabsf(y_hi) : 0.f);
        const float e2 = 2.02f * 4.8e-7f * (mag + 64.f);
        equal = run && !fin_lo;
        u_lo = sortable_u32(fin_lo ? y_lo - e2 : y_lo);
        u_hi = sortable_u32(fin_hi ? y_hi + e2 : y_hi);
      }
#pragma unroll
      for (int c = 0; c < ITEMS; ++c) {
        const uint32_t bit = cand & (1u << c);
        keep |= image[c] > u_hi ? bit : 0u;
        und |= image[c] >= u_lo && image[c] <= u_hi ? bit : 0u;
      }
      const int n_und = wave_incl_scan(__popc(und)), n_above = wave_incl_scan(__popc(keep & cand));
      if (lane == 63) {
        s_wave[wave] = n_und;
        s_above[wave] = n_above;
      }
      if (!equal) list_undecided(s_n_again);
      __syncthreads();
      m = uniform(s_n_again);
      if (equal || run || m > kMaxCand) {         // uniform
        // Equal values, or a run that may be one (the same score, votes and count in all slots): the first ones in slot order.
        bool same = true;
        if (!equal) {                             // uniform
          if (und != 0) s_ref = first + 64 * (__ffs((int)und) - 1);   // any of them
          __syncthreads();
          const size_t ref = base + slot_of(s_ref);
          const int ls_r = __builtin_bit_cast(int, p.log_s[ref]), pv_r = p.votes[ref], born_r = p.born[ref];
          int differs = 0;
#pragma unroll 1
          for (int c0 = 0; c0 < cpw; c0 += 4)     // (four slots a round trip; not listed: the reference again)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int i = c0 + u < ITEMS && ((und >> (c0 + u)) & 1) ? first + 64 * (c0 + u) : s_ref;
              const size_t at = base + slot_of(i);
              differs |= (__builtin_bit_cast(int, p.log_s[at]) ^ ls_r) | (p.votes[at] ^ pv_r) | (p.born[at] ^ born_r);
            }
          same = uniform(__syncthreads_or(differs)) == 0;
        }
        if (same) {                               // uniform
          int before = 0, want = n_heavy;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            before += w < wave ? s_wave[w] : 0;
            want -= s_above[w];
          }
#pragma unroll
          for (int c = 0; c < ITEMS; ++c)
            if (c < cpw) {                        // uniform
              const uint64_t mask = __ballot((und >> c) & 1);
              if (((und >> c) & 1) && before + rank_in_wave(mask) < want) keep |= 1u << c;
              before += __popcll(mask);
            }
          m = 0;
          __syncthreads();                        // s_wave has been read
        } else {
          radix = m > kMaxCand;
        }
      }
    }
  }
  if (__builtin_expect(radix, 0)) {               // uniform
    select_radix<EXT, AGED>(p, unit, n);
    return;
  }
  if (m > 0) {                                    // uniform: the listed slots' f64 values, ranked by counting
    int need = n_heavy;                           // how many of them are kept
#pragma unroll
    for (int w = 0; w < kWaves; ++w) need -= s_above[w];
    if (tid < m) {
      const int i = s_cand_i[tid];
      const size_t at = base + slot_of(i);
      double x = (double)p.log_s[at];
      if constexpr (EXT) {
        if (!(x == x)) x = -INFINITY;
      } else {
        const int cnt = t_head - p.born[at];
        const double t = (double)cnt * p.ln_alpha;
        const int pv_i = p.votes[at];
        // (ln 1 = 0; and with t <= -40 alpha^n is below half an ulp of 1 and the term is 0)
        const double lp = pv_i == 1 ? 0.0 : log_f64((double)pv_i);
        const double term = t > -40.0 ? log_1m_exp_f64(t) : 0.0;
        x = (lp + x) - term;
        if (cnt <= 0) x = -INFINITY;
      }
      s_cand[tid] = x;
    }
    __syncthreads();
    if (tid < 4 * m) {                            // four lanes a slot
      const int at = tid >> 2;
      const double k = s_cand[at];
      const int i = s_cand_i[at];
      int rank = 0;                               // larger values, and equal ones at lower indices
      for (int j0 = tid & 3; j0 < m; j0 += 16) {  // four of the others a round trip
        double kj[4];
        int ij[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          kj[u] = s_cand[min(j0 + 4 * u, m - 1)];
          ij[u] = s_cand_i[min(j0 + 4 * u, m - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += (j0 + 4 * u < m) & ((kj[u] > k) | ((kj[u] == k) & (ij[u] < i)));
      }
      rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
      rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
      if ((tid & 3) == 0 && rank < need) atomicOr(&s_bits[i >> 6], 1ull << (i & 63));
    }
    __syncthreads();
  }
  KS_TS(10);

  // ---- ordered compaction: positions inside a chunk from a ballot, the wavefronts' totals through LDS ------
  auto kept_mask = [&](int c) -> uint64_t { return __ballot((keep >> c) & 1) | s_bits[wave * cpw + c]; };
  int nk = 0;
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c < cpw) nk += __popcll(kept_mask(c));    // uniform
  if (lane == 0) s_wave[wave] = nk;
  __syncthreads();
  KS_TS(11);
  int kpos = 0;                                   // kept slots at lower indices
#pragma unroll
  for (int w = 0; w < kWaves; ++w) kpos += w < wave ? s_wave[w] : 0;
  int32_t* keep_out = p.keep_idx + (size_t)unit * budget;
  int32_t* evict_out = p.evict_idx + (size_t)unit * (capacity - budget);
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    if (c < cpw) {                                // uniform
      const int i = first + 64 * c;
      const uint64_t mask = kept_mask(c);
      const int at = kpos + rank_in_wave(mask);
      if (i < n) {
        const int s = slot_of(i);
        if ((mask >> lane) & 1) keep_out[at] = s;
        else evict_out[i - at] = s;
      }
      kpos += __popcll(mask);
    }
  }
  if (tid == 0) p.n_evict[unit] = n - budget;
  KS_TS(12);
}

}  // namespace

constexpr int kSelRegSlots = 32 * kSelThreads;   // up to this capacity the values of a head are kept in registers

template <bool EXT, bool AGED = false>
void launch_select(int units, hipStream_t st, const float* log_s, const int32_t* born, const int32_t* t_obs,
                   const int32_t* votes, const int32_t* len, uint64_t* keys, int32_t* keep_idx, int32_t* evict_idx, int32_t* n_evict,
                   int capacity, int budget, int n_sink, int n_recent, double ln_alpha, const int32_t* order = nullptr) {
  // counts from which alpha^n is below half an ulp of 1 (n ln alpha <= -40) need no table entry
  int n_table = 0;
  if (!EXT && ln_alpha > -INFINITY && ln_alpha < 0.0) {
    const double n_zero = ceil(40.0 / -ln_alpha) + 1.0;
    n_table = n_zero < (double)kTermTable ? (int)n_zero : kTermTable;
  }
  const SelectParams p{log_s, born, t_obs, votes, len, keys, keep_idx, evict_idx, n_evict, capacity, budget, n_sink, n_recent,
                       ln_alpha, n_table, order};
  auto go = [&](void (*kernel)(SelectParams)) { kernel<<<units, kSelThreads, 0, st>>>(p); };
  const int cpw = (capacity + kSelThreads - 1) / kSelThreads;
  if (capacity > kSelRegSlots) go(select_long_kernel<EXT, AGED>);
  else if (cpw <= 1) go(select_kernel<EXT, AGED, 1>);
  else if (cpw <= 4) go(select_kernel<EXT, AGED, 4>);
  else if (cpw <= 8) go(select_kernel<EXT, AGED, 8>);
  else if (cpw <= 16) go(select_kernel<EXT, AGED, 16>);
  else go(select_kernel<EXT, AGED, 32>);
}

SelectPlan plan_select(const keepkv_layout* L, int capacity) {
  SelectPlan pl;
  pl.keys_off = kWorkspaceHead;
  pl.bytes = kWorkspaceHead + align_up((size_t)L->batch * L->n_kv_heads * capacity * sizeof(uint64_t), 256);
  return pl;
}

}  // namespace kk

extern "C" keepkv_status keepkv_select(const keepkv_layout* layout, const keepkv_cache* cache, int32_t budget,
                                       int32_t n_sink, int32_t n_recent, float alpha, int32_t* keep_idx,
                                       int32_t* evict_idx, int32_t* n_evict, void* workspace, size_t workspace_bytes,
                                       void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(cache) || !keep_idx || !n_evict) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (budget < 1 || budget > cache->capacity || n_sink < 0 || n_recent < 0 || n_sink + n_recent > budget)
    return KEEPKV_ERR_INVALID_ARG;
  if (budget < cache->capacity && !evict_idx) return KEEPKV_ERR_INVALID_ARG;
  if (!(alpha >= 0.f && alpha < 1.f)) return KEEPKV_ERR_INVALID_ARG;
  const SelectPlan pl = plan_select(layout, cache->capacity);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  const int units = layout->batch * layout->n_kv_heads;
  const double la = alpha > 0.f ? log((double)alpha) : -INFINITY;
  launch_select<false>(units, reinterpret_cast<hipStream_t>(stream),
      cache->log_s, cache->born, cache->t_obs, cache->votes, cache->len,
      reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(workspace) + pl.keys_off), keep_idx, evict_idx, n_evict,
      cache->capacity, budget, n_sink, n_recent, la);
  return launch_status();
}

extern "C" keepkv_status keepkv_select_aged(const keepkv_layout* layout, const keepkv_cache* cache,
                                            const int32_t* order, int32_t budget, int32_t n_sink, int32_t n_recent,
                                            float alpha, int32_t* keep_idx, int32_t* evict_idx, int32_t* n_evict,
                                            void* workspace, size_t workspace_bytes, void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(cache) || !order || !keep_idx || !n_evict) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (budget < 1 || budget > cache->capacity || n_sink < 0 || n_recent < 0 || n_sink + n_recent > budget)
    return KEEPKV_ERR_INVALID_ARG;
  if (budget < cache->capacity && !evict_idx) return KEEPKV_ERR_INVALID_ARG;
  if (!(alpha >= 0.f && alpha < 1.f)) return KEEPKV_ERR_INVALID_ARG;
  const SelectPlan pl = plan_select(layout, cache->capacity);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  const int units = layout->batch * layout->n_kv_heads;
  const double la = alpha > 0.f ? log((double)alpha) : -INFINITY;
  launch_select<false, true>(units, reinterpret_cast<hipStream_t>(stream),
      cache->log_s, cache->born, cache->t_obs, cache->votes, cache->len,
      reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(workspace) + pl.keys_off), keep_idx, evict_idx, n_evict,
      cache->capacity, budget, n_sink, n_recent, la, order);
  return launch_status();
}

extern "C" keepkv_status keepkv_select_by_key(const keepkv_layout* layout, const keepkv_cache* cache,
                                              const float* rank, int32_t budget, int32_t n_sink, int32_t n_recent,
                                              int32_t* keep_idx, int32_t* evict_idx, int32_t* n_evict,
                                              void* workspace, size_t workspace_bytes, void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache || !cache->len || !rank || !keep_idx || !n_evict) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (cache->capacity < 1 || cache->capacity > (1 << 20) || !aligned16(rank)) return KEEPKV_ERR_INVALID_ARG;
  if (budget < 1 || budget > cache->capacity || n_sink < 0 || n_recent < 0 || n_sink + n_recent > budget)
    return KEEPKV_ERR_INVALID_ARG;
  if (budget < cache->capacity && !evict_idx) return KEEPKV_ERR_INVALID_ARG;
  const SelectPlan pl = plan_select(layout, cache->capacity);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  const int units = layout->batch * layout->n_kv_heads;
  launch_select<true>(units, reinterpret_cast<hipStream_t>(stream),
      rank, nullptr, nullptr, nullptr, cache->len,
      reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(workspace) + pl.keys_off), keep_idx, evict_idx, n_evict,
      cache->capacity, budget, n_sink, n_recent, 0.0);
  return launch_status();
}

#ifdef KEEPKV_TRACE
extern "C" int keepkv_trace_read_select(long long* host, int n) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(kk::kk_trace_select), sizeof(long long) * n);
}
#endif
