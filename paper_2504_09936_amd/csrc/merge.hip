// keepkv_merge: multi-way Zero Inference-Perturbation Merging (Eq. 7 in the many-to-one form of
// App. A.3, with the EMA scores of App. A.4; Alg. 1, merging step) and compaction into the
// destination cache.
//
// Two kernels.  (1) Per head, the evicted slots are grouped by merge target into a CSR list: an LDS
// histogram of match[], a block scan for the row starts, and each group's members put in order by
// counting, so every group lists its members in ascending slot order (deterministic summation order,
// no float atomics).  With few evictable slots per head this kernel is not launched: the second one finds each
// group's members in the match list itself.  (2) One lane group (LPS lanes, 16 bytes of a row each) per retained
// position: the merge weights w_i = p_i s_hat_i are formed in f64 relative to the group's largest
// ln s_hat, one member per lane; the K and V rows of a position are then accumulated in f32 by the whole
// wavefront and scaled once at the end.  Positions without members are copied bit for bit.
#include "kk_common.hpp"

namespace kk {
#ifdef KEEPKV_TRACE
__device__ long long kk_trace_merge[8 * 1024];
#define KM_TS(i) do { if (threadIdx.x == 0 && blockIdx.x < 1024) kk_trace_merge[blockIdx.x * 8 + (i)] = wall_clock64(); } while (0)
#else
#define KM_TS(i) do { } while (0)
#endif
namespace {

constexpr int kGroupThreads = 1024;
constexpr int kMaxBudget = 4096;
constexpr int kMaxGroupShares = 32;       // workgroups that share one head's targets in the grouping kernel
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2_t;
constexpr int kRankMax = 256;             // longest group that is ordered by counting
constexpr int kMaxEvict = 32768;          // positions in the evict list fit 16 bits
constexpr double kEllGuard = 1.0e-3;

// Groups the evicted slots of one head by merge target into a CSR list whose members are in ascending order.
// A histogram of the targets and a block scan give every group its range; the entries (their positions in the
// evict list, 16 bits) are dropped into their group's range of an LDS array in arrival order; then every entry
// takes the place given by the number of smaller positions in its group.  That last step runs over the grouped
// array, so that neighbouring lanes belong to one group: their reads are broadcasts and their trip counts agree.
// A group longer than kRankMax would make that quadratic: one wavefront scans the head's match list in order
// for it instead.  With few heads up to kMaxGroupShares workgroups share a head, each taking a range of the
// targets: every one of them reads the whole match list, so none waits for another.
// What bounds it: the latency of one workgroup's steps (list, histogram, scan, places, ranks).
// Measured (MI355X): 8 heads x 29491 entries, clustered keys, all matched: 275 us with a sorting network of one workgroup
// per head, 103 with counting, 35 with eight workgroups per head, 20 with 32 (the ranks of lists of up to 230 members are most of the work) and
// the list read once; 1024 heads x 7372: 186 -> 90 us, 24 heads x about 3500 (D 64): 40 -> 12 -> 10 us.
// ITEMS: entries per thread that its registers hold from the histogram (the target and the place in the group that the add returned)
// until the group's range is known: the list is requested once, all of it before the first wait.
template <int ITEMS>
__global__ __launch_bounds__(kGroupThreads) void merge_group_kernel(
    const int32_t* __restrict__ match, const int32_t* __restrict__ evict_idx, const int32_t* __restrict__ n_evict,
    const int32_t* __restrict__ votes, int32_t* __restrict__ start, int32_t* __restrict__ members,
    int64_t* __restrict__ dropped_votes, int capacity, int budget, int max_evict, int shares) {
  extern __shared__ __align__(16) uint16_t s_place[];   // [max_evict] positions in the evict list, grouped by target
  __shared__ int s_cnt[kMaxBudget + 1];            // members per target; after the scan the group's first place
  __shared__ int s_wave[kGroupThreads / 64];
  __shared__ int s_long[kMaxEvict / kRankMax];     // targets of the long groups
  __shared__ long long s_drop;
  __shared__ int s_n_long, s_below;
  const int unit = blockIdx.x / shares, share = blockIdx.x % shares;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // this workgroup's targets: [t_lo, t_hi)
  const int t_lo = (int)((long)budget * share / shares), t_hi = (int)((long)budget * (share + 1) / shares);
  const int n_ev = n_evict[unit];
  const int32_t* mt = match + (size_t)unit * max_evict;
  const int32_t* ev = evict_idx + (size_t)unit * max_evict;
  int32_t* st = start + (size_t)unit * (budget + 1);
  int32_t* mem = members + (size_t)unit * capacity;

  KM_TS(0);
  for (int r = t_lo + tid; r < t_hi; r += kGroupThreads) s_cnt[r] = 0;
  if (tid == 0) {
    s_drop = 0;
    s_n_long = s_below = 0;
  }
  __syncthreads();
  // histogram of targets, and the number of entries whose targets lie below this workgroup's; unmatched slots (of
  // every shares-th batch here) give up their votes.
  constexpr int kBatch = 8;
  static_assert(ITEMS % kBatch == 0 && kMaxBudget <= 1 << 13 && kMaxEvict <= 1 << 16, "entries by batches; a target and a place in one word");
  long long drop = 0;
  int below = 0;
  int entry[ITEMS];                                // target; then target << 16 | place in the group, or -1
#pragma unroll
  for (int b = 0; b < ITEMS; b += kBatch)
    if (b * kGroupThreads < n_ev) {                // uniform over the workgroup
#pragma unroll
      for (int u = b; u < b + kBatch; ++u) entry[u] = mt[min(tid + u * kGroupThreads, n_ev - 1)];
    }
#pragma unroll
  for (int b = 0; b < ITEMS; b += kBatch)
    if (b * kGroupThreads < n_ev) {
      const bool votes_here = dropped_votes != nullptr && (b / kBatch) % shares == share;   // uniform over the workgroup
      int pv[kBatch];
      if (votes_here) {
        int e[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) e[u] = ev[min(tid + (b + u) * kGroupThreads, n_ev - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) pv[u] = votes[(size_t)unit * capacity + e[u]];
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int t = tid + (b + u) * kGroupThreads < n_ev ? entry[b + u] : kMaxBudget;
        entry[b + u] = -1;
        if (t >= t_lo && t < t_hi) entry[b + u] = t << 16 | atomicAdd(&s_cnt[t], 1);
        else if (t >= 0 && t < t_lo) ++below;
        else if (t < 0 && votes_here) drop += pv[u];
      }
    }
  // one LDS add per wavefront: adds to one word are served a lane at a time
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    drop += __shfl_xor(drop, off);
    below += __shfl_xor(below, off);
  }
  if (lane == 0) {
    if (drop != 0) atomicAdd((unsigned long long*)&s_drop, (unsigned long long)drop);
    if (below != 0) atomicAdd(&s_below, below);
  }
  __syncthreads();
  KM_TS(1);

  // exclusive scan of s_cnt[t_lo .. t_hi): thread t owns a contiguous run of positions.  Places in s_place count
  // from this workgroup's first member, places in the CSR list from the head's (s_below more).
  const int per = (t_hi - t_lo + kGroupThreads - 1) / kGroupThreads;
  const int r0 = min(t_hi, t_lo + tid * per), r1 = min(t_hi, r0 + per);
  int mine = 0;
  for (int r = r0; r < r1; ++r) {
    const int cnt = s_cnt[r];
    mine += cnt;
    if (cnt > kRankMax) s_long[atomicAdd(&s_n_long, 1)] = r;
  }
  int incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off);
    if (lane >= off) incl += u;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int before = 0, n_matched = 0;
#pragma unroll
  for (int w = 0; w < kGroupThreads / 64; ++w) {
    const int v = s_wave[w];
    if (w < wave) before += v;
    n_matched += v;
  }
  const int base = s_below;
  mem += base;
  int run = before + incl - mine;
  for (int r = r0; r < r1; ++r) {
    const int cnt = s_cnt[r];
    st[r] = base + run;
    s_cnt[r] = run;                                  // from here on: the group's first place
    run += cnt;
  }
  if (tid == 0 && t_hi == budget) st[budget] = base + n_matched;
  if (tid == 0) s_cnt[t_hi] = n_matched;             // (t_hi <= kMaxBudget)
  if (tid == 0 && s_drop != 0) atomicAdd((unsigned long long*)&dropped_votes[unit], (unsigned long long)s_drop);
  KM_TS(2);
  if (n_matched == 0) return;                       // uniform over the block
  __syncthreads();                                  // starts complete

#pragma unroll
  for (int b = 0; b < ITEMS; b += kBatch)
    if (b * kGroupThreads < n_ev) {
#pragma unroll
      for (int u = b; u < b + kBatch; ++u)
        if (entry[u] >= 0) s_place[s_cnt[entry[u] >> 16] + (entry[u] & 0xFFFF)] = (uint16_t)(tid + u * kGroupThreads);
    }
  __syncthreads();
  KM_TS(3);

  for (int i0 = tid; i0 < n_matched; i0 += kBatch * kGroupThreads) {
    int j[kBatch], t[kBatch], slot[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) j[u] = s_place[min(i0 + u * kGroupThreads, n_matched - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      t[u] = mt[j[u]];
      slot[u] = ev[j[u]];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int g0 = s_cnt[t[u]], g1 = s_cnt[t[u] + 1];
      if (i0 + u * kGroupThreads >= n_matched || g1 - g0 > kRankMax) continue;
      // eight members per LDS read, two per instruction: min(max(j - o, 0), 1) counts the smaller ones.  The first
      // and the last eight may hold neighbours' members, which are replaced by the largest value.
      u16x2_t rank2 = {0, 0};
      const u16x2_t one = {1, 1}, jj = {(uint16_t)j[u], (uint16_t)j[u]};
      for (int m = g0 & ~7; m < g1; m += 8) {
        const uint4 x = *reinterpret_cast<const uint4*>(s_place + m);
        uint32_t o[4] = {x.x, x.y, x.z, x.w};
        if (m < g0 || m + 8 > g1) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (m + 2 * q < g0 || m + 2 * q >= g1) o[q] |= 0xFFFFu;
            if (m + 2 * q + 1 < g0 || m + 2 * q + 1 >= g1) o[q] |= 0xFFFF0000u;
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          rank2 += __builtin_elementwise_min(__builtin_elementwise_sub_sat(jj, __builtin_bit_cast(u16x2_t, o[q])), one);
      }
      mem[g0 + rank2[0] + rank2[1]] = slot[u];
    }
  }
  const int n_long = s_n_long;
  for (int l = wave; l < n_long; l += kGroupThreads / 64) {   // uniform over the wavefront
    const int r = s_long[l];
    int at = s_cnt[r];
    for (int j0 = 0; j0 < n_ev; j0 += kBatch * 64) {
      int t[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) t[u] = mt[min(j0 + u * 64 + lane, n_ev - 1)];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u * 64 + lane;
        const bool hit = j < n_ev && t[u] == r;
        const unsigned long long m = __ballot(hit);
        if (hit) mem[at + __popcll(m & ((1ull << lane) - 1ull))] = ev[j];
        at += __popcll(m);
      }
    }
  }
  KM_TS(4);
}

struct MergeParams {
  const void *sk, *sv;
  const int32_t* svotes;
  const float* slog_s;
  const int32_t* sborn;        // a slot's observation count is t_obs - born
  const int32_t* st_obs;       // [units]
  const int32_t* slen;
  void *dk, *dv;
  int32_t* dvotes;
  float* dlog_s;
  int32_t* dborn;
  int32_t* dt_obs;             // receives st_obs
  int32_t* dlen;
  const int32_t* keep_idx;
  const int32_t* n_evict;
  const int32_t* start;
  const int32_t* members;
  const int32_t* match;        // the direct variant reads the match and evict lists itself
  const int32_t* evict_idx;
  int64_t* dropped_votes;
  int scap, dcap, budget, max_evict;
  int positions_per_wave;      // merge_apply_kernel without DIRECT
  int write_len;               // 0: the caller's grouping kernel has set dst.len (prefill pass)
  double ln_alpha;
};

constexpr int kDirectMaxEvict = 256;   // up to this many evictable slots per head no CSR list is built

// The f64 library routines as calls: inlined, their polynomial coefficients kept some forty registers busy all
// through the kernels, and with 135 registers instead of 95 the apply kernel took 1450 us instead of 1024 on the batch-128
// first event.
__device__ __attribute__((noinline)) double log_f64(double x) { return log(x); }
__device__ __attribute__((noinline)) double exp_f64(double x) { return exp(x); }
__device__ __attribute__((noinline)) double log_1m_exp_f64(double t) { return log(-expm1(t)); }

// ln(1 - alpha^n), the bias correction of Eq. 8.  It depends on the count alone and exactly 0 is left of it once
// n ln alpha <= -40 (alpha^n is then below half an ulp of 1); the f64 library routines behind it are hundreds of
// instructions.  So a wavefront evaluates it only where one of its lanes needs a value that is neither 0 nor the
// lane's last one (after a prefill all slots of a head have the same count).
struct CountTerm {
  int n = 0;
  double value = 0.0;
  __device__ __forceinline__ double of(int m, double ln_alpha) {
    const double t = (double)m * ln_alpha;         // (-inf with alpha == 0)
    const bool zero = m <= 0 || !(t > -40.0);
    if (__any(!zero && m != n)) {
      value = zero ? 0.0 : log_1m_exp_f64(t);
      n = m;
    }
    return zero ? 0.0 : value;
  }
};

// ln s_hat_i = ln S_i - ln(1 - alpha^n_i); -inf when never observed
__device__ __forceinline__ double log_s_hat(float log_s, int n, double ln_alpha, CountTerm& term) {
  const double t = term.of(n, ln_alpha);
  return n <= 0 ? -INFINITY : (double)log_s - t;
}

// Over aligned groups of LANES lanes, every lane receives the result; the pairs are those of an exchange with lane ^ 1, ^ 2, ^ 4, ...
// By register moves between lanes: an exchange through LDS takes a hundred cycles, and a position has 16 to 24 in a row.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int LANES, typename F>
__device__ __forceinline__ double group_reduce_f64(double x, F f) {
  x = f(x, dpp_f64<0xB1>(x));                             // quad_perm [1,0,3,2]
  x = f(x, dpp_f64<0x4E>(x));                             // quad_perm [2,3,0,1]
  if constexpr (LANES >= 8) x = f(x, dpp_f64<0x141>(x));  // row_half_mirror
  if constexpr (LANES >= 16) x = f(x, dpp_f64<0x140>(x)); // row_mirror
  auto pair = [&](auto swap) {                            // the two rows, then halves, that an exchange brings together
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const auto lo = swap((uint32_t)b), hi = swap((uint32_t)(b >> 32));
    const uint32_t lo0 = lo[0], lo1 = lo[1], hi0 = hi[0], hi1 = hi[1];
    x = f(__builtin_bit_cast(double, (uint64_t)hi0 << 32 | lo0), __builtin_bit_cast(double, (uint64_t)hi1 << 32 | lo1));
  };
  if constexpr (LANES >= 32) pair([](uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
  if constexpr (LANES >= 64) pair([](uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
  return x;
}
template <int LANES>
__device__ __forceinline__ double group_max_f64(double x) {
  return group_reduce_f64<LANES>(x, [](double a, double b) { return fmax(a, b); });
}
template <int LANES>
__device__ __forceinline__ double group_sum_f64(double x) {
  return group_reduce_f64<LANES>(x, [](double a, double b) { return a + b; });
}

// Each lane group of a wavefront (LPS lanes, 64 / LPS groups) brings one retained slot c, the nm evicted slots
// list[off .. off + nm) that it absorbs (nm = 0: nothing to do for this group) and the destination slot: the multi-way
// merge of App. A.3 / A.4 over the entries (c, list[off], ..., list[off + nm - 1]) with weights p * s_hat formed in
// f64 relative to the largest ln s_hat, rows accumulated in f32 and scaled once.  Called by whole wavefronts.
// The scalars of positions with up to LPS entries (most of them) are worked out side by side, one entry per lane, so
// that the f64 routines run once for all groups; a longer list has its scalars spread over the whole wavefront.
// Up to kOwnRows entries a lane group sums the rows of its position itself, in list order, so that one or two round trips
// serve all positions of the wavefront.  Longer lists are summed one position after the other by the whole wavefront, entry e by
// lane group e mod (64 / LPS), and the groups' partial sums meet in a fixed tree.  Either way a position's bits depend on its list
// alone and not on the kernel or on its place in the wavefront.
// Why: the members per target vary widely (mean 9, largest 147 on the clustered keys of the long-context
// workload).  With one lane group per position a wavefront took as long as its largest group, one dependent round
// trip for every LPS scalars and every few rows.
// What bounds it: HBM for the members' rows, and the f64 arithmetic.  Measured against one lane group per position
// (MI355X): 1024 heads x 820 positions, 7372 evicted rows each, 4.6 GB moved: 1637 -> 1020 us (4.5 TB/s; a plain copy
// reaches 5.1); 8 heads x 3277, 29491 rows: 163 -> 65 us; 24 heads x 501 of D 64: 64 -> 25 us; the in-place event of 128
// heads: 14.6 -> 13.7 us.  Merge-first prefill where every second slot is absorbed by its neighbour (lists of two; D 64, whole
// call): 56 heads x 4386 slots 58 us with one lane group per position, 82 with whole wavefronts for all lists, 49 now; 88 x 978
// 31.7, 45.5, 27.5.
template <typename T, int D>
__device__ __forceinline__ void merge_positions(const MergeParams& p, int unit, int t_head, int c, const int32_t* list,
                                                int off, int nm, int dst) {
  constexpr int EPL = 16 / (int)sizeof(T), LPS = D / EPL, GPW = 64 / LPS;
  // entries per lane group and round trip.  With 2 / 3 / 4 (81 / 91 / 101 registers), the whole first event: 1024 heads 3236 / 3200 / 3286
  // us, 8 heads with lists of up to 230 entries 350.5 / 344.9 / 341.1, 24 heads of D 64 74.3 / 73.7 / 74.5.  Lists all of one length (1 to 40
  // entries, 4 to 128 heads), 2 / 3: bf16 1 to 12 % faster with 3 and nowhere more than 2 % slower; f32 up to 14 % faster (8 heads x 100 lists of 40, D 128,
  // 22.3 / 19.3), 5 % slower at worst (64 heads x 820 lists of 12, D 64, 103 / 108).
  constexpr int kRowBatch = 3;
  constexpr int kOwnRows = LPS == 8 ? 8 : 4;                       // up to this many entries a lane group sums its position by itself
  const size_t sbase = (size_t)unit * p.scap, dbase = (size_t)unit * p.dcap;
  const uint4* sk = reinterpret_cast<const uint4*>(p.sk) + sbase * LPS;
  const uint4* sv = reinterpret_cast<const uint4*>(p.sv) + sbase * LPS;
  const int lane = threadIdx.x & 63, sub = lane % LPS, grp = lane / LPS;
  const int ne = nm > 0 ? nm + 1 : 0;               // entries of this group's position

  struct Entry {
    int s, pv, n;
    double E;
  };
  CountTerm term;
  auto entry = [&](int slot_c, int first, int i, int n_entries) {   // scalars of entry i (beyond the list: slot c, no weight)
    Entry x{slot_c, 0, 0, -INFINITY};
    float ls = 0.f;
    if (i < n_entries) {
      if (i > 0) x.s = list[first + i - 1];
      x.pv = p.svotes[sbase + x.s];
      ls = p.slog_s[sbase + x.s];
      x.n = t_head - p.sborn[sbase + x.s];
    }
    x.E = log_s_hat(ls, x.n, p.ln_alpha, term);
    return x;
  };
  auto weight = [](const Entry& x, double mx) {
    if (!(mx > -INFINITY)) return (double)x.pv;     // nothing observed: vote weights
    return x.E > -INFINITY ? (double)x.pv * exp_f64(x.E - mx) : 0.0;
  };
  auto weighted_e = [](double w, const Entry& x, double mx) { return (w > 0.0 && mx > -INFINITY) ? w * x.E : 0.0; };
  // the merged slot's scalars and the factors of its rows, from the sums over its entries
  struct Scales {
    float fk, fv, log_s;
    int votes, n_r;
  };
  auto scales = [&](double mx, double P, double W, double WE, int n_c) {
    Scales o;
    o.votes = (int)(long long)P;
    o.log_s = -INFINITY;
    o.n_r = 0;
    double kscale = 1.0 / W;                        // nothing observed: W = P, the vote-weighted mean stays unobserved
    o.fv = (float)kscale;
    if (mx > -INFINITY) {
      const double L = mx + log_f64(W / P);             // ln(sum p s_hat / sum p)
      // ell = WE / W = sum w ln s_hat / W: (L / ell) / W is L / WE (a division in f64 is some twenty instructions)
      if (!(fabs(WE) < kEllGuard * W)) kscale = L / WE;
      o.n_r = n_c > 1 ? n_c : 1;
      o.log_s = (float)(L + term.of(o.n_r, p.ln_alpha));
    }
    o.fk = (float)kscale;
    return o;
  };
  auto fma_row = [](const uint4& x, float w, float* a) {
    const uint32_t u[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (sizeof(T) == 2) {
        a[2 * q] = fmaf(w, bf16_lo(u[q]), a[2 * q]);
        a[2 * q + 1] = fmaf(w, bf16_hi(u[q]), a[2 * q + 1]);
      } else {
        a[q] = fmaf(w, __builtin_bit_cast(float, u[q]), a[q]);
      }
    }
  };
  float acc[2 * EPL];                               // this lane's channels of the K sum, then of the V sum
  // adds the rows of entries 0 .. cnt - 1 whose slots and weights lanes first, first + 1, ... hold
  auto add_rows = [&](int s, float wf, int first, int cnt) {
    for (int q0 = 0; q0 < cnt; q0 += kRowBatch * GPW) {
      uint4 kr[kRowBatch], vr[kRowBatch];
      float wq[kRowBatch];
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u) {
        const int at = first + min(q0 + u * GPW + grp, cnt - 1);     // (surplus: the last entry again, not added)
        const uint32_t row = (uint32_t)__shfl(s, at) * LPS + sub;
        wq[u] = __shfl(wf, at);
        kr[u] = sk[row];
        vr[u] = sv[row];
      }
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u)
        if (q0 + u * GPW + grp < cnt) {
          fma_row(kr[u], wq[u], acc);
          fma_row(vr[u], wq[u], acc + EPL);
        }
    }
  };

  auto store_scalars = [&](int to, const Scales& sc) {
    p.dvotes[dbase + to] = sc.votes;
    p.dlog_s[dbase + to] = sc.log_s;
    p.dborn[dbase + to] = t_head - sc.n_r;
  };
  auto clear = [&]() {
#pragma unroll
    for (int e = 0; e < 2 * EPL; ++e) acc[e] = 0.f;
  };
  auto sum2 = [](uint32_t a, uint32_t b) { return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b); };
  auto store_rows = [&](int g, float fk, float fv) {            // the sums of group g's position, scaled
    // The lane groups' sums meet, and are dealt out on the way: an exchange of half-wavefronts between value e and
    // value e + half of the list adds both pairs with one addition and leaves half as many values in each lane.
    // Lanes 0 - 31 end up with K, lanes 32 - 63 with V.
    if constexpr (LPS == 8) {
#pragma unroll
      for (int e = 0; e < 2 * EPL; ++e) acc[e] += dpp_f32<0x128>(acc[e]);     // row_ror:8: the other group of this row
    }
    constexpr int kLeft = LPS >= 32 ? EPL : EPL / 2;            // values per lane at the end
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, acc[e]),
                                                      __builtin_bit_cast(uint32_t, acc[e + EPL]), false, false);
      acc[e] = sum2(r[0], r[1]);
    }
    if constexpr (LPS < 32) {
#pragma unroll
      for (int e = 0; e < EPL / 2; ++e) {
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, acc[e]),
                                                        __builtin_bit_cast(uint32_t, acc[e + EPL / 2]), false, false);
        acc[e] = sum2(r[0], r[1]);
      }
    }
    const float f = lane < 32 ? fk : fv;
    const size_t row = (dbase + __builtin_amdgcn_readlane(dst, g * LPS)) * D;
    const int ch = sub * EPL + (LPS < 32 ? ((lane >> 4) & 1) * kLeft : 0);   // this lane's first channel
    T* out = reinterpret_cast<T*>(lane < 32 ? p.dk : p.dv) + row + ch;
    if (LPS > 8 || (lane & 8) == 0) {
      if constexpr (sizeof(T) == 2) {
        static_assert(sizeof(T) != 2 || kLeft == 4, "one 8-byte store");
        *reinterpret_cast<uint2*>(out) = make_uint2(pack_bf16x2(acc[0] * f, acc[1] * f), pack_bf16x2(acc[2] * f, acc[3] * f));
      } else {
#pragma unroll
        for (int e = 0; e < kLeft; ++e) out[e] = acc[e] * f;
      }
    }
  };

  // ---- short lists: scalars side by side, then the rows position by position
  if (__any(ne > 0 && ne <= LPS)) {
    const Entry x = entry(c, off, sub, ne <= LPS ? ne : 0);
    const double mx = group_max_f64<LPS>(x.E);
    const double w = weight(x, mx);
    const float wf = (float)w;
    const Scales sc = scales(mx, group_sum_f64<LPS>((double)x.pv), group_sum_f64<LPS>(w),
                             group_sum_f64<LPS>(weighted_e(w, x, mx)), __shfl(x.n, grp * LPS));
    if (ne > 0 && ne <= LPS && sub == 0) store_scalars(dst, sc);
    const int own = ne <= kOwnRows ? ne : 0;
    if (__any(own > 0)) {                          // the shortest: every lane group sums its own position, in list order
      clear();
#pragma unroll
      for (int q0 = 0; q0 < kOwnRows; q0 += 4) {   // four rows a round trip
        if (q0 > 0 && !__any(own > q0)) break;
        uint4 kr[4], vr[4];
        float wq[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t row = (uint32_t)__shfl(x.s, grp * LPS + q0 + u) * LPS + sub;
          wq[u] = __shfl(wf, grp * LPS + q0 + u);
          if (q0 + u < own) {
            kr[u] = sk[row];
            vr[u] = sv[row];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (q0 + u < own) {
            fma_row(kr[u], wq[u], acc);
            fma_row(vr[u], wq[u], acc + EPL);
          }
      }
      if (own > 0) {
        auto row_of = [](const float* a, float f) {
          if constexpr (sizeof(T) == 2)
            return make_uint4(pack_bf16x2(a[0] * f, a[1] * f), pack_bf16x2(a[2] * f, a[3] * f),
                              pack_bf16x2(a[4] * f, a[5] * f), pack_bf16x2(a[6] * f, a[7] * f));
          else
            return make_uint4(__builtin_bit_cast(uint32_t, a[0] * f), __builtin_bit_cast(uint32_t, a[1] * f),
                              __builtin_bit_cast(uint32_t, a[2] * f), __builtin_bit_cast(uint32_t, a[3] * f));
        };
        reinterpret_cast<uint4*>(p.dk)[(dbase + dst) * LPS + sub] = row_of(acc, sc.fk);
        reinterpret_cast<uint4*>(p.dv)[(dbase + dst) * LPS + sub] = row_of(acc + EPL, sc.fv);
      }
    }
#pragma unroll 1
    for (int g = 0; g < GPW; ++g) {
      const int n = __builtin_amdgcn_readlane(ne, g * LPS);     // uniform: entries of group g's position
      if (n <= kOwnRows || n > LPS) continue;
      clear();
      add_rows(x.s, wf, g * LPS, n);
      store_rows(g, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sc.fk), g * LPS)),
                 __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sc.fv), g * LPS)));
    }
  }
  // ---- long lists, one after the other
  if (!__any(ne > LPS)) return;
#pragma unroll 1
  for (int g = 0; g < GPW; ++g) {
    const int n = __builtin_amdgcn_readlane(ne, g * LPS);
    if (n <= LPS) continue;
    const int c_g = __builtin_amdgcn_readlane(c, g * LPS), off_g = __builtin_amdgcn_readlane(off, g * LPS);
    Entry x = entry(c_g, off_g, lane, n);
    const int n_c = __builtin_amdgcn_readfirstlane(x.n);
    double mx = group_max_f64<64>(x.E), P = group_sum_f64<64>((double)x.pv);
    for (int i0 = 64; i0 < n; i0 += 64) {
      const Entry y = entry(c_g, off_g, i0 + lane, n);
      mx = fmax(mx, group_max_f64<64>(y.E));
      P += group_sum_f64<64>((double)y.pv);
    }
    double W = 0.0, WE = 0.0;
    clear();
    for (int i0 = 0; i0 < n; i0 += 64) {
      if (i0 > 0) x = entry(c_g, off_g, i0 + lane, n);
      const double w = weight(x, mx);
      W += group_sum_f64<64>(w);
      WE += group_sum_f64<64>(weighted_e(w, x, mx));
      add_rows(x.s, (float)w, 0, min(64, n - i0));
    }
    const Scales sc = scales(mx, P, W, WE, n_c);
    if (lane == 0) store_scalars(__builtin_amdgcn_readlane(dst, g * LPS), sc);
    store_rows(g, sc.fk, sc.fv);
  }
}

// DIRECT (few evictable slots per head, the steady state): no CSR list has been built; the workgroup reads
// the head's match and evict lists into LDS and every lane group picks its own members out of them, in list
// (= ascending slot) order, so the summation order is the CSR variant's.  The first workgroup of a head
// also adds the votes of the unmatched evicted slots to the head's dropped count.
template <typename T, int D, bool DIRECT>
__global__ __launch_bounds__(256) void merge_apply_kernel(MergeParams p) {
  constexpr int EPL = 16 / (int)sizeof(T), LPS = D / EPL, GPB = 256 / LPS;
  __shared__ int s_match[DIRECT ? kDirectMaxEvict : 1], s_evict[DIRECT ? kDirectMaxEvict : 1];
  __shared__ int s_mem[DIRECT ? GPB : 1][DIRECT ? kDirectMaxEvict : 1];
  __shared__ long long s_drop;
  const int unit = blockIdx.y;
  const int sub = threadIdx.x % LPS;
  const int lane = threadIdx.x & 63;
  const int gbase = lane - sub;                 // first lane of this group within the wavefront
  // positions per wavefront: one for each lane group, or fewer (the other groups then only help with the rows)
  const int ppw = DIRECT ? 64 / LPS : p.positions_per_wave;
  const int r = lane / LPS < ppw ? ((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)) * ppw + lane / LPS : p.budget;
  const int t_head = p.st_obs[unit];            // the head's step counter: unchanged by a merge
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    p.dt_obs[unit] = t_head;
    if (p.write_len) {
      const int n = p.slen[unit];
      p.dlen[unit] = n < p.budget ? n : p.budget;
    }
  }
  const size_t sbase = (size_t)unit * p.scap, dbase = (size_t)unit * p.dcap;
  const uint4* sk = reinterpret_cast<const uint4*>(p.sk);
  const uint4* sv = reinterpret_cast<const uint4*>(p.sv);
  // The slot number of this position is requested first, and with DIRECT the retained row and its scalars are
  // requested before the head's lists are waited for: requests complete in the order of issue, so the
  // lists' round trip and the row's overlap instead of following each other.
  const int c = r < p.budget ? p.keep_idx[(size_t)unit * p.budget + r] : -1;   // (-1: nothing to write)
  int n_ev = 0;
  uint4 kc = make_uint4(0, 0, 0, 0), vc = make_uint4(0, 0, 0, 0);
  int p_c = 0, n_c = 0;
  float ls_c = 0.f;
  auto request_row = [&]() {
    const size_t at = sbase + max(c, 0);           // (a negative slot number: slot 0 stands in, unused)
    kc = sk[at * LPS + sub];
    vc = sv[at * LPS + sub];
    p_c = p.svotes[at];
    ls_c = p.slog_s[at];
    n_c = t_head - p.sborn[at];
  };
  if constexpr (DIRECT) {
    n_ev = min(p.n_evict[unit], kDirectMaxEvict);
    if (threadIdx.x == 0) s_drop = 0;
    int mt[kDirectMaxEvict / 256], ev[kDirectMaxEvict / 256];
    static_assert(kDirectMaxEvict == 256, "one list entry per thread");
    mt[0] = ev[0] = 0;
    if (n_ev > 0) {                                // uniform over the workgroup (the lists may be absent otherwise)
      const int li = min((int)threadIdx.x, n_ev - 1);
      mt[0] = p.match[(size_t)unit * p.max_evict + li];
      ev[0] = p.evict_idx[(size_t)unit * p.max_evict + li];
    }
    request_row();
    if ((int)threadIdx.x < n_ev) {
      s_match[threadIdx.x] = mt[0];
      s_evict[threadIdx.x] = ev[0];
    }
    __syncthreads();
    if (blockIdx.x == 0 && p.dropped_votes != nullptr) {       // uniform over the workgroup
      long long drop = 0;
      for (int i = threadIdx.x; i < n_ev; i += 256)
        if (s_match[i] < 0) drop += p.svotes[sbase + s_evict[i]];
      if (drop != 0) atomicAdd((unsigned long long*)&s_drop, (unsigned long long)drop);
      __syncthreads();
      if (threadIdx.x == 0 && s_drop != 0) p.dropped_votes[unit] += s_drop;   // no other workgroup touches it
    }
  }
  // (without DIRECT: two dependent round trips per row, (slot number, member range), then (rows, scalars))
  int m0 = 0, m1 = 0;
  if constexpr (!DIRECT) {
    if (r < p.budget) {
      m0 = p.start[(size_t)unit * (p.budget + 1) + r];
      m1 = p.start[(size_t)unit * (p.budget + 1) + r + 1];
    }
  } else {
    // this group's members: positions of the evict list whose target is r, LPS candidates at a time
    int* mine = s_mem[threadIdx.x / LPS];
    for (int i0 = 0; i0 < n_ev; i0 += LPS) {
      const bool hit = i0 + sub < n_ev && s_match[i0 + sub] == r;
      const unsigned long long wave_hits = __ballot(hit);
      const unsigned int hits = (unsigned int)(wave_hits >> gbase) & (unsigned int)((1ull << LPS) - 1ull);   // LPS <= 32
      if (hit) mine[m1 + __popc(hits & ((1u << sub) - 1u))] = s_evict[i0 + sub];
      m1 += __popc(hits);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the list is read back by this group's own lanes
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  uint4* dk = reinterpret_cast<uint4*>(p.dk);
  uint4* dv = reinterpret_cast<uint4*>(p.dv);
  const int nm = c >= 0 ? m1 - m0 : 0;           // evicted members of this group
  const size_t at = dbase + r;
  if (c >= 0 && nm == 0) {                       // nothing merged here: copy
    if constexpr (!DIRECT) request_row();
    dk[at * LPS + sub] = kc;
    dv[at * LPS + sub] = vc;
    if (sub == 0) {
      p.dvotes[at] = p_c;
      p.dlog_s[at] = ls_c;
      p.dborn[at] = t_head - n_c;
    }
  }
  if (!__any(nm > 0)) return;                    // uniform over the wavefront
  const int32_t* list = DIRECT ? &s_mem[0][0] : p.members + sbase;
  merge_positions<T, D>(p, unit, t_head, max(c, 0), list, DIRECT ? (int)(threadIdx.x / LPS) * kDirectMaxEvict : m0, nm, r);
}

// ---------------------------------------------------------------------------------------------------
// Merge-first prefill pass (App. B.4), grouping.  near[i] is slot i's most similar earlier key above the
// threshold, or -1: the links form a forest.  A slot is absorbed by the slot it links to unless that slot is
// itself absorbed, i.e. slots at odd depth of their tree are absorbed by their parent and slots at even depth
// stay and receive their children.  Depth parity comes from pointer jumping in LDS (links point to lower
// slot numbers; at most ceil(log2 len) rounds, ended when no slot moves any more: two or three where few slots link);
// the receiving slots are numbered in ascending order by a block scan,
// the absorbed slots grouped by receiver (histogram, scan, scatter) and put in ascending slot order inside
// each group by counting, so the merge sums in a fixed order.  Output in the form merge_apply_kernel reads:
// keep_idx (receivers, -1 behind them), CSR starts and members, all with pitch `capacity`; dst.len = receivers.
// The two per-slot work arrays live in LDS up to kPrefillLdsSlots slots per head; beyond that (GLOBAL) they are
// in the workspace and are read and written with device-scope accesses: the same steps, an L2 round trip each.
// What bounds it: LDS accesses of one workgroup per head.  Neighbouring lanes hold neighbouring slots: with a run of 8 slots
// per thread every access hit the banks eight times over, and with all 13 rounds 64 heads x 8192 slots took 58 us (now
// 20 us).  Whether a slot moved is a word of LDS per round (a barrier that also joins a flag over the workgroup cost a quarter more
// where long chains take all rounds).
constexpr int kPrefillLdsSlots = 16384;          // two int arrays of that many words fit in LDS
constexpr int kPrefillMaxSlots = 32768;
constexpr int kPfRounds = 15;                    // ceil(log2 kPrefillMaxSlots)

template <int kPfItems, bool GLOBAL>
__global__ __launch_bounds__(kGroupThreads) void prefill_group_kernel(
    const int32_t* __restrict__ near, const int32_t* __restrict__ slen, int32_t* __restrict__ keep_idx,
    int32_t* __restrict__ start, int32_t* __restrict__ members, int32_t* __restrict__ dlen, int capacity,
    int32_t* __restrict__ gwork) {
  extern __shared__ int s_pf[];                   // [2][n_pad] (unused when GLOBAL)
  __shared__ int s_wave[kGroupThreads / 64];
  __shared__ int s_moved[kPfRounds];              // by round: some slot moved
  // (device-scope stores of this workgroup are awaited before a barrier that publishes them to its other threads)
  auto sync = [] {
    if constexpr (GLOBAL) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  auto ld = [](const int* q, int i) -> int {
    if constexpr (GLOBAL) return __hip_atomic_load(q + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return q[i];
  };
  auto st_ = [](int* q, int i, int v) {
    if constexpr (GLOBAL) __hip_atomic_store(q + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else q[i] = v;
  };
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = min(slen[unit], capacity);
  const int per = (capacity + kGroupThreads - 1) / kGroupThreads;     // slots per thread (<= kPfItems)
  const int i0 = wave * per * 64 + lane;           // its u-th slot is i0 + 64 u: a wavefront takes a run of 64-slot chunks
  const int32_t* nr = near + (size_t)unit * capacity;
  int* A = GLOBAL ? gwork + (size_t)unit * 2 * per * kGroupThreads : s_pf;
  int* B = A + per * kGroupThreads;

  // (ancestor << 1) | parity of the distance to it; a slot without a link is its own ancestor
  int link[kPfItems];
#pragma unroll
  for (int u = 0; u < kPfItems; ++u) {
    const int i = i0 + 64 * u;
    link[u] = -1;
    if (u < per && i < n) {
      const int l = nr[i];
      link[u] = (l >= 0 && l < i) ? l : -1;       // (a link that does not point to an earlier slot is ignored)
      st_(A, i, link[u] >= 0 ? ((link[u] << 1) | 1) : (i << 1));
    }
  }
  if (tid < kPfRounds) s_moved[tid] = 0;
  sync();
  int rounds = 0;
  while ((1 << rounds) < n) ++rounds;
  int* cur = A;
  int* nxt = B;
  for (int r = 0; r < rounds; ++r) {              // uniform trip count
    int moved = 0;
#pragma unroll
    for (int u = 0; u < kPfItems; ++u) {
      const int i = i0 + 64 * u;
      if (u < per && i < n) {
        const int x = ld(cur, i);
        const int y = ld(cur, x >> 1);
        st_(nxt, i, (y & ~1) | ((x ^ y) & 1));
        moved |= (x ^ y) & ~1;
      }
    }
    if (__any(moved != 0) && lane == 0) s_moved[r] = 1;
    sync();
    int* t = cur; cur = nxt; nxt = t;
    if (s_moved[r] == 0) break;                   // uniform: every slot has its root
  }
  // absorbed = odd depth; receivers numbered in slot order: positions in a chunk by ballot
  bool absorbed[kPfItems];
  int recv_wave = 0;
#pragma unroll
  for (int u = 0; u < kPfItems; ++u) {
    const int i = i0 + 64 * u;
    absorbed[u] = (u < per && i < n) ? (ld(cur, i) & 1) != 0 : false;
    recv_wave += __popcll(__ballot(u < per && i < n && !absorbed[u]));
  }
  auto block_exclusive = [&](int mine, int& total) {   // exclusive prefix of `mine` over the threads, and the sum
    int incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    __syncthreads();                              // previous use of s_wave is over
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < kGroupThreads / 64; ++w) {
      const int v = s_wave[w];
      if (w < wave) before += v;
      all += v;
    }
    total = all;
    return before + incl - mine;
  };
  if (lane == 0) s_wave[wave] = recv_wave;
  __syncthreads();
  int n_recv = 0, rbase = 0;
  for (int w = 0; w < kGroupThreads / 64; ++w) {
    if (w < wave) rbase += s_wave[w];
    n_recv += s_wave[w];
  }
  // nxt: receiver number of every receiving slot; then cur is free
#pragma unroll
  for (int u = 0; u < kPfItems; ++u) {
    const int i = i0 + 64 * u;
    const bool receives = u < per && i < n && !absorbed[u];
    const uint64_t mask = __ballot(receives);
    if (receives) {
      const int rpos = rbase + __popcll(mask & ((1ull << lane) - 1));
      st_(nxt, i, rpos);
      keep_idx[(size_t)unit * capacity + rpos] = i;
    }
    rbase += __popcll(mask);
  }
  for (int r = n_recv + tid; r < capacity; r += kGroupThreads) keep_idx[(size_t)unit * capacity + r] = -1;
  sync();
  int* cnt = cur;                                 // histogram over receiver numbers, then cursors
  for (int r = tid; r < n_recv; r += kGroupThreads) st_(cnt, r, 0);
  int pos[kPfItems];                              // receiver number of this thread's absorbed slots
#pragma unroll
  for (int u = 0; u < kPfItems; ++u) pos[u] = absorbed[u] ? ld(nxt, link[u]) : -1;
  sync();
#pragma unroll
  for (int u = 0; u < kPfItems; ++u)
    if (absorbed[u]) atomicAdd(&cnt[pos[u]], 1);
  sync();
  // exclusive scan of cnt[0 .. n_recv): thread t owns a contiguous run of receiver numbers
  const int rper = (n_recv + kGroupThreads - 1) / kGroupThreads;
  const int q0 = min(n_recv, tid * rper), q1 = min(n_recv, q0 + rper);
  int mine = 0;
  for (int r = q0; r < q1; ++r) mine += ld(cnt, r);
  int n_abs = 0;
  int run = block_exclusive(mine, n_abs);
  int32_t* st = start + (size_t)unit * (capacity + 1);
  for (int r = q0; r < q1; ++r) {
    const int c = ld(cnt, r);
    st[r] = run;
    st_(cnt, r, run);                             // where the group's next member goes
    run += c;
  }
  for (int r = n_recv + tid; r <= capacity; r += kGroupThreads) st[r] = n_abs;
  if (tid == 0) dlen[unit] = n_recv;
  sync();
  int* tmp = nxt;                                 // the receiver numbers are in registers now: members in arrival order
#pragma unroll
  for (int u = 0; u < kPfItems; ++u)
    if (absorbed[u]) st_(tmp, atomicAdd(&cnt[pos[u]], 1), i0 + 64 * u);
  sync();                                // cnt[r] is now the end of group r
  int32_t* mem = members + (size_t)unit * capacity;
#pragma unroll
  for (int u = 0; u < kPfItems; ++u) {
    if (!absorbed[u]) continue;
    const int g0 = pos[u] > 0 ? ld(cnt, pos[u] - 1) : 0, g1 = ld(cnt, pos[u]);
    int rank = 0;
    for (int m = g0; m < g1; ++m) rank += ld(tmp, m) < i0 + 64 * u;
    mem[g0 + rank] = i0 + 64 * u;
  }
}


// ---------------------------------------------------------------------------------------------------
// In-place event (the steady state without rewriting the cache).  The live slots are not kept in age order:
// the caller's `order` lists the slots below `budget` from oldest to newest and the slots from `budget` on
// (appended since the last event) follow in slot order.  The merged slots are rewritten where they are, the
// retained slots that absorb nothing are not touched at all, and the retained tokens of the append region move
// into the slots that evicted tokens leave below `budget` (there are exactly as many), so that afterwards the
// slots below `budget` are all live, len = budget, and decode steps append behind them as before.
//
// merge_inplace_kernel, one workgroup per head.  The head's match list (at most kDirectMaxEvict entries) is
// grouped by target in LDS: every entry counts the earlier entries with its target (its place in the group,
// so members keep list order, the compacting kernel's summation order) and all of them (the group's size); the
// first entry of each target is its leader, the leaders are numbered by a ballot compaction and a scan over
// their sizes gives each group its range of the member array.  The targets are then dealt to the lane groups,
// which write the merged row over the retained slot.  Nothing that any group reads (its own retained row,
// evicted rows) is written by another group.  The same workgroup then moves the append region's retained tokens.
constexpr int kInplaceThreads = 512;
template <typename T, int D>
__global__ __launch_bounds__(kInplaceThreads) void merge_inplace_kernel(MergeParams p, int32_t* __restrict__ order) {
  constexpr int EPL = 16 / (int)sizeof(T), LPS = D / EPL, GPB = kInplaceThreads / LPS, kWaves = kInplaceThreads / 64;
  static_assert(kInplaceThreads >= kDirectMaxEvict, "one list entry per thread");
  __shared__ int s_match[kDirectMaxEvict], s_evict[kDirectMaxEvict];
  __shared__ int s_tgt[kDirectMaxEvict], s_cnt[kDirectMaxEvict], s_start[kDirectMaxEvict], s_tidx[kDirectMaxEvict];
  __shared__ int s_members[kDirectMaxEvict];
  __shared__ int s_hole[kDirectMaxEvict], s_mover[kDirectMaxEvict];
  __shared__ int s_wcnt[kWaves];
  __shared__ long long s_drop;
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = tid % LPS, grp = tid / LPS;
  const int t_head = p.st_obs[unit];
  const int n_ev = min(p.n_evict[unit], kDirectMaxEvict);
  if (n_ev <= 0) return;                              // uniform over the workgroup
  const size_t sbase = (size_t)unit * p.scap;
  int mt = -1, ev = 0;
  if (tid < n_ev) {
    mt = p.match[(size_t)unit * p.max_evict + tid];
    ev = p.evict_idx[(size_t)unit * p.max_evict + tid];
    s_match[tid] = mt;
    s_evict[tid] = ev;
  }
  if (tid == 0) s_drop = 0;
  __syncthreads();
  if (p.dropped_votes != nullptr && tid < n_ev && mt < 0) {
    const long long drop = p.svotes[sbase + ev];
    if (drop != 0) atomicAdd((unsigned long long*)&s_drop, (unsigned long long)drop);
  }
  const bool matched = tid < n_ev && mt >= 0 && mt < p.budget;
  int place = 0, size = 0, first = tid;               // among the entries with this entry's target
  if (matched)
    for (int j = 0; j < n_ev; ++j) {
      const bool same = s_match[j] == mt;
      size += same;
      place += same && j < tid;
      if (same && j < first) first = j;
    }
  const bool leader = matched && place == 0;
  // uniform helper: flagged threads below the caller, and in total (two barriers)
  auto compact = [&](bool flag, int& total) -> int {
    const unsigned long long m = __ballot(flag);
    __syncthreads();                                  // the previous use of s_wcnt is over
    if (lane == 0) s_wcnt[wave] = __popcll(m);
    __syncthreads();
    int below = 0;
    total = 0;
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) below += s_wcnt[w];
      total += s_wcnt[w];
    }
    return below + __popcll(m & ((1ull << lane) - 1ull));
  };
  int nt = 0;
  const int my_t = compact(leader, nt);               // the leader's group number (list order of first entries)
  if (leader) {
    s_tgt[my_t] = mt;
    s_cnt[my_t] = size;
    s_tidx[tid] = my_t;
  }
  __syncthreads();
  if (tid < nt) {                                     // start of each group's range: a scan over at most 256 sizes
    int run = 0;
    for (int t = 0; t < tid; ++t) run += s_cnt[t];
    s_start[tid] = run;
  }
  __syncthreads();
  if (matched) s_members[s_start[s_tidx[first]] + place] = ev;
  __syncthreads();
  if (tid == 0 && p.dropped_votes != nullptr && s_drop != 0) p.dropped_votes[unit] += s_drop;

  const uint4* sk = reinterpret_cast<const uint4*>(p.sk);
  const uint4* sv = reinterpret_cast<const uint4*>(p.sv);
  uint4* dk = reinterpret_cast<uint4*>(p.dk);
  uint4* dv = reinterpret_cast<uint4*>(p.dv);
  for (int t0 = 0; t0 < nt; t0 += GPB) {              // uniform trip count: a group without a target has nothing to merge
    // (the targets are dealt to the wavefronts in turn: a wavefront sums its positions' rows one after the other)
    const int t = t0 + (grp % (64 / LPS)) * kWaves + wave;
    const bool active = t < nt;
    const int ti = active ? t : 0;
    const int r = s_tgt[ti];
    const int c = p.keep_idx[(size_t)unit * p.budget + r];
    const int nm = active && c >= 0 ? s_cnt[ti] : 0;
    merge_positions<T, D>(p, unit, t_head, max(c, 0), s_members, s_start[ti], nm, max(c, 0));
  }

  // ---- move the retained tokens of the append region into the evicted slots below `budget`.  Every read of an
  // evicted row of this head happened above, in this workgroup: the barriers inside compact() order them before
  // the writes below.  The k-th retained token at or beyond `budget` (in keep-list order) goes to the k-th
  // evicted slot below `budget` (in evict-list order); `order` becomes the keep list with the moved tokens at
  // their new slots; len becomes the number of retained tokens.  Sources and destinations are disjoint.
  int32_t* ord = order + (size_t)unit * p.budget;
  const int32_t* keep = p.keep_idx + (size_t)unit * p.budget;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wavefront's merged rows are written (a mover may be one of them)
  int n_hole = 0;
  {
    const bool hole = tid < n_ev && ev >= 0 && ev < p.budget;
    const int at = compact(hole, n_hole);
    if (hole) s_hole[at] = ev;
  }
  int n_mover = 0;
  for (int r0 = 0; r0 < p.budget; r0 += kInplaceThreads) {   // uniform trip count
    const int r = r0 + tid;
    const int c = r < p.budget ? keep[r] : -1;
    const bool mover = c >= p.budget;
    int cnt = 0;
    const int at = n_mover + compact(mover, cnt);
    if (mover && at < kDirectMaxEvict) s_mover[at] = r;
    if (r < p.budget && !mover && c >= 0) ord[r] = c;
    n_mover += cnt;
  }
  __syncthreads();
  const int n_move = min(min(n_mover, n_hole), kDirectMaxEvict);
  for (int k = grp; k < n_move; k += GPB) {
    const int r = s_mover[k];
    const size_t src = sbase + keep[r], dst = sbase + s_hole[k];
    dk[dst * LPS + sub] = sk[src * LPS + sub];
    dv[dst * LPS + sub] = sv[src * LPS + sub];
    if (sub == 0) {
      p.dvotes[dst] = p.svotes[src];
      p.dlog_s[dst] = p.slog_s[src];
      p.dborn[dst] = p.sborn[src];
      ord[r] = s_hole[k];
    }
  }
  if (tid == 0) p.dlen[unit] = p.slen[unit] - n_ev;
}

}  // namespace

// Positions that a wavefront of merge_apply_kernel takes (lps lanes each).  Side by side they share the f64 scalars;
// but a wavefront sums the rows of long lists one position after the other, so with few positions on the chip it takes
// fewer, until there are kApplyWaves wavefronts (four for each SIMD): 24 heads x 501 positions
// of D 64 take 38 us with eight positions per wavefront and 25 with four; more wavefronts than that lose (64 heads x
// 820 positions, mostly copies: 16.7 us at 4096, 20.4 at 16384, 27.6 at 65536).  Short prefills have short lists and take
// half as many (whole call, D 64, 4096 / 2048: 56 heads x 217 slots 21.7 / 18.5 us, 16 x 523 20.4 / 19.2; but 16 x 1450
// 27.1 / 28.2, 8 x 3238 with lists of hundreds 173 / 253).
constexpr int kApplyWaves = 4096;
static int positions_per_wave(unsigned units, int positions, int lps, int waves = kApplyWaves) {
  int ppw = 64 / lps;
  while (ppw > 1 && (long)units * positions / ppw < waves) ppw /= 2;
  return ppw;
}

PrefillMergePlan plan_prefill_merge(const keepkv_layout* L, int capacity) {
  PrefillMergePlan pl;
  const size_t units = (size_t)L->batch * L->n_kv_heads;
  pl.keep_off = kWorkspaceHead;
  pl.start_off = pl.keep_off + align_up(units * capacity * sizeof(int32_t), 256);
  pl.member_off = pl.start_off + align_up(units * ((size_t)capacity + 1) * sizeof(int32_t), 256);
  pl.work_off = pl.member_off + align_up(units * capacity * sizeof(int32_t), 256);
  const size_t pad = (size_t)((capacity + kGroupThreads - 1) / kGroupThreads) * kGroupThreads;
  pl.bytes = pl.work_off + (capacity > kPrefillLdsSlots ? align_up(units * 2 * pad * sizeof(int32_t), 256) : 0);
  return pl;
}

MergePlan plan_merge(const keepkv_layout* L, int capacity, int budget) {
  MergePlan pl;
  const size_t units = (size_t)L->batch * L->n_kv_heads;
  pl.start_off = kWorkspaceHead;
  pl.member_off = kWorkspaceHead + align_up(units * (budget + 1) * sizeof(int32_t), 256);
  pl.bytes = pl.member_off + align_up(units * capacity * sizeof(int32_t), 256);
  return pl;
}

}  // namespace kk

extern "C" keepkv_status keepkv_merge(const keepkv_layout* layout, const keepkv_cache* src, keepkv_cache* dst,
                                      int32_t budget, const int32_t* keep_idx, const int32_t* evict_idx,
                                      const int32_t* n_evict, const int32_t* match, float alpha,
                                      int64_t* dropped_votes, void* workspace, size_t workspace_bytes, void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(src) || !cache_ok(dst) || !keep_idx || !n_evict) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (budget < 1 || budget > src->capacity || dst->capacity < budget) return KEEPKV_ERR_INVALID_ARG;
  const int max_evict = src->capacity - budget;
  if (max_evict > 0 && (!evict_idx || !match)) return KEEPKV_ERR_INVALID_ARG;
  if (!(alpha >= 0.f && alpha < 1.f)) return KEEPKV_ERR_INVALID_ARG;
  if (src->k == dst->k || src->v == dst->v || src->votes == dst->votes || src->log_s == dst->log_s ||
      src->born == dst->born || src->t_obs == dst->t_obs)
    return KEEPKV_ERR_INVALID_ARG;
  if (!aligned16(src->k) || !aligned16(src->v) || !aligned16(dst->k) || !aligned16(dst->v)) return KEEPKV_ERR_INVALID_ARG;
  if (layout->head_dim != 64 && layout->head_dim != 128) return KEEPKV_ERR_UNSUPPORTED;
  if (budget > kMaxBudget || max_evict > kMaxEvict) return KEEPKV_ERR_UNSUPPORTED;
  const MergePlan pl = plan_merge(layout, src->capacity, budget);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  const unsigned units = (unsigned)(layout->batch * layout->n_kv_heads);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  int32_t* start = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.start_off);
  int32_t* members = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.member_off);

  const size_t place_bytes = ((size_t)max_evict * sizeof(uint16_t) + 15) / 16 * 16;   // (read 16 bytes at a time)
  static const bool allowed = hipFuncSetAttribute((const void*)merge_group_kernel<8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                  8 * kGroupThreads * (int)sizeof(uint16_t)) == hipSuccess &&
                              hipFuncSetAttribute((const void*)merge_group_kernel<32>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                  kMaxEvict * (int)sizeof(uint16_t)) == hipSuccess;
  if (!allowed) return KEEPKV_ERR_DEVICE;
  const bool direct = max_evict <= kDirectMaxEvict;   // the steady state: the apply kernel finds its members itself
  if (!direct) {
    int shares = (int)(256 / units);
    // (more than eight only with 128 entries for each: 8 heads of 300 entries, the whole event, 12.2 us with eight, 12.8 with 32; of 4000 17.1 and 15.6)
    const int most = max_evict / 128 < 8 ? 8 : (max_evict / 128 > kMaxGroupShares ? kMaxGroupShares : max_evict / 128);
    shares = shares < 1 ? 1 : (shares > most ? most : shares);
    if (shares > budget) shares = budget;
    auto group = [&](auto kernel) {
      kernel<<<units * shares, kGroupThreads, place_bytes, st>>>(match, evict_idx, n_evict, src->votes, start, members, dropped_votes,
                                                                 src->capacity, budget, max_evict, shares);
    };
    if (max_evict <= 8 * kGroupThreads) group(merge_group_kernel<8>);
    else group(merge_group_kernel<32>);
  }
  MergeParams p;
  p.sk = src->k; p.sv = src->v; p.svotes = src->votes; p.slog_s = src->log_s; p.sborn = src->born; p.st_obs = src->t_obs; p.slen = src->len;
  p.dk = dst->k; p.dv = dst->v; p.dvotes = dst->votes; p.dlog_s = dst->log_s; p.dborn = dst->born; p.dt_obs = dst->t_obs; p.dlen = dst->len;
  p.keep_idx = keep_idx; p.n_evict = n_evict; p.start = start; p.members = members;
  p.match = match; p.evict_idx = evict_idx; p.dropped_votes = dropped_votes;
  p.scap = src->capacity; p.dcap = dst->capacity; p.budget = budget; p.max_evict = max_evict;
  p.write_len = 1;
  p.ln_alpha = alpha > 0.f ? log((double)alpha) : -INFINITY;
  const int esz = layout->dtype == KEEPKV_BF16 ? 2 : 4;
  p.positions_per_wave = direct ? 64 / (layout->head_dim * esz / 16) : positions_per_wave(units, budget, layout->head_dim * esz / 16);
  const dim3 grid((budget + 4 * p.positions_per_wave - 1) / (4 * p.positions_per_wave), units);
  if (layout->dtype == KEEPKV_BF16) {
    if (layout->head_dim == 128) {
      if (direct) merge_apply_kernel<uint16_t, 128, true><<<grid, 256, 0, st>>>(p);
      else merge_apply_kernel<uint16_t, 128, false><<<grid, 256, 0, st>>>(p);
    } else {
      if (direct) merge_apply_kernel<uint16_t, 64, true><<<grid, 256, 0, st>>>(p);
      else merge_apply_kernel<uint16_t, 64, false><<<grid, 256, 0, st>>>(p);
    }
  } else {
    if (layout->head_dim == 128) {
      if (direct) merge_apply_kernel<float, 128, true><<<grid, 256, 0, st>>>(p);
      else merge_apply_kernel<float, 128, false><<<grid, 256, 0, st>>>(p);
    } else {
      if (direct) merge_apply_kernel<float, 64, true><<<grid, 256, 0, st>>>(p);
      else merge_apply_kernel<float, 64, false><<<grid, 256, 0, st>>>(p);
    }
  }
  return launch_status();
}

extern "C" keepkv_status keepkv_merge_inplace(const keepkv_layout* layout, keepkv_cache* cache, int32_t* order,
                                              int32_t budget, const int32_t* keep_idx, const int32_t* evict_idx,
                                              const int32_t* n_evict, const int32_t* match, float alpha,
                                              int64_t* dropped_votes, void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(cache) || !order || !keep_idx || !n_evict) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (budget < 1 || budget > cache->capacity) return KEEPKV_ERR_INVALID_ARG;
  const int max_evict = cache->capacity - budget;
  if (max_evict > 0 && (!evict_idx || !match)) return KEEPKV_ERR_INVALID_ARG;
  if (!(alpha >= 0.f && alpha < 1.f)) return KEEPKV_ERR_INVALID_ARG;
  if (!aligned16(cache->k) || !aligned16(cache->v)) return KEEPKV_ERR_INVALID_ARG;
  if (layout->head_dim != 64 && layout->head_dim != 128) return KEEPKV_ERR_UNSUPPORTED;
  if (budget > kMaxBudget || max_evict > kDirectMaxEvict) return KEEPKV_ERR_UNSUPPORTED;
  if (max_evict == 0) return KEEPKV_OK;                // nothing can have been evicted
  const unsigned units = (unsigned)(layout->batch * layout->n_kv_heads);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  MergeParams p;
  p.sk = cache->k; p.sv = cache->v; p.svotes = cache->votes; p.slog_s = cache->log_s; p.sborn = cache->born; p.st_obs = cache->t_obs; p.slen = cache->len;
  p.dk = cache->k; p.dv = cache->v; p.dvotes = cache->votes; p.dlog_s = cache->log_s; p.dborn = cache->born; p.dt_obs = cache->t_obs; p.dlen = cache->len;
  p.keep_idx = keep_idx; p.n_evict = n_evict; p.start = nullptr; p.members = nullptr;
  p.match = match; p.evict_idx = evict_idx; p.dropped_votes = dropped_votes;
  p.scap = cache->capacity; p.dcap = cache->capacity; p.budget = budget; p.max_evict = max_evict;
  p.write_len = 0;
  p.ln_alpha = alpha > 0.f ? log((double)alpha) : -INFINITY;
  if (layout->dtype == KEEPKV_BF16) {
    if (layout->head_dim == 128) {
      merge_inplace_kernel<uint16_t, 128><<<units, kInplaceThreads, 0, st>>>(p, order);
    } else {
      merge_inplace_kernel<uint16_t, 64><<<units, kInplaceThreads, 0, st>>>(p, order);
    }
  } else {
    if (layout->head_dim == 128) {
      merge_inplace_kernel<float, 128><<<units, kInplaceThreads, 0, st>>>(p, order);
    } else {
      merge_inplace_kernel<float, 64><<<units, kInplaceThreads, 0, st>>>(p, order);
    }
  }
  return launch_status();
}

extern "C" keepkv_status keepkv_prefill_merge(const keepkv_layout* layout, const keepkv_cache* src, keepkv_cache* dst,
                                              const int32_t* near, float alpha, void* workspace,
                                              size_t workspace_bytes, void* stream) {
  using namespace kk;
  if (!layout_ok(layout) || !cache_ok(src) || !cache_ok(dst) || !near) return KEEPKV_ERR_INVALID_ARG;
  if (!units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  if (dst->capacity < src->capacity || !(alpha >= 0.f && alpha < 1.f)) return KEEPKV_ERR_INVALID_ARG;
  if (src->k == dst->k || src->v == dst->v || src->votes == dst->votes || src->log_s == dst->log_s ||
      src->born == dst->born || src->t_obs == dst->t_obs || src->len == dst->len)
    return KEEPKV_ERR_INVALID_ARG;
  if (!aligned16(src->k) || !aligned16(src->v) || !aligned16(dst->k) || !aligned16(dst->v)) return KEEPKV_ERR_INVALID_ARG;
  if (layout->head_dim != 64 && layout->head_dim != 128) return KEEPKV_ERR_UNSUPPORTED;
  const int cap = src->capacity;
  if (cap > kPrefillMaxSlots) return KEEPKV_ERR_UNSUPPORTED;
  const PrefillMergePlan pl = plan_prefill_merge(layout, cap);
  if (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace)) return KEEPKV_ERR_WORKSPACE;
  const unsigned units = (unsigned)(layout->batch * layout->n_kv_heads);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  int32_t* keep = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.keep_off);
  int32_t* start = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.start_off);
  int32_t* members = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.member_off);

  const int per = (cap + kGroupThreads - 1) / kGroupThreads;
  if (cap <= kPrefillLdsSlots) {
    const size_t lds = (size_t)2 * per * kGroupThreads * sizeof(int);
    static const hipError_t attr = hipFuncSetAttribute((const void*)prefill_group_kernel<kPrefillLdsSlots / kGroupThreads, false>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       2 * kPrefillLdsSlots * (int)sizeof(int));
    if (attr != hipSuccess) return KEEPKV_ERR_DEVICE;
    prefill_group_kernel<kPrefillLdsSlots / kGroupThreads, false><<<units, kGroupThreads, lds, st>>>(
        near, src->len, keep, start, members, dst->len, cap, nullptr);
  } else {
    int32_t* work = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + pl.work_off);
    prefill_group_kernel<kPrefillMaxSlots / kGroupThreads, true><<<units, kGroupThreads, 0, st>>>(
        near, src->len, keep, start, members, dst->len, cap, work);
  }

  MergeParams p;
  p.sk = src->k; p.sv = src->v; p.svotes = src->votes; p.slog_s = src->log_s; p.sborn = src->born; p.st_obs = src->t_obs; p.slen = src->len;
  p.dk = dst->k; p.dv = dst->v; p.dvotes = dst->votes; p.dlog_s = dst->log_s; p.dborn = dst->born; p.dt_obs = dst->t_obs; p.dlen = dst->len;
  p.keep_idx = keep; p.n_evict = nullptr; p.start = start; p.members = members;
  p.match = nullptr; p.evict_idx = nullptr; p.dropped_votes = nullptr;
  p.scap = cap; p.dcap = dst->capacity; p.budget = cap; p.max_evict = 0;
  p.write_len = 0;
  p.ln_alpha = alpha > 0.f ? log((double)alpha) : -INFINITY;
  const int esz = layout->dtype == KEEPKV_BF16 ? 2 : 4;
  p.positions_per_wave = positions_per_wave(units, cap, layout->head_dim * esz / 16, cap <= 1024 ? kApplyWaves / 2 : kApplyWaves);
  const dim3 grid((cap + 4 * p.positions_per_wave - 1) / (4 * p.positions_per_wave), units);
  if (layout->dtype == KEEPKV_BF16) {
    if (layout->head_dim == 128) merge_apply_kernel<uint16_t, 128, false><<<grid, 256, 0, st>>>(p);
    else merge_apply_kernel<uint16_t, 64, false><<<grid, 256, 0, st>>>(p);
  } else {
    if (layout->head_dim == 128) merge_apply_kernel<float, 128, false><<<grid, 256, 0, st>>>(p);
    else merge_apply_kernel<float, 64, false><<<grid, 256, 0, st>>>(p);
  }
  return launch_status();
}

#ifdef KEEPKV_TRACE
extern "C" int keepkv_trace_read_merge(long long* host, int n) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(kk::kk_trace_merge), sizeof(long long) * n);
}
#endif
