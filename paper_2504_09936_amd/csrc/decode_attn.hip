// keepkv_decode_attn / keepkv_decode_step: vote-weighted flash-decode attention (Eq. 6) with
// split-K over slots, optionally fused with the cache append (Sec. 3.1) and the EMA score update
// (Eq. 8) so that one decode step of one layer is a single kernel.
//
// One workgroup handles one (batch, kv head, split).  bf16 caches run both contractions on the matrix
// cores (decode_mfma_kernel below, 4 or 8 wavefronts per workgroup).  In the vector-ALU kernel (f32
// caches, 4 wavefronts) a slot's row (D elements) is spread over LPS consecutive lanes, 16 bytes per lane, so one wavefront load instruction
// streams 64/LPS whole rows, fully coalesced.  Each lane group computes the G logits of its
// slot with bf16 dot2 (or f32 fma) plus a DPP all-reduce inside the group, keeps its own
// online-softmax state in the log2 domain with log2(votes) folded into the logit, and
// accumulates p * v for its 16-byte slice of V.  Lane groups and wavefronts are combined through
// shuffles and LDS; splits are combined by the last workgroup of each head to finish (a ticket
// counter in the workspace head), so no second kernel is launched.
#include <math.h>
#include <string.h>

#include <mutex>

#include <type_traits>
#include <utility>

#include "kk_common.hpp"

namespace kk {

// Phase timestamps for kernel tuning; compiled in only with -DKEEPKV_TRACE (never in the product build).
#ifdef KEEPKV_TRACE
__device__ long long kk_trace[8 * 8192];
#define KK_TS(i) do { const int b_ = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x; if (threadIdx.x == 0 && b_ < 8192) \
  kk_trace[b_ * 8 + (i)] = wall_clock64(); } while (0)
#else
#define KK_TS(i) do { } while (0)
#endif

namespace {

struct DecodeParams {
  const void* q;
  void* k;            // written only in step mode (the appended row)
  void* v;
  int32_t* votes;
  float* log_s;       // step mode / score fusion
  int32_t* born;      // step mode: the new slot's origin (a slot's observation count is t_obs - born)
  int32_t* t_obs;     // step mode: [B * Hkv] steps observed by the head, += 1 per step
  int32_t* len;
  const void* k_t;    // step mode: [B, Hkv, D] new token, else null
  const void* v_t;
  int32_t* overflow;
  void* out;
  float* logits_out;
  float* lse_out;
  float* partial;     // [B*Hkv, nsplit, split_stride]
  int32_t* ticket;    // [B*Hkv] zero between launches
  uint64_t* arrivals; // [B*Hkv] zero between launches: where the head's workgroups run (null: not recorded, any XCD)
  int32_t* ticket_xcd;   // [B*Hkv] zero between launches, like `ticket` but counted in the L2 of the head's XCD
  int split_stride;   // floats between the partial results of two splits
  int n_kv_heads;
  int capacity;
  int nsplit;
  int per;          // slots per split
  int len_hint;     // caller's upper bound on len (0: none)
  int waves;        // wavefronts per workgroup of the matrix-core kernel (4 or 8)
  float scale;
  float ln_alpha, ln_1m_alpha;
};

constexpr int kWavesPerBlock = 4;   // the vector-ALU kernel

// Control words of heads whose workgroups may share an XCD: at most kMaxXcdUnits heads, behind their tickets.
constexpr int kMaxXcdUnits = 2048;
constexpr size_t kXcdTicketsOff = 16 * 1024, kArrivalsOff = 32 * 1024;
static_assert(kMaxXcdUnits * sizeof(int32_t) <= kXcdTicketsOff && kXcdTicketsOff + kMaxXcdUnits * sizeof(int32_t) <= kArrivalsOff &&
              kArrivalsOff + kMaxXcdUnits * sizeof(uint64_t) <= kMatchCountersOff, "control words");
constexpr size_t kLine = 128;       // bytes of a cache line
inline int xcd_split_stride(const keepkv_layout* L) {           // floats of a split's partial result, whole lines
  return (int)align_up((size_t)L->n_q_heads / L->n_kv_heads * (L->head_dim + 2), kLine / sizeof(float));
}
// The matrix-core kernel comes with 4 and with 8 wavefronts per workgroup (64 / 128 KB of tile buffers at
// D = 128: two workgroups or one per compute unit); plan_decode picks.


// Asynchronous copy of 16 bytes per lane from base + lane_off + off (`bytes` long from base: beyond it reads give zero) to
// LDS, through a buffer descriptor: the compiler counts these in the order of issue, while behind a global_load_lds it
// waits for everything before it uses any register load.
template <int AUX>
__device__ __forceinline__ void copy_to_lds(const unsigned char* base, size_t bytes, unsigned char* lds, uint32_t lane_off,
                                            uint32_t off) {
#ifdef __HIP_DEVICE_COMPILE__                    // (the descriptor's type does not exist in the host pass)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, (int)bytes, 0x00027000),
      (__attribute__((address_space(3))) void*)lds, 16, lane_off, off, 0, AUX);
#endif
}

constexpr float kLowest = -3.402823466e38f;   // lower end of the running maxima: finite, so that maxima can be subtracted

__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// loads of what another workgroup of this XCD wrote (see all_on_this_xcd): L1 holds none of these lines, so L2 serves them
__device__ __forceinline__ float ld_xcd(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void ld_xcd2(const float* p, float& a, float& b) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  a = __builtin_bit_cast(float, (uint32_t)v);
  b = __builtin_bit_cast(float, (uint32_t)(v >> 32));
}

// Two floats that live side by side, as one device-scope access.
__device__ __forceinline__ void st_agent2(float* p, float a, float b) {
  const uint64_t v = (uint64_t)__builtin_bit_cast(uint32_t, a) | (uint64_t)__builtin_bit_cast(uint32_t, b) << 32;
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ld_agent2(const float* p, float& a, float& b) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  a = __builtin_bit_cast(float, (uint32_t)v);
  b = __builtin_bit_cast(float, (uint32_t)(v >> 32));
}

// a <- {a of the lower half, b of the lower half}, b <- {a of the upper half, b of the upper half} (lanes 0 .. 31 / 32 .. 63)
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  const uint32_t ra = r[0], rb = r[1];           // (a bit cast of a vector element itself reads element 0)
  a = __builtin_bit_cast(float, ra);
  b = __builtin_bit_cast(float, rb);
}
// the same for the rows of 16 lanes of each half: a <- {a row 0, b row 0, a row 2, b row 2}, b <- {a row 1, b row 1, a 3, b 3}
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  const uint32_t ra = r[0], rb = r[1];           // (a bit cast of a vector element itself reads element 0)
  a = __builtin_bit_cast(float, ra);
  b = __builtin_bit_cast(float, rb);
}
// maximum / sum over the lanes that hold the same head: equal l16 mod G in all four rows of 16 lanes
template <int G, typename F>
__device__ __forceinline__ float over_head_lanes(float x, F op) {
  if constexpr (G <= 1) x = op(x, dpp_f32<0x121>(x));   // row_ror:1
  if constexpr (G <= 2) x = op(x, dpp_f32<0x122>(x));   // row_ror:2
  if constexpr (G <= 4) x = op(x, dpp_f32<0x124>(x));   // row_ror:4
  x = op(x, dpp_f32<0x128>(x));                         // row_ror:8
  float y = x;
  swap_rows(x, y);
  x = y = op(x, y);
  swap_halves(x, y);
  return op(x, y);
}

// over the 16 lanes of a row
template <typename F>
__device__ __forceinline__ float row_reduce(float x, F op) {
  x = op(x, dpp_f32<0xB1>(x));                          // quad_perm [1,0,3,2]
  x = op(x, dpp_f32<0x4E>(x));                          // quad_perm [2,3,0,1]
  x = op(x, dpp_f32<0x141>(x));                         // row_half_mirror
  return op(x, dpp_f32<0x140>(x));                      // row_mirror
}

// ---- heads whose workgroups all run on one XCD ----------------------------------------------------------------
// Partial results and a ticket that travel at device scope go to memory and back three times (store, ticket, load), about
// 2.5 us of a 10 us step; through the L2 that the workgroups of one XCD share it is a third of that.  Workgroups are dealt to the
// eight XCDs in turn, so the grid puts the splits of a head eight workgroup ids apart; but that order is a habit of
// the hardware and nothing documented, so a workgroup only relies on what it can read: its own XCD's number.  It adds it to the head's
// `arrivals` when it starts (byte x: workgroups on XCD x; device scope, nothing waits for it) and looks at the word before it publishes its
// result, some microseconds later.  If by then all splits have arrived, all on its own XCD, it publishes within that XCD; every
// other workgroup of the head sees the same word and does the same, because a workgroup that finds the word incomplete
// marks it (kArriveMark, compare-and-swap on the incomplete word), and a marked word stays marked, so that those who look later
// use device scope too.
// What it gives stands at xcd_pays.  Arriving behind the copies of the query rows (whose address translation it then waits for) made short
// last splits look in vain: 8 heads x 1180 slots in six 8.0 us, 7.1 so, 7.4 through memory.
constexpr uint64_t kArriveMark = 1ull << 63;
constexpr int kMaxLocalSplits = 16;             // (at most 127: a byte of `arrivals`, less the mark)
__device__ __forceinline__ int xcd_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)); }   // XCC_ID[3:0]
__device__ __forceinline__ uint64_t ld_arrivals(const DecodeParams& p, int unit) {
  return __hip_atomic_load(&p.arrivals[unit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// v: the word as last read.  One thread per workgroup.  A workgroup with a short split may be done before the others of its head have
// arrived; it looks a few times more before it gives up.
constexpr int kLooks = 6;
__device__ __forceinline__ bool all_on_this_xcd(const DecodeParams& p, int unit, uint64_t v) {
  const uint64_t here = (uint64_t)p.nsplit << (8 * xcd_id());
  int looks = 0;
  while (v != here && !(v & kArriveMark)) {
    int sum = 0;
    for (int x = 0; x < 64; x += 8) sum += (int)(v >> x) & 255;
    if (sum >= p.nsplit) break;                  // complete, on several XCDs
    if (looks++ < kLooks) {
      v = ld_arrivals(p, unit);
      continue;
    }
    // still incomplete: mark it (at most nsplit attempts fail, one for each arrival)
    if (__hip_atomic_compare_exchange_strong(&p.arrivals[unit], &v, v | kArriveMark, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT))
      break;
  }
  return v == here;
}

// Everything after the workgroup's kParts partial softmax states (m, l, acc[D] per head) have been
// deposited in LDS and a barrier has passed: reduce them; a single split finishes the head, otherwise the
// partial result goes to the workspace and the last workgroup of the head to arrive combines the splits,
// resets the ticket and (step mode) publishes the new len.
// acc of a part: [D][G] (kInner) or [G][D]; parts are acc_stride / ml_stride floats apart.  A split's partial result in
// the workspace: acc in the same order, then (m, l) per head.
// one_xcd (uniform): every workgroup of the head runs on this XCD and knows it (see all_on_this_xcd).
// An empty part or split has l = 0 and any m; maxima are held at or above the lowest finite value, so that they can be
// subtracted without a test for -inf.
template <typename T, int D, int G, int kParts, bool STEP, int WAVES, bool kInner, bool kSolo, bool kMayShareXcd>
__device__ __forceinline__ void combine_and_finish(const DecodeParams& p, const float* s_m, const float* s_l,
                                                   const float* s_acc, int ml_stride, int acc_stride, int* s_last_p,
                                                   int unit, int split, bool grow, int len, int t_old, bool one_xcd_) {
  const bool one_xcd = kMayShareXcd && one_xcd_;
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int kThreads = WAVES * kWave;
  int& s_last = *s_last_p;
  auto head_of = [](int idx) { return kInner ? idx % G : idx / D; };
  auto finish = [&](int idx, float M, float L, float A) {
    const int g = head_of(idx), d = kInner ? idx / G : idx % D;
    const size_t row = (size_t)unit * G + g;   // == b * Hq + h * G + g
    const float o = (L > 0.f) ? A / L : 0.f;
    if constexpr (kBf16)
      reinterpret_cast<uint16_t*>(p.out)[row * D + d] = (uint16_t)f32_to_bf16_bits(o);
    else
      reinterpret_cast<float*>(p.out)[row * D + d] = o;
    if (d == 0 && p.lse_out != nullptr) p.lse_out[row] = (L > 0.f) ? (M + fast_log2(L)) * kLn2 : -INFINITY;
  };

  float* const partials = p.partial + (size_t)unit * p.nsplit * p.split_stride;   // this head's splits
  // kInner: a lane's head is lane mod G for all of its elements, and what the splits weigh in that head is the same for
  // every channel, so lane i works out the weight of split i / G and the lanes of a head hand them around through a table of the wavefront's
  // own in LDS: one exponential per lane instead of one per split and element.  weigh(): n splits; m, l: those of split
  // lane / G (-inf and 0 beyond nsplit); leaves the head's M, its L (added up in the order of the splits) and the n weights.
  // (Not for the parts of a workgroup, whose maxima LDS holds at hand: the maximum over lanes, the exponential and the table
  // are one chain of latencies there, and an unsplit step of 100 to 300 slots took 0.1 us longer with them.)
  const int lane = threadIdx.x & 63;
  float* const s_c = const_cast<float*>(s_acc) + (threadIdx.x >> 6) * acc_stride + G * D + 16;   // 2 x [G][n], behind this wavefront's deposit
  auto weigh = [&](float m, float l, auto n_tag, float& M, float& L, float (&c)[decltype(n_tag)::value]) {
    constexpr int n = decltype(n_tag)::value;
    static_assert(n % 4 == 0 && n * G <= kWave, "one weight per lane");
    M = over_head_lanes<G>(m, [](float a, float b) { return fmaxf(a, b); });
    const float mine = lane < n * G ? fast_exp2(m - M) : 0.f;
    if (lane < n * G) {
      s_c[(lane % G) * n + lane / G] = mine;
      s_c[n * G + (lane % G) * n + lane / G] = l;
    }
    L = 0.f;
#pragma unroll
    for (int i = 0; i < n; i += 4) {
      const float4 t = *reinterpret_cast<const float4*>(s_c + (lane % G) * n + i);
      const float4 u = *reinterpret_cast<const float4*>(s_c + n * G + (lane % G) * n + i);
      c[i] = t.x; c[i + 1] = t.y; c[i + 2] = t.z; c[i + 3] = t.w;
      L = fmaf(u.w, t.w, fmaf(u.z, t.z, fmaf(u.y, t.y, fmaf(u.x, t.x, L))));
    }
  };
  for (int idx = threadIdx.x; idx < G * D; idx += kThreads) {
    const int g = head_of(idx);
    float M = kLowest, L = 0.f, A = 0.f;
    if constexpr (kInner) {
#pragma unroll
      for (int w = 0; w < kParts; ++w) M = fmaxf(M, s_m[w * ml_stride + g]);
#pragma unroll
      for (int w = 0; w < kParts; ++w) {
        const float c = fast_exp2(s_m[w * ml_stride + g] - M);
        L = fmaf(s_l[w * ml_stride + g], c, L);
        A = fmaf(s_acc[w * acc_stride + idx], c, A);
      }
    } else {                                     // a wavefront's elements are of one head: lane i of a row weighs part i
      // (sixteen exponentials per element before: 32 steps of 4 heads x 52 .. 84 slots and their event 145.4 us, now 143.3)
      static_assert(kInner || (kParts == 16 && D % kWave == 0), "one weight a lane");
      const int gw = __builtin_amdgcn_readfirstlane(g);
      const float m = s_m[(lane & 15) * ml_stride + gw];
      M = fmaxf(M, row_reduce(m, [](float a, float b) { return fmaxf(a, b); }));
      const float c = fast_exp2(m - M);
      L = row_reduce(s_l[(lane & 15) * ml_stride + gw] * c, [](float a, float b) { return a + b; });
#pragma unroll
      for (int w = 0; w < kParts; ++w)
        A = fmaf(s_acc[w * acc_stride + idx], __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, c), w)), A);
    }
    if (kSolo || p.nsplit == 1) {
      finish(idx, M, L, A);
    } else {
      float* dst = partials + (size_t)split * p.split_stride;
      const bool has_ml = (kInner ? idx / G : idx % D) == 0;
      if (one_xcd) {
        dst[idx] = A;
        if (has_ml) *reinterpret_cast<float2*>(dst + G * D + 2 * g) = make_float2(M, L);
      } else {                                   // device-coherent (write-through): the combining workgroup may run on another XCD
        st_agent(dst + idx, A);
        if (has_ml) st_agent2(dst + G * D + 2 * g, M, L);
      }
    }
  }

  if (kSolo || p.nsplit == 1) {
    if (STEP && threadIdx.x == 0) p.t_obs[unit] = t_old + 1;   // one more observation of every slot of the head
    if (STEP && threadIdx.x == 0 && grow) p.len[unit] = len;   // every wavefront read len before the barrier above
    if (STEP && threadIdx.x == 0 && !grow && p.overflow != nullptr) *p.overflow = 1;
    return;
  }

  KK_TS(3);
  // ---- the last workgroup of this head to arrive combines the splits ------------------------------
  // The partial results were stored write-through at device scope (or, one_xcd, into the L2 that all of the head's
  // workgroups share, where the ticket is counted too), so it is enough that every
  // wavefront's stores have completed before the ticket is taken: each wavefront waits on its own
  // memory counter (stores count there on this part), then the barrier orders all of them before
  // thread 0's ticket.  A workgroup-scope release fence emits no such wait here (the workgroup shares
  // one L2, so the compiler needs none for that scope), and a device-scope release fence would write
  // back the whole L2 per workgroup.  The combining workgroup reads the partials with device-scope loads; one_xcd: with loads
  // that find nothing in its L1, because a split's result has cache lines of its own (split_stride) that nobody reads but the
  // combining workgroup, once a launch.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int before = one_xcd ? __hip_atomic_fetch_add(&p.ticket_xcd[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                               : __hip_atomic_fetch_add(&p.ticket[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = before == p.nsplit - 1;
  }
  __syncthreads();
  KK_TS(4);
  if (!s_last) return;
  // CH splits of EB output elements are fetched per round trip of device-scope loads: 4 or 8 splits of two
  // elements when that covers all splits (the common case; surplus loads would only cost), else 16 of one
  constexpr int kPerThread = (G * D + kThreads - 1) / kThreads;   // output elements per thread
  auto combine = [&](auto ch_tag, auto eb_tag, auto xcd_tag) {
    constexpr int CH = decltype(ch_tag)::value, EB = decltype(eb_tag)::value;
    constexpr bool kXcd = decltype(xcd_tag)::value;
    for (int e0 = 0; e0 < kPerThread; e0 += EB) {
      int idx[EB];
      float M[EB], L[EB], A[EB];
#pragma unroll
      for (int j = 0; j < EB; ++j) {
        idx[j] = min((int)threadIdx.x + (e0 + j) * kThreads, G * D - 1);   // surplus threads repeat the last element
        M[j] = kLowest;
        L[j] = 0.f;
        A[j] = 0.f;
      }
      for (int s0 = 0; s0 < p.nsplit; s0 += CH) {
        float ms[EB][CH], ls[EB][CH], as[EB][CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const float* src = partials + (size_t)min(s0 + i, p.nsplit - 1) * p.split_stride;
#pragma unroll
          for (int j = 0; j < EB; ++j) {
            const float* ml = src + G * D + 2 * head_of(idx[j]);
            if constexpr (kXcd) {
              ld_xcd2(ml, ms[j][i], ls[j][i]);
              as[j][i] = ld_xcd(src + idx[j]);
            } else {
              ld_agent2(ml, ms[j][i], ls[j][i]);
              as[j][i] = ld_agent(src + idx[j]);
            }
          }
        }
#pragma unroll
        for (int j = 0; j < EB; ++j) {
          float mc = M[j];
#pragma unroll
          for (int i = 0; i < CH; ++i) mc = fmaxf(mc, ms[j][i]);
          const float c0 = fast_exp2(M[j] - mc);
          L[j] *= c0;
          A[j] *= c0;
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            const float c = s0 + i < p.nsplit ? fast_exp2(ms[j][i] - mc) : 0.f;
            L[j] = fmaf(ls[j][i], c, L[j]);
            A[j] = fmaf(as[j][i], c, A[j]);
          }
          M[j] = mc;
        }
      }
#pragma unroll
      for (int j = 0; j < EB; ++j)
        if ((int)threadIdx.x + (e0 + j) * kThreads < G * D) finish(idx[j], M[j], L[j], A[j]);
    }
  };
  // kInner and no more than CH splits: the weights once per lane (see weigh), CH values of every element per round trip
  auto combine_few = [&](auto ch_tag, auto xcd_tag) {
    constexpr int CH = decltype(ch_tag)::value;
    constexpr bool kXcd = decltype(xcd_tag)::value;
    const int mine = lane / G;
    const float* ml = partials + (size_t)min(mine, p.nsplit - 1) * p.split_stride + G * D + 2 * (lane % G);
    float m, l, as[kPerThread][CH];
    if constexpr (kXcd) ld_xcd2(ml, m, l);
    else ld_agent2(ml, m, l);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const float* src = partials + (size_t)min(i, p.nsplit - 1) * p.split_stride;
#pragma unroll
      for (int j = 0; j < kPerThread; ++j) {
        const int idx = min((int)threadIdx.x + j * kThreads, G * D - 1);   // surplus threads repeat the last element
        as[j][i] = kXcd ? ld_xcd(src + idx) : ld_agent(src + idx);
      }
    }
    float M, L, c[CH];
    weigh(mine < p.nsplit ? m : -INFINITY, mine < p.nsplit ? l : 0.f, ch_tag, M, L, c);
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
      float A = 0.f;
#pragma unroll
      for (int i = 0; i < CH; ++i) A = fmaf(as[j][i], c[i], A);
      const int idx = (int)threadIdx.x + j * kThreads;
      if (idx < G * D) finish(idx, M, L, A);
    }
  };
  constexpr int kTwo = kPerThread >= 2 ? 2 : 1;
  auto combine_all = [&](auto xcd_tag) {
    if constexpr (kInner) {
      if (p.nsplit <= 4) return combine_few(std::integral_constant<int, 4>{}, xcd_tag);
      if (p.nsplit <= 8) return combine_few(std::integral_constant<int, 8>{}, xcd_tag);
      if constexpr (G <= 4)
        if (p.nsplit <= 16) return combine_few(std::integral_constant<int, 16>{}, xcd_tag);
    }
    if (p.nsplit <= 4) combine(std::integral_constant<int, 4>{}, std::integral_constant<int, kTwo>{}, xcd_tag);
    else if (p.nsplit <= 8) combine(std::integral_constant<int, 8>{}, std::integral_constant<int, kTwo>{}, xcd_tag);
    else combine(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{}, xcd_tag);
  };
  bool combined = false;
  if constexpr (kMayShareXcd) {
    if (one_xcd) combine_all(std::true_type{});
    combined = one_xcd;
  }
  if (!combined) combine_all(std::false_type{});
  KK_TS(5);
  if (threadIdx.x == 0) {                        // the control words are ready for the next launch
    if (one_xcd) __hip_atomic_store(&p.ticket_xcd[unit], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(&p.ticket[unit], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // (every workgroup of the head looked at this word before it took its ticket)
    if (kMayShareXcd) __hip_atomic_store(&p.arrivals[unit], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (STEP) p.t_obs[unit] = t_old + 1;             // (every workgroup of the head read it before taking its ticket)
    if (STEP && grow) p.len[unit] = len;
    if (STEP && !grow && p.overflow != nullptr) *p.overflow = 1;
  }
}

// ---------------------------------------------------------------------------------------------------
// LPS lanes share one slot's row, each holding VPL 16-byte vectors of it (vector v of lane `sub` is
// row vector v * LPS + sub, so the LPS lanes of a group read LPS * 16 contiguous bytes per load).
// kUnroll slots per lane group are in flight per iteration.
// STEP: append (k_t, v_t) as a new slot, attend over old + new, update the EMA scores, bump len.
template <typename T, int D, int G, int LPS, int kUnroll, bool STEP>
__global__ __launch_bounds__(kWavesPerBlock* kWave) void decode_attn_kernel(DecodeParams p) {
  constexpr int EPV = 16 / (int)sizeof(T);              // elements per 16-byte vector
  constexpr int RV = D / EPV;                           // vectors per row
  constexpr int VPL = RV / LPS;                         // vectors per lane
  constexpr int EPL = EPV * VPL;                        // elements per lane
  constexpr int GPW = kWave / LPS;                      // slots per load instruction
  constexpr int TILE = GPW * kUnroll;                   // slots per wavefront per iteration
  constexpr bool kBf16 = sizeof(T) == 2;
  static_assert(VPL >= 1 && RV % LPS == 0 && kUnroll <= LPS, "bad lane mapping");

  extern __shared__ __align__(16) float smem[];
  __shared__ int s_last;
  __shared__ uint4 s_new[2 * RV];             // step mode: the appended token's K row, then its V row

  const int unit = blockIdx.y, split = blockIdx.x;   // unit = b * Hkv + h
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / LPS, sub = lane % LPS;
  KK_TS(0);
  const int len_old = p.len[unit];          // needed only once the row loads are in flight (see `bound`)
  const int t_old = STEP ? p.t_obs[unit] : 0;   // used at the very end only
  // step mode: the new token becomes slot len_old (unless the head is full); it is attended as one
  // extra slot after the cache slots, so the streaming loop below never depends on it
  const int start = split * p.per;
  // The wavefront that will attend the appended token copies it to LDS asynchronously (no registers,
  // no wait), so that its extra slot costs no memory round trip after the streaming loop.
  // (the last wavefront of the last split: its own share of the cache is the shortest)
  const bool takes_new = STEP && split == p.nsplit - 1 && wave == kWavesPerBlock - 1;
  if (takes_new && lane < 2 * RV) {
    const uint4* src = (lane < RV ? reinterpret_cast<const uint4*>(p.k_t) : reinterpret_cast<const uint4*>(p.v_t)) +
                       (size_t)unit * RV + (lane % RV);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)s_new, 16, 0, 0);
  }
  // Rows are fetched up to `bound`: the caller's upper bound on len if given, so that the loads do
  // not wait for the len load; otherwise len itself.  Slots at or beyond len are masked out.
  const int bound = p.len_hint > 0 ? min(p.len_hint, p.capacity) : len_old;
  const int lim = min(bound, start + p.per);

  // query slice of this lane for each head of the group
  uint4 qv[G][VPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int v = 0; v < VPL; ++v)
      qv[g][v] = reinterpret_cast<const uint4*>(p.q)[((size_t)unit * G + g) * RV + v * LPS + sub];

  float m[G], l[G], acc[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
  }

  const size_t ubase = (size_t)unit * p.capacity;
  uint4* kbase = reinterpret_cast<uint4*>(p.k) + ubase * RV + sub;
  uint4* vbase = reinterpret_cast<uint4*>(p.v) + ubase * RV + sub;
  const float sl2 = p.scale * kLog2e;

  // One tile: kUnroll slots per lane group.  `extra` is the appended token (step mode): lane group 0
  // takes it from (k_t, v_t) as its slot 0, every other slot of the tile is masked.
  auto tile = [&](int base, bool extra) {
    const int s0 = extra ? len_old : base + grp * kUnroll;
    uint4 kk_[kUnroll][VPL], vv_[kUnroll][VPL];
    int pv[kUnroll];
    bool live[kUnroll];
#pragma unroll
    for (int j = 0; j < kUnroll; ++j) {
      if (extra) {                               // only slot 0 is real; it comes from LDS
        pv[j] = 1;
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
          kk_[j][v] = (j == 0) ? s_new[v * LPS + sub] : make_uint4(0, 0, 0, 0);
          vv_[j][v] = (j == 0) ? s_new[RV + v * LPS + sub] : make_uint4(0, 0, 0, 0);
        }
      } else {
        const int s = min(s0 + j, bound - 1);   // clamp: slots at or beyond `bound` are never read
        const uint4* ka = kbase + (size_t)s * RV;
        const uint4* va = vbase + (size_t)s * RV;
        pv[j] = p.votes[ubase + s];              // unconditional and in bounds: a branch behind a
#pragma unroll                                   // load would serialise the row loads
        for (int v = 0; v < VPL; ++v) {
          kk_[j][v] = load_once(ka + v * LPS);
          vv_[j][v] = load_once(va + v * LPS);
        }
      }
    }
    // EMA state of the slot this lane will update (lane `sub` < kUnroll owns slot s0 + sub)
    const int s_mine = s0 + (extra ? 0 : sub);
    float ls_old = -INFINITY;
    if (STEP && !extra) ls_old = p.log_s[ubase + min(s_mine, bound - 1)];
    // ---- first use of len: everything above was issued without waiting for it
    const int live_end = min(len_old, start + p.per);
#pragma unroll
    for (int j = 0; j < kUnroll; ++j) live[j] = extra ? (grp == 0 && j == 0) : (s0 + j < live_end);
    if (extra || base + TILE > live_end) {       // uniform over the wavefront: the tile holds masked slots;
#pragma unroll                                   // zero their V so that 0 * garbage cannot make a NaN
      for (int j = 0; j < kUnroll; ++j) {
        const uint32_t keepmask = live[j] ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
          vv_[j][v].x &= keepmask; vv_[j][v].y &= keepmask; vv_[j][v].z &= keepmask; vv_[j][v].w &= keepmask;
        }
      }
    }

    float z[G][kUnroll];
    float mean_logit[kUnroll];
#pragma unroll
    for (int j = 0; j < kUnroll; ++j) {
      const float lp = fast_log2((float)pv[j]);
      float sum = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float d = 0.f;
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
          const uint4 a = kk_[j][v], b = qv[g][v];
          if constexpr (kBf16) {
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.x), __builtin_bit_cast(bf16x2_t, b.x), d, false);
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.y), __builtin_bit_cast(bf16x2_t, b.y), d, false);
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.z), __builtin_bit_cast(bf16x2_t, b.z), d, false);
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.w), __builtin_bit_cast(bf16x2_t, b.w), d, false);
          } else {
            d = fmaf(__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, b.x), d);
            d = fmaf(__builtin_bit_cast(float, a.y), __builtin_bit_cast(float, b.y), d);
            d = fmaf(__builtin_bit_cast(float, a.z), __builtin_bit_cast(float, b.z), d);
            d = fmaf(__builtin_bit_cast(float, a.w), __builtin_bit_cast(float, b.w), d);
          }
        }
        d = group_sum<LPS>(d);
        sum += d;
        z[g][j] = live[j] ? fmaf(d, sl2, lp) : -INFINITY;
      }
      mean_logit[j] = sum * (p.scale * (1.0f / G));
    }

    {
      // every lane evaluates the update of slot s0 + (sub mod kUnroll); only the owning lanes store
      float x = mean_logit[0];
      if (!extra) {
#pragma unroll
        for (int j = 1; j < kUnroll; ++j) x = ((sub & (kUnroll - 1)) == j) ? mean_logit[j] : x;
      }
      const bool mine = extra ? (grp == 0 && sub == 0) : (sub < kUnroll && s_mine < live_end);
      if (p.logits_out != nullptr && mine) p.logits_out[ubase + s_mine] = x;
      if constexpr (STEP) {
        // log_s <- ln(alpha S + (1 - alpha) e^x)  (Eq. 8); the count advances with the head's t_obs
        const float a = p.ln_alpha + ls_old, b = p.ln_1m_alpha + x;
        const float hi = fmaxf(a, b), lo = fminf(a, b);
        const float r = (lo == -INFINITY) ? hi : hi + log1pf(expf(lo - hi));
        if (mine) p.log_s[ubase + s_mine] = r;
      }
    }
    if (STEP && extra && grp == 0) {
      // store the new token into the cache
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        kbase[(size_t)len_old * RV + v * LPS] = kk_[0][v];
        vbase[(size_t)len_old * RV + v * LPS] = vv_[0][v];
      }
      if (sub == 0) {
        p.votes[ubase + len_old] = 1;
        p.born[ubase + len_old] = t_old;          // first observed in this step
      }
    }

    // online softmax update for this group's kUnroll slots
    float pw[G][kUnroll];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float tm = z[g][0];
#pragma unroll
      for (int j = 1; j < kUnroll; ++j) tm = fmaxf(tm, z[g][j]);
      const float mn = fmaxf(m[g], tm);
      const float c = (mn == -INFINITY) ? 0.f : fast_exp2(m[g] - mn);
      m[g] = mn;
      float ps = 0.f;
#pragma unroll
      for (int j = 0; j < kUnroll; ++j) {
        pw[g][j] = (mn == -INFINITY) ? 0.f : fast_exp2(z[g][j] - mn);
        ps += pw[g][j];
      }
      l[g] = fmaf(l[g], c, ps);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] *= c;
    }
#pragma unroll
    for (int j = 0; j < kUnroll; ++j) {
      float vf[EPL];
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        const uint4 x = vv_[j][v];
        if constexpr (kBf16) {
          vf[v * 8 + 0] = bf16_lo(x.x); vf[v * 8 + 1] = bf16_hi(x.x);
          vf[v * 8 + 2] = bf16_lo(x.y); vf[v * 8 + 3] = bf16_hi(x.y);
          vf[v * 8 + 4] = bf16_lo(x.z); vf[v * 8 + 5] = bf16_hi(x.z);
          vf[v * 8 + 6] = bf16_lo(x.w); vf[v * 8 + 7] = bf16_hi(x.w);
        } else {
          vf[v * 4 + 0] = __builtin_bit_cast(float, x.x); vf[v * 4 + 1] = __builtin_bit_cast(float, x.y);
          vf[v * 4 + 2] = __builtin_bit_cast(float, x.z); vf[v * 4 + 3] = __builtin_bit_cast(float, x.w);
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(pw[g][j], vf[e], acc[g][e]);
    }
  };

  for (int base = start + wave * TILE; base < lim; base += kWavesPerBlock * TILE) tile(base, false);
  KK_TS(1);
  const bool grow = STEP && len_old < p.capacity;
  const int len = grow ? len_old + 1 : len_old;
  if (takes_new) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the asynchronous copy of the new token has landed
    if (grow) tile(0, true);
  }

  // ---- combine lane groups and wavefronts through LDS ----------------------------------------------
  // With 8 lanes per slot the two groups of a 16-lane row are merged first with one DPP rotation;
  // each row then deposits its (m, l, acc) and the workgroup reduces kParts partial states.
  if constexpr (LPS == 8) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float mo = dpp_f32<0x128>(m[g]);        // row_ror:8 = the other group of this row
      const float mw = fmaxf(m[g], mo);
      const float c = (m[g] == -INFINITY) ? 0.f : fast_exp2(m[g] - mw);
      const float lc = l[g] * c;
      l[g] = lc + dpp_f32<0x128>(lc);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float a = acc[g][e] * c;
        acc[g][e] = a + dpp_f32<0x128>(a);
      }
      m[g] = mw;
    }
  }
  constexpr int LPR = LPS < 16 ? 16 : LPS;            // lanes per deposited part
  constexpr int kParts = kWavesPerBlock * (kWave / LPR);
  float* s_m = smem;                                  // [kParts][G]
  float* s_l = s_m + kParts * G;                      // [kParts][G]
  float* s_acc = s_l + kParts * G;                    // [kParts][G][D]
  {
    const int part = wave * (kWave / LPR) + lane / LPR;
    if ((lane % LPR) < LPS) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (sub == 0) {
          s_m[part * G + g] = m[g];
          s_l[part * G + g] = l[g];
        }
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
          float4 t;
          if constexpr (EPV == 8) {
            t = make_float4(acc[g][v * 8 + 0], acc[g][v * 8 + 1], acc[g][v * 8 + 2], acc[g][v * 8 + 3]);
            *reinterpret_cast<float4*>(&s_acc[(part * G + g) * D + (v * LPS + sub) * 8]) = t;
            t = make_float4(acc[g][v * 8 + 4], acc[g][v * 8 + 5], acc[g][v * 8 + 6], acc[g][v * 8 + 7]);
            *reinterpret_cast<float4*>(&s_acc[(part * G + g) * D + (v * LPS + sub) * 8 + 4]) = t;
          } else {
            t = make_float4(acc[g][v * 4 + 0], acc[g][v * 4 + 1], acc[g][v * 4 + 2], acc[g][v * 4 + 3]);
            *reinterpret_cast<float4*>(&s_acc[(part * G + g) * D + (v * LPS + sub) * 4]) = t;
          }
        }
      }
    }
  }
  __syncthreads();
  KK_TS(2);

  combine_and_finish<T, D, G, kParts, STEP, kWavesPerBlock, false, false, false>(p, s_m, s_l, s_acc, G, G * D, &s_last, unit, split,
                                                                  grow, len, t_old, false);
}

// ---------------------------------------------------------------------------------------------------
// bf16 caches: the same decode step with both contractions on the matrix cores (16x16x32 bf16 MFMA).
//
// A wavefront owns 32-slot tiles.  Their K and V rows go global -> LDS without passing through
// registers (rows XOR-swizzled in 16-byte chunks).  Scores are formed transposed, S^T = K Q^T: the A
// operand is the K tile (row = slot), the B operand the query heads (column = head, heads repeated
// to fill 16 columns), so lane (column c, quarter q) receives the logits of head c mod G for the
// slots 16 st + 4 q + i (st = 0, 1; i = 0..3).  That is already the layout of an A operand whose row
// is the head and whose contraction index runs over those 8 slots, so the probabilities feed the
// second product O = P V without leaving their lanes; its B operand, 8 slots of one channel per
// lane, is what the LDS transpose read (ds_read_b64_tr_b16) returns from the row-major V tile.
// P is split into two bf16 terms (hi + lo, 16 significant bits), V is bf16 already, accumulation f32.
// Output rows are heads again (row r = head r mod G), 16 channels per MFMA.
constexpr int kMTile = 32;
// Cache policy of the K / V row loads: every row is read once per launch, so the loads carry the non-temporal
// hint (the `nt` bit) and do not displace what the caches hold for reuse (a plain stream of 453 MB read this way
// measured 6.9 TB/s against 6.0 TB/s without the hint, and the small read-modify-write traffic of the EMA state
// beside it cost 1 us instead of 12).
constexpr int kStreamOnce = 2;
// Per wavefront, behind the tile buffers: the head group's query rows (whole 1 KB pieces, one asynchronous
// 16-byte copy per lane each) and the tile's votes and ln S (4 bytes per lane each); the tile loop stages its
// updated ln S here instead.
constexpr int mfma_stage_bytes(int D, int G) { return (G * D * 2 + 1023) / 1024 * 1024 + 3 * 256; }

// LDS reads that the compiler does not see as such.  It orders an LDS read that it cannot tell apart from an
// outstanding global -> LDS copy behind ALL outstanding copies; these are for data whose copy the caller has
// already awaited, while later copies (to other addresses) are still under way.  The wait for the read itself
// is part of the statement.
typedef __attribute__((ext_vector_type(4))) int i32x4_t;

template <int G>
__device__ __forceinline__ float head_sum(float x) {   // sum over the G heads held by G consecutive lanes
  if constexpr (G >= 2) x += dpp_f32<0xB1>(x);          // quad_perm [1,0,3,2]
  if constexpr (G >= 4) x += dpp_f32<0x4E>(x);          // quad_perm [2,3,0,1]
  if constexpr (G >= 8) x += dpp_f32<0x141>(x);         // row_half_mirror
  return x;
}

__device__ __forceinline__ uint32_t pack_hi16(float lo_elem, float hi_elem) {   // {bf16 trunc(lo_elem), bf16 trunc(hi_elem)}
  return (__builtin_bit_cast(uint32_t, lo_elem) >> 16) | (__builtin_bit_cast(uint32_t, hi_elem) & 0xFFFF0000u);
}

// The vector ALU's share.  A SIMD has two of these wavefronts and issues one 64-lane instruction in four cycles, so what a
// tile costs beyond its loads is its instruction count: with every lane working out all 8 slots of its column (16 / G
// lanes then do the same work) a tile took 430 instructions, 0.8 us alone and 1.6 us beside a second wavefront, most of
// it after the last row had arrived.  The 16 / G lanes (c mod G equal) of a head therefore share the column's slots: lane
// r = c / G takes NV of the 8 and leaves the others' places in its row of P empty, so that row r G + g of the second
// product is head g's sum over lane r's slots and the rows of a head are added once at the end (permlane swaps).
// Addresses: a tile's base is uniform (scalar registers), a lane adds a 32-bit offset that K and V share.
// Measured before / after, graph replays, one step (D 128): 64 heads x 852 slots (G 4) 10.6 / 9.8 us, 8 heads 7.9 / 7.0,
// 128 heads x 828 16.6 / 15.7, 1024 heads x 852 (G 8) 81.9 / 80.8.  Of the 9.6 us that the first takes now the rows need 5.3 (28.6 MB), the
// reduction over the wavefronts 0.5, publishing a split's result and taking the ticket 0.8, the combination 0.8, launch and drain 2.
//
// kMode: how many tiles a wavefront has at most, and where the splits of a head meet.
// - one tile (a split of 128 or 256 slots): no tile loop, no prefetch and no rescaling of the accumulators (the common
//   steady-state shape);
// - two tiles: everything is requested before the first wait.  The loop, which requests the second tile's rows when the
//   first have landed, took 15.7 us for 128 heads x 828 slots and 16.3 us for 64 x 1683; this way 14.8 and 14.5;
// - more: a loop that requests the next tile's rows while it works on the current one.
// A launch fetches code that it does not run, too, so there are instances without what they cannot need: Solo for heads that are not
// split (without the combination 1024 heads x 852 slots 82.3 us and with it 83.0, 8 heads x 113 slots 4.0 and 4.35), Mem for splits that meet through memory, Xcd for
// those that may meet within an XCD (36 heads x 334 slots in four splits, which cannot: 6.5 us without its code, 6.95 with it).
constexpr int kLoopSolo = 0, kOneXcd = 1, kTwoMem = 2, kLoopMem = 3, kOneSolo = 4, kTwoSolo = 5, kOneMem = 6, kTwoXcd = 7, kModes = 8;
template <int D, int G, bool STEP, int kMode, int kMfmaWaves>
__global__ __launch_bounds__(kMfmaWaves* kWave, 2) void decode_mfma_kernel(DecodeParams p) {
  using T = uint16_t;
  constexpr int ROWB = D * 2, CHUNKS = ROWB / 16, KS = D / 32, NTILE = D / 16;
  constexpr int TILE_BYTES = kMTile * ROWB;
  constexpr int LOADS = TILE_BYTES / (kWave * 16);
  constexpr int kParts = kMfmaWaves;
  constexpr int NV = G >= 2 ? G / 2 : 1;         // slots of a tile whose weights one lane works out
  constexpr bool ONE = kMode == kOneXcd || kMode == kOneMem || kMode == kOneSolo;
  constexpr bool TWO = kMode == kTwoXcd || kMode == kTwoMem || kMode == kTwoSolo;
  constexpr bool LOOP = !ONE && !TWO;
  constexpr bool kSolo = kMode == kOneSolo || kMode == kTwoSolo || kMode == kLoopSolo;
  constexpr bool kMayShareXcd = kMode == kOneXcd || kMode == kTwoXcd;
  extern __shared__ __align__(256) unsigned char smem_tiles[];   // [wave][two tile buffers]; later each wave's deposit
  __shared__ int s_last, s_one_xcd;
  __shared__ __align__(16) unsigned char s_new[2 * ROWB];       // step mode: the appended token's K row, V row

  const int unit = kMayShareXcd ? (int)(blockIdx.z * 8 + blockIdx.x) : (int)blockIdx.y;
  const int split = kMayShareXcd ? blockIdx.y : blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  KK_TS(0);
  const int len_old = p.len[unit];
  const int t_old = STEP ? p.t_obs[unit] : 0;   // used at the very end only
  const int start = split * p.per;
  // This workgroup has arrived (the last wavefront, whose share is the shortest; its rows land behind this).  With one tile ahead of
  // every request, so that a workgroup whose split is short does not look too early; with two a little later, ahead of the rows: 32 heads x 2640
  // slots of 3300 in eight splits, attention alone, took 15.4 us with the former and 13.7 with the latter.
  auto arrive = [&]() {
    if (kMayShareXcd && wave == kMfmaWaves - 1 && lane == 0)
      __hip_atomic_fetch_add(&p.arrivals[unit], 1ull << (8 * xcd_id()), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if constexpr (ONE) arrive();
  const bool takes_new = STEP && split == p.nsplit - 1 && wave == kMfmaWaves - 1;
  if (takes_new) {                             // asynchronous copy of (k_t, v_t) into LDS, awaited after the loop
    const size_t at = (size_t)unit * ROWB;
    if (lane < CHUNKS)
      copy_to_lds<0>(reinterpret_cast<const unsigned char*>(p.k_t) + at, ROWB, s_new, lane * 16, 0);
    else if (lane < 2 * CHUNKS)
      copy_to_lds<0>(reinterpret_cast<const unsigned char*>(p.v_t) + at, ROWB, s_new, (lane - CHUNKS) * 16, 0);
  }
  const int bound = p.len_hint > 0 ? min(p.len_hint, p.capacity) : len_old;
  const int lim = min(bound, start + p.per);
  const size_t ubase = (size_t)unit * p.capacity;
  const unsigned char* kbytes = reinterpret_cast<const unsigned char*>(p.k) + ubase * ROWB;
  const unsigned char* vbytes = reinterpret_cast<const unsigned char*>(p.v) + ubase * ROWB;
  // ONE: [K tile | V tile] of the wavefront's single tile.  Otherwise the K rows travel straight into registers
  // (below) and the two buffers hold the V rows of the current and of the next tile.
  unsigned char* const Tb = smem_tiles + wave * (2 * TILE_BYTES);
  unsigned char* const Kb = Tb;
  unsigned char* Vb = ONE ? Tb + TILE_BYTES : Tb;
  // This lane's head and its NV slots of every tile, rows row0 .. row0 + NV - 1: the places pos0 .. of the 8 slots
  // 16 st + 4 q + i that its column of the score product holds.  row_mine: the slot whose votes and EMA state it loads
  // (one of the NV; lanes 0 .. 3 of its quad hold all of them) and, if `writer`, updates.
  const int g_l = l16 % G, r_l = l16 / G;
  const int pos0 = (r_l * NV) & 7;
  const int row0 = 16 * (pos0 >> 2) + 4 * q + (pos0 & 3);
  const int row_mine = row0 + (g_l & (NV - 1));
  const bool writer = G == 1 ? r_l < 8 : g_l < NV;
  // ONE: everything this wavefront waits for travels as asynchronous global -> LDS copies, requested in the
  // order query rows, K rows, votes and EMA state, V rows.  Such copies complete in the order of issue, so a
  // wait that leaves the V rows' LOADS copies outstanding guarantees all the others: the score product and
  // the softmax run while the V rows still travel.  (Loads into registers in the same queue would make the
  // compiler wait for everything at their first use.)
  constexpr int Q_PIECES = (G * ROWB + 1023) / 1024;
  unsigned char* s_q = smem_tiles + kMfmaWaves * 2 * TILE_BYTES + wave * mfma_stage_bytes(D, G);
  unsigned char* s_sc = s_q + Q_PIECES * 1024;                  // [votes | ln S][64] 4-byte words
  if constexpr (ONE) {                           // chunk c of head g sits at position c ^ (4 g mod CHUNKS) of its row
    const unsigned char* qbase = reinterpret_cast<const unsigned char*>(p.q) + (size_t)unit * G * ROWB;
#pragma unroll
    for (int j = 0; j < Q_PIECES; ++j) {
      const int c = min(j * kWave + lane, G * CHUNKS - 1);       // surplus lanes repeat the last chunk
      const uint32_t off = (uint32_t)((c ^ ((4 * (c / CHUNKS)) & (CHUNKS - 1))) * 16);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(qbase + off),
                                       (__attribute__((address_space(3))) void*)(s_q + j * 1024), 16, 0, 0);
    }
  }

  // chunk c of row r of a tile sits at position c ^ (r mod CHUNKS); rows at or beyond `bound` are never read
  auto issue_rows = [&](const unsigned char* rows, unsigned char* buf, int tbase) {
    const unsigned char* tile_rows = rows + (size_t)tbase * ROWB;
    const int rel = bound - 1 - tbase;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int row = lane / CHUNKS + i * (kWave / CHUNKS), phys = lane % CHUNKS;
      const uint32_t off = (uint32_t)(min(row, rel) * ROWB + ((phys ^ (row & (CHUNKS - 1))) * 16));
      if constexpr (TWO)
        copy_to_lds<kStreamOnce>(rows, (size_t)bound * ROWB, buf + i * (kWave * 16), off, tbase * ROWB);
      else
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(tile_rows + off),
                                         (__attribute__((address_space(3))) void*)(buf + i * (kWave * 16)), 16, 0, kStreamOnce);
    }
  };
  // !ONE: the K rows of a tile are loaded in the layout of the score product's A operand (lane (l16, q): rows
  // l16 and 16 + l16 of the tile, chunk 4 ks + q of the row for k-step ks), one tile ahead, so a tile's K rows
  // pass through no LDS at all and a wavefront has a whole tile (K in registers, V on its way to the other LDS
  // buffer) in flight during all of the arithmetic on the current one.
  // (TWO: the second tile's K rows in kreg.)
  bf16x8_t kn[2][KS], kreg[2][KS];
  auto issue_k = [&](int tbase, bf16x8_t (&to)[2][KS]) {
    const unsigned char* tile_rows = kbytes + (size_t)tbase * ROWB;
    const int rel = bound - 1 - tbase;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const uint32_t off = (uint32_t)(min(16 * st + l16, rel) * ROWB + q * 16);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        to[st][ks] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t*>(tile_rows + off + ks * 64));
    }
  };
  int base = start + wave * kMTile;
  const int wave_lim = lim;
  constexpr int kTileStep = kMfmaWaves * kMTile;
  const bool has_tile = base < wave_lim;
  if constexpr (ONE) {
    if (has_tile) {
      issue_rows(kbytes, Kb, base);
      // slot base + lane of the tile (lanes beyond the tile repeat a slot)
      const uint32_t at = (uint32_t)min(min(lane, kMTile - 1), bound - 1 - base);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p.votes + ubase + base + at),
                                       (__attribute__((address_space(3))) void*)s_sc, 4, 0, 0);
      if constexpr (STEP)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p.log_s + ubase + base + at),
                                         (__attribute__((address_space(3))) void*)(s_sc + 256), 4, 0, 0);
      issue_rows(vbytes, Vb, base);
    }
  }
  // Otherwise the votes and EMA state of a tile are requested with its rows, into registers.
  int pv_next = 1;
  float ls_next = -INFINITY;
  auto request_scalars = [&](int tbase, int& pv, float& ls) {
    const uint32_t at = (uint32_t)min(row_mine, bound - 1 - tbase);
    pv = (p.votes + ubase + tbase)[at];
    if constexpr (STEP) ls = (p.log_s + ubase + tbase)[at];
  };
  if constexpr (LOOP) {
    if (has_tile) {
      issue_k(base, kn);
      issue_rows(vbytes, Vb, base);
      request_scalars(base, pv_next, ls_next);
    }
  }

  if constexpr (TWO) arrive();

  // B operand of the score product: column l16 is head l16 mod G, this lane's 8 channels of every k-step
  bf16x8_t qb[KS];
  auto read_q = [&]() {                          // ONE: from this wavefront's LDS copy, once it has landed
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qb[ks] = *reinterpret_cast<const bf16x8_t*>(s_q + g_l * ROWB + (((4 * ks + q) ^ ((4 * g_l) & (CHUNKS - 1))) * 16));
  };
  if constexpr (!ONE) {
    const unsigned char* qrow = reinterpret_cast<const unsigned char*>(p.q) + ((size_t)unit * G + g_l) * ROWB;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qb[ks] = *reinterpret_cast<const bf16x8_t*>(qrow + ks * 64 + q * 16);
  }

  // Tile loop, step mode: the updated EMA state (ln S, n) of a split is collected in LDS (the staging area the
  // single-tile variant uses for queries and scalars) and written out by the whole workgroup once all tiles
  // are done, when it fits: many small stores spread over the streaming phase slow the row stream down more
  // than their bytes account for, one burst per workgroup less so.
  unsigned char* const s_stage = smem_tiles + kMfmaWaves * 2 * TILE_BYTES;
  const bool staged = !ONE && STEP && (size_t)p.per * 4 <= (size_t)kMfmaWaves * mfma_stage_bytes(D, G);
  const float sl2 = p.scale * kLog2e;
  float m_run = kLowest, l_run = 0.f;
  f32x4_t O[NTILE];
#pragma unroll
  for (int nt = 0; nt < NTILE; ++nt) O[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  bool first = true;
  const int live_end = min(len_old, start + p.per);

  // One tile.  `extra`: the appended token alone (row 0 of the tile, copied from s_new).
  // `next`: the wavefront's next tile (or -1); its K rows are requested as soon as the score product has
  // consumed the K buffer, its V rows after the second product, so both travel during the arithmetic.
  // v_wait: the V rows have landed when at most that many requests are outstanding; negative: they have landed.
  // k_rows: the K operand (unless ONE).  lp_lane: log2(votes) of slot row_mine.  x_out: the group-mean logit of slot row_mine (of a `writer` lane), and the
  // return value whether this lane stores it.
  // The first wavefront requests the head's `arrivals` in its last tile, when that tile's rows have landed, to have the
  // word when the tile is done.
  uint64_t seen = 0;
  bool looked = !kMayShareXcd || wave != 0;   // uniform
  auto look = [&]() {
    if (!looked) seen = ld_arrivals(p, unit);
    looked = true;
  };
  auto compute = [&](int tbase, bool extra, int next, const bf16x8_t (&k_rows)[2][KS], float lp_lane, auto v_wait,
                     float& x_out, bool last) -> bool {
    constexpr int kVWait = decltype(v_wait)::value;
    const int n_live = extra ? 1 : max(0, min(kMTile, live_end - tbase));
    auto clear_masked_v = [&]() {
      if (n_live < kMTile) {                     // uniform: clear the V rows of masked slots (0 * garbage could be NaN)
        for (int c = n_live * CHUNKS + lane; c < kMTile * CHUNKS; c += kWave)
          *reinterpret_cast<uint4*>(Vb + c * 16) = make_uint4(0, 0, 0, 0);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    };
    if constexpr (kVWait < 0) clear_masked_v();
    if (LOOP && next >= 0) {
      // the next tile: K rows and scalars into registers, V rows into the other buffer (after the clearing
      // stores above: the compiler orders LDS stores behind outstanding copies into LDS)
      issue_k(next, kn);
      request_scalars(next, pv_next, ls_next);
      issue_rows(vbytes, Tb + (Vb == Tb ? TILE_BYTES : 0), next);
    }
    // ---- S^T = K Q^T
    f32x4_t s[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
    if constexpr (!ONE) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_rows[0][ks], qb[ks], s[0], 0, 0, 0);
        s[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_rows[1][ks], qb[ks], s[1], 0, 0, 0);
      }
    } else {
      // the K tile through reads that the compiler does not order behind the V rows' copies (see above).  The buffer is
      // aligned to its rows, so chunk (4 ks + q) ^ (l16 mod CHUNKS) is that of k-step 0 with 64 ks XORed into the address.
      i32x4_t a0[KS], a1[KS];
      uint32_t ad[KS];
      const uint32_t ad0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)Kb +
                           (uint32_t)(l16 * ROWB + ((q ^ (l16 & (CHUNKS - 1))) * 16));
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) ad[ks] = ad0 ^ (uint32_t)(ks * 64);
      if constexpr (KS == 4) {                   // D = 128: rows 16 .. 31 of the tile are 4096 bytes further
        static_assert(KS != 4 || 16 * ROWB == 4096, "offset in the statement below");
        asm volatile(
            "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:4096\n\t"
            "ds_read_b128 %2, %9\n\tds_read_b128 %3, %9 offset:4096\n\t"
            "ds_read_b128 %4, %10\n\tds_read_b128 %5, %10 offset:4096\n\t"
            "ds_read_b128 %6, %11\n\tds_read_b128 %7, %11 offset:4096\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(a0[0]), "=&v"(a1[0]), "=&v"(a0[1]), "=&v"(a1[1]), "=&v"(a0[2]), "=&v"(a1[2]), "=&v"(a0[3]), "=&v"(a1[3])
            : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3])
            : "memory");
      } else {                                   // D = 64: 2048 bytes further
        static_assert(KS == 4 || (KS == 2 && 16 * ROWB == 2048), "offset in the statement below");
        asm volatile(
            "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:2048\n\t"
            "ds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:2048\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(a0[0]), "=&v"(a1[0]), "=&v"(a0[1]), "=&v"(a1[1])
            : "v"(ad[0]), "v"(ad[1])
            : "memory");
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a0[ks]), qb[ks], s[0], 0, 0, 0);
        s[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a1[ks]), qb[ks], s[1], 0, 0, 0);
      }
    }
    // ---- this lane's NV values of the column
    float sv[NV];
    if constexpr (NV == 4) {
#pragma unroll
      for (int v = 0; v < 4; ++v) sv[v] = (r_l & 1) ? s[1][v] : s[0][v];
    } else if constexpr (NV == 2) {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const float t0 = (r_l & 1) ? s[0][2 + v] : s[0][v], t1 = (r_l & 1) ? s[1][2 + v] : s[1][v];
        sv[v] = (r_l & 2) ? t1 : t0;
      }
    } else {
      float t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] = (pos0 & 1) ? s[j >> 1][2 * (j & 1) + 1] : s[j >> 1][2 * (j & 1)];
      const float u0 = (pos0 & 2) ? t[1] : t[0], u1 = (pos0 & 2) ? t[3] : t[2];
      sv[0] = (pos0 & 4) ? u1 : u0;
    }
    // ---- logits (log2 domain, log2(votes) folded in), group-mean logit for the EMA
    float z[NV], xm[NV], lp[NV];
    if constexpr (NV == 1) lp[0] = lp_lane;
    else {                                       // slot row0 + v is loaded by lane v of the quad
      lp[0] = dpp_f32<0x00>(lp_lane);
      lp[1] = dpp_f32<0x55>(lp_lane);
      if constexpr (NV == 4) {
        lp[2] = dpp_f32<0xAA>(lp_lane);
        lp[3] = dpp_f32<0xFF>(lp_lane);
      }
    }
    float tm = -INFINITY;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const bool live = row0 + v < n_live && (G > 1 || r_l < 8);
      z[v] = live ? fmaf(sv[v], sl2, lp[v]) : -INFINITY;
      tm = fmaxf(tm, z[v]);
      xm[v] = head_sum<G>(sv[v]);
    }
    const float mn = fmaxf(m_run, over_head_lanes<G>(tm, [](float a, float b) { return fmaxf(a, b); }));
    const float c = fast_exp2(m_run - mn);       // (both finite or the tile holds an infinite logit)
    float pr[NV], ps = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      pr[v] = fast_exp2(z[v] - mn);
      ps += pr[v];
    }
    l_run = fmaf(l_run, c, ps);
    m_run = mn;
    if (!first && __any(c != 1.f)) {             // uniform: rescale the accumulators, row r = head r mod G
                                                 // (with ONE only the extra tile of the appended token gets here)
      const float c_other = dpp_f32<0x124>(c);   // G = 8: of the head four further (every lane reads: not inside the choice)
      const float cq = G < 8 || ((l16 >> 2) & 1) == (q & 1) ? c : c_other;
      const float ci[4] = {dpp_f32<0x00>(cq), dpp_f32<G == 1 ? 0x00 : 0x55>(cq), dpp_f32<G <= 2 ? 0x00 : 0xAA>(cq),
                           dpp_f32<G == 1 ? 0x00 : G == 2 ? 0x55 : 0xFF>(cq)};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int nt = 0; nt < NTILE; ++nt) O[nt][i] *= ci[i];
    }
    first = false;
    if constexpr (kVWait >= 0) {                 // before any store is issued
      // (tied to the softmax sum, so that the wait is not scheduled ahead of the arithmetic it is meant to hide)
      asm volatile("s_waitcnt vmcnt(%1)" : "+v"(l_run) : "n"(kVWait) : "memory");
      if (last) look();
      clear_masked_v();
    }
    // ---- O += P V with P = hi + lo in bf16.  The places of the slots that other lanes took hold the smallest normal
    // number and not zero: against any finite V it vanishes beside the head's largest weight (1), and an infinity in V
    // stays one, where zero would make it a NaN.
    constexpr uint32_t kNone = 0x00800080u;
    uint32_t ah[4], al[4];
    if constexpr (NV == 1) {
      const uint32_t hb = __builtin_bit_cast(uint32_t, pr[0]) & 0xFFFF0000u;
      const uint32_t lb = __builtin_bit_cast(uint32_t, pr[0] - __builtin_bit_cast(float, hb)) & 0xFFFF0000u;
      const uint32_t wh = (pos0 & 1) ? hb | (kNone & 0xFFFFu) : hb >> 16 | (kNone & 0xFFFF0000u);
      const uint32_t wl = (pos0 & 1) ? lb | (kNone & 0xFFFFu) : lb >> 16 | (kNone & 0xFFFF0000u);
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        ah[d] = (pos0 >> 1) == d && (G > 1 || r_l < 8) ? wh : kNone;
        al[d] = (pos0 >> 1) == d && (G > 1 || r_l < 8) ? wl : kNone;
      }
    } else {
      constexpr int NW = NV / 2;
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        const float p0 = pr[2 * j], p1 = pr[2 * j + 1];
        const float l0 = p0 - __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, p0) & 0xFFFF0000u);
        const float l1 = p1 - __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, p1) & 0xFFFF0000u);
        const uint32_t wh = pack_hi16(p0, p1), wl = pack_hi16(l0, l1);
#pragma unroll
        for (int d = j; d < 4; d += NW) {        // dword d holds the places 2 d, 2 d + 1
          ah[d] = r_l == d / NW ? wh : kNone;
          al[d] = r_l == d / NW ? wl : kNone;
        }
      }
    }
    const bf16x8_t a_hi = __builtin_bit_cast(bf16x8_t, make_uint4(ah[0], ah[1], ah[2], ah[3]));
    const bf16x8_t a_lo = __builtin_bit_cast(bf16x8_t, make_uint4(al[0], al[1], al[2], al[3]));
    // transpose read: lane s of a 16-lane block supplies the address of row s / 4, columns 4 (s mod 4) .. + 3, and
    // receives column s of the block's four rows (channel tile nt: chunk 2 nt + c, so 32 nt XORed into the address)
    // The V tile has landed (awaited above or at the top of the loop) while the next tile's K rows may be on
    // their way: the reads go through a statement the compiler does not order behind those copies.
    const int vrow = 4 * q + (l16 >> 2);
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
    u32x2_t b0[NTILE], b1[NTILE];
    uint32_t va[NTILE];
    const uint32_t va0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)Vb +
                         (uint32_t)(vrow * ROWB + ((((l16 & 3) >> 1) ^ (vrow & (CHUNKS - 1))) * 16) + (l16 & 1) * 8);
#pragma unroll
    for (int nt = 0; nt < NTILE; ++nt) va[nt] = va0 ^ (uint32_t)(nt * 32);
    if constexpr (NTILE == 8) {                  // D = 128: rows 16 .. 31 of the tile are 4096 bytes further
      static_assert(NTILE != 8 || 16 * ROWB == 4096, "offset in the statement below");
      asm volatile(
          "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:4096\n\t"
          "ds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:4096\n\t"
          "ds_read_b64_tr_b16 %4, %18\n\tds_read_b64_tr_b16 %5, %18 offset:4096\n\t"
          "ds_read_b64_tr_b16 %6, %19\n\tds_read_b64_tr_b16 %7, %19 offset:4096\n\t"
          "ds_read_b64_tr_b16 %8, %20\n\tds_read_b64_tr_b16 %9, %20 offset:4096\n\t"
          "ds_read_b64_tr_b16 %10, %21\n\tds_read_b64_tr_b16 %11, %21 offset:4096\n\t"
          "ds_read_b64_tr_b16 %12, %22\n\tds_read_b64_tr_b16 %13, %22 offset:4096\n\t"
          "ds_read_b64_tr_b16 %14, %23\n\tds_read_b64_tr_b16 %15, %23 offset:4096\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(b0[0]), "=&v"(b1[0]), "=&v"(b0[1]), "=&v"(b1[1]), "=&v"(b0[2]), "=&v"(b1[2]), "=&v"(b0[3]), "=&v"(b1[3]),
            "=&v"(b0[4]), "=&v"(b1[4]), "=&v"(b0[5]), "=&v"(b1[5]), "=&v"(b0[6]), "=&v"(b1[6]), "=&v"(b0[7]), "=&v"(b1[7])
          : "v"(va[0]), "v"(va[1]), "v"(va[2]), "v"(va[3]), "v"(va[4]), "v"(va[5]), "v"(va[6]), "v"(va[7])
          : "memory");
    } else {                                     // D = 64: 2048 bytes further
      static_assert(NTILE == 8 || (NTILE == 4 && 16 * ROWB == 2048), "offset in the statement below");
      asm volatile(
          "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:2048\n\t"
          "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:2048\n\t"
          "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:2048\n\t"
          "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:2048\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(b0[0]), "=&v"(b1[0]), "=&v"(b0[1]), "=&v"(b1[1]), "=&v"(b0[2]), "=&v"(b1[2]), "=&v"(b0[3]), "=&v"(b1[3])
          : "v"(va[0]), "v"(va[1]), "v"(va[2]), "v"(va[3])
          : "memory");
    }
#pragma unroll
    for (int part = 0; part < 2; ++part)         // (all of one part, then all of the other: no two in a row depend on each other)
#pragma unroll
      for (int nt = 0; nt < NTILE; ++nt) {
        const uint4 bw = make_uint4(b0[nt][0], b0[nt][1], b1[nt][0], b1[nt][1]);
        O[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part ? a_lo : a_hi, __builtin_bit_cast(bf16x8_t, bw), O[nt], 0, 0, 0);
      }
    // ---- group-mean logit of the slot that this lane updates
    float x = xm[0];
#pragma unroll
    for (int v = 1; v < NV; ++v) x = (g_l & (NV - 1)) == v ? xm[v] : x;
    x_out = x * (p.scale * (1.0f / G));
    return writer && row_mine < n_live;
  };
  // ln(alpha S + (1 - alpha) e^x)  (Eq. 8):  ln(e^hi + e^lo) = hi + ln(1 + e^(lo - hi)) with the hardware exp2 / log2
  // (absolute error ~1e-7)
  auto ema = [&](float ls_old, float x) {
    const float a = p.ln_alpha + ls_old, b = p.ln_1m_alpha + x;
    const float hi = fmaxf(a, b), lo = fminf(a, b);
    return (lo == -INFINITY) ? hi : hi + kLn2 * fast_log2(1.f + fast_exp2((lo - hi) * kLog2e));
  };

  // ONE: results per slot that are stored at the very end (a store here would be waited for, with its whole round trip
  // to memory, before this wavefront may deposit its sums)
  bool own_store = false;
  float own_x = 0.f, own_ema = 0.f;
  constexpr std::integral_constant<int, -1> kLanded{};
  constexpr std::integral_constant<int, 0> kAwaitAll{};
  auto publish = [&](int tbase, bool mine, float x, float ls_old) {   // the results per slot of one tile of several
    if (p.logits_out != nullptr && mine) p.logits_out[ubase + tbase + row_mine] = x;
    if constexpr (STEP) {
      const float r = ema(ls_old, x);
      if (mine) {
        if (staged) {
          // (a statement the compiler does not see as an LDS store: it would order one behind the next
          // tile's outstanding copies into LDS)
          const uint32_t sa = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)(
              s_stage + (size_t)(tbase - start + row_mine) * 4);
          asm volatile("ds_write_b32 %0, %1" : : "v"(sa), "v"(r) : "memory");
        } else {
          p.log_s[ubase + tbase + row_mine] = r;
        }
      }
    }
  };
  if constexpr (TWO) {
    // Requests complete in the order of issue: with the second tile's outstanding the first one has landed.  (The
    // scheduling barriers keep the two tiles' requests apart and ahead of the arithmetic.)
    constexpr std::integral_constant<int, 2 * KS + LOADS + (STEP ? 2 : 1)> kAwaitFirst{};
    const int second = base + kTileStep;
    if (second < wave_lim) {
      int pv2;
      float ls2 = -INFINITY, x, x2;
      issue_k(base, kn);
      request_scalars(base, pv_next, ls_next);
      issue_rows(vbytes, Tb, base);
      __builtin_amdgcn_sched_barrier(0);
      issue_k(second, kreg);
      request_scalars(second, pv2, ls2);
      issue_rows(vbytes, Tb + TILE_BYTES, second);
      __builtin_amdgcn_sched_barrier(0);
      const bool mine = compute(base, false, -1, kn, fast_log2((float)pv_next), kAwaitFirst, x, false);
      Vb = Tb + TILE_BYTES;
      const bool mine2 = compute(second, false, -1, kreg, fast_log2((float)pv2), kAwaitAll, x2, true);
      publish(base, mine, x, ls_next);
      publish(second, mine2, x2, ls2);
    } else if (has_tile) {
      float x;
      issue_k(base, kn);
      request_scalars(base, pv_next, ls_next);
      issue_rows(vbytes, Tb, base);
      const bool mine = compute(base, false, -1, kn, fast_log2((float)pv_next), kAwaitAll, x, true);
      publish(base, mine, x, ls_next);
    }
    base = lim;
  }
  while (!TWO && base < wave_lim) {              // a single pass with ONE
    if constexpr (ONE) {
      // all copies but the youngest LOADS (the V rows) have landed: query rows, K rows, votes and EMA state
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
      read_q();
      uint64_t sc;                               // votes and ln S of slot row_mine
      const uint32_t sa = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)(s_sc + row_mine * 4);
      asm volatile("ds_read2_b32 %0, %1 offset1:64\n\ts_waitcnt lgkmcnt(0)" : "=v"(sc) : "v"(sa) : "memory");
      const float lp_lane = fast_log2((float)(int32_t)(uint32_t)sc);
      own_store = compute(base, false, -1, kreg, lp_lane, kAwaitAll, own_x, true);
      if constexpr (STEP) own_ema = ema(__builtin_bit_cast(float, (uint32_t)(sc >> 32)), own_x);
      base = lim;
    } else {
      // the tile's K rows (registers), V rows (LDS) and scalars have landed; the K registers pass through the
      // statement so that no use of them is scheduled ahead of the wait
      if constexpr (KS == 4)
        asm volatile("s_waitcnt vmcnt(0)"
                     : "+v"(kn[0][0]), "+v"(kn[0][1]), "+v"(kn[0][2]), "+v"(kn[0][3]), "+v"(kn[1][0]), "+v"(kn[1][1]),
                       "+v"(kn[1][2]), "+v"(kn[1][3])
                     :
                     : "memory");
      else
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(kn[0][0]), "+v"(kn[0][1]), "+v"(kn[1][0]), "+v"(kn[1][1]) : : "memory");
#pragma unroll
      for (int st = 0; st < 2; ++st) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kreg[st][ks] = kn[st][ks];
      }
      const float lp_lane = fast_log2((float)pv_next);
      const float ls_old = ls_next;
      const int next = base + kTileStep;
      float x;
      const bool mine = compute(base, false, next < wave_lim ? next : -1, kreg, lp_lane, kLanded, x, next >= wave_lim);
      // After the second product: the compiler orders the V reads behind every outstanding memory operation,
      // and stores issued before them would be waited for.
      publish(base, mine, x, ls_old);
      Vb = Tb + (Vb == Tb ? TILE_BYTES : 0);
      base = next;
    }
  }
  KK_TS(1);
  const bool grow = STEP && len_old < p.capacity;
  const int len = grow ? len_old + 1 : len_old;
  float new_x = 0.f;
  if (takes_new) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the copy of the new token has landed
    if constexpr (ONE) read_q();                 // (a wavefront without a tile of its own has not read them yet)
    if (grow) {
      if constexpr (!ONE) {                      // the K operand of a tile whose row 0 is the new key, zero elsewhere
        Vb = Tb;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const uint4 x = *reinterpret_cast<const uint4*>(s_new + (4 * ks + q) * 16);
          const uint4 z4 = make_uint4(0, 0, 0, 0);
          kreg[0][ks] = __builtin_bit_cast(bf16x8_t, l16 == 0 ? x : z4);
          kreg[1][ks] = __builtin_bit_cast(bf16x8_t, z4);
        }
      }
      if (lane < 2 * CHUNKS) {                   // row 0 of the tile (its swizzle is the identity)
        const uint4 x = *reinterpret_cast<const uint4*>(s_new + lane * 16);
        if (ONE || lane >= CHUNKS) *reinterpret_cast<uint4*>((lane < CHUNKS ? Kb : Vb) + (lane % CHUNKS) * 16) = x;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      compute(0, true, -1, kreg, 0.f, kLanded, new_x, false);   // one vote: log2 = 0
    }
  }

  // ---- deposit this wavefront's state in its own tile buffers; the workgroup reduces kParts of them --------------------
  // Rows of the second product: row 4 q + i is head (4 q + i) mod G, lane share (4 q + i) / G.  The shares are added in
  // the lane (G <= 2), then over the lane halves and (G <= 4) the rows of 16 lanes; each exchange pairs two channel
  // tiles, so the lanes end up with different channel tiles and the LDS stores are wide.
  const float l_tot = over_head_lanes<G>(l_run, [](float a, float b) { return a + b; });
  constexpr int NH = G < 4 ? G : 4;              // heads per lane
  float o[NTILE][NH];
#pragma unroll
  for (int nt = 0; nt < NTILE; ++nt)
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      if constexpr (G == 1) o[nt][h] = (O[nt][0] + O[nt][1]) + (O[nt][2] + O[nt][3]);
      else if constexpr (G == 2) o[nt][h] = O[nt][h] + O[nt][h + 2];
      else o[nt][h] = O[nt][h];
    }
#pragma unroll
  for (int nt = 0; nt < NTILE / 2; ++nt)
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      swap_halves(o[nt][h], o[nt + NTILE / 2][h]);
      o[nt][h] += o[nt + NTILE / 2][h];
    }
  constexpr int NO = G <= 4 ? NTILE / 4 : NTILE / 2;   // channel tiles per lane
  if constexpr (G <= 4) {
#pragma unroll
    for (int nt = 0; nt < NO; ++nt)
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        swap_rows(o[nt][h], o[nt + NO][h]);
        o[nt][h] += o[nt + NO][h];
      }
  }
  constexpr int kPartStride = 2 * TILE_BYTES / (int)sizeof(float);     // floats between the wavefronts' deposits
  float* s_acc = reinterpret_cast<float*>(smem_tiles);                 // [kParts] x [D][G]
  float* s_ml = s_acc + G * D;                                         // [kParts] x ([G] maxima, [G] sums)
  {
    float* acc_mine = s_acc + wave * kPartStride;
    const int nt0 = (NTILE / 2) * (q >> 1) + (G <= 4 ? NO * (q & 1) : 0);
    const int h0 = G == 8 ? 4 * (q & 1) : 0;
#pragma unroll
    for (int nt = 0; nt < NO; ++nt) {
      float* at = acc_mine + (16 * (nt0 + nt) + l16) * G + h0;
      if constexpr (NH == 4) *reinterpret_cast<float4*>(at) = make_float4(o[nt][0], o[nt][1], o[nt][2], o[nt][3]);
      else if constexpr (NH == 2) *reinterpret_cast<float2*>(at) = make_float2(o[nt][0], o[nt][1]);
      else *at = o[nt][0];
    }
    if (q == 0 && l16 < G) {
      s_ml[wave * kPartStride + l16] = m_run;
      s_ml[wave * kPartStride + G + l16] = l_tot;
    }
  }
  if (threadIdx.x == 0) {
    look();                                      // (a wavefront without a tile)
    s_one_xcd = kMayShareXcd && all_on_this_xcd(p, unit, seen);
  }
  if constexpr (!ONE && STEP) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the staged EMA state is in LDS
  __syncthreads();
  KK_TS(2);
  if constexpr (ONE) {
    const size_t at = ubase + start + wave * kMTile + row_mine;
    if (p.logits_out != nullptr && own_store) p.logits_out[at] = own_x;
    if (STEP && own_store) p.log_s[at] = own_ema;
  }
  if constexpr (!ONE && STEP) {
    if (staged) {                                // the split's updated EMA state, slot by slot
      for (int j = threadIdx.x; j < live_end - start; j += kMfmaWaves * kWave) {
        // (write-through: measured faster at batch 128 than leaving megabytes of dirty lines to the caches)
        __hip_atomic_store(&p.log_s[ubase + start + j], *reinterpret_cast<const float*>(s_stage + (size_t)j * 4),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (takes_new && grow) {                       // the appended token joins the cache
    if (lane < 2 * CHUNKS) {
      unsigned char* dst = reinterpret_cast<unsigned char*>(lane < CHUNKS ? p.k : p.v) + (ubase + len_old) * ROWB;
      *reinterpret_cast<uint4*>(dst + (lane % CHUNKS) * 16) = *reinterpret_cast<const uint4*>(s_new + lane * 16);
    }
    if (lane == 0) {                             // (row 0 of its tile is this lane's)
      p.votes[ubase + len_old] = 1;
      p.born[ubase + len_old] = t_old;           // first observed in this step
      if (p.logits_out != nullptr) p.logits_out[ubase + len_old] = new_x;
      p.log_s[ubase + len_old] = ema(-INFINITY, new_x);
    }
  }
  combine_and_finish<T, D, G, kParts, STEP, kMfmaWaves, true, kSolo, kMayShareXcd>(p, s_ml, s_ml + G, s_acc, kPartStride, kPartStride, &s_last,
                                                              unit, split, grow, len, t_old,
                                                              __builtin_amdgcn_readfirstlane(s_one_xcd) != 0);
}

template <int D, int G, int WAVES, int... kMode>
bool allow_lds(int bytes, std::integer_sequence<int, kMode...>) {
  auto allow = [&](const void* kernel) {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
  };
  return ((allow((const void*)decode_mfma_kernel<D, G, true, kMode, WAVES>) &&
           allow((const void*)decode_mfma_kernel<D, G, false, kMode, WAVES>)) && ...);
}

template <typename T, int D, int G>
keepkv_status launch_decode(const DecodeParams& p, int units, bool step, bool valu, hipStream_t st) {
  // 8 lanes per slot (16 channels each at D = 128 bf16) halves the cross-lane reduction work; the
  // widest group keeps 16 lanes per slot so that its accumulators still fit two waves per SIMD.
  constexpr int RV = D * (int)sizeof(T) / 16;                       // 16-byte vectors per row
  constexpr int LPS = (G >= 8 && RV >= 16) ? RV / (RV >= 32 ? 2 : 1) : (RV >= 32 ? 16 : 8);
  constexpr int U = 4;
  // (x, then y, is dealt first: with 8 heads along x the splits of a head come to one XCD, see all_on_this_xcd)
  const dim3 grid = p.arrivals != nullptr ? dim3(8, p.nsplit, units / 8) : dim3(p.nsplit, units), block(kWavesPerBlock * kWave);
  if constexpr (sizeof(T) == 2) {
    if (!valu) {
      auto go = [&](auto waves_tag) -> keepkv_status {
        constexpr int WV = decltype(waves_tag)::value;
        constexpr size_t tiles = (size_t)WV * 2 * kMTile * D * 2 + (size_t)WV * mfma_stage_bytes(D, G);
        // 64 or 128 KB of tile buffers at D = 128, the per-wavefront staging of queries and scalars, plus the
        // kernel's static LDS: allow it explicitly (once per process, for all instances)
        static const bool allowed = allow_lds<D, G, WV>((int)tiles, std::make_integer_sequence<int, kModes>{});
        if (!allowed) return KEEPKV_ERR_DEVICE;
        const dim3 mblock(WV * kWave);
        auto launch = [&](auto step_tag, auto mode_tag) -> keepkv_status {
          decode_mfma_kernel<D, G, decltype(step_tag)::value, decltype(mode_tag)::value, WV><<<grid, mblock, tiles, st>>>(p);
          return KEEPKV_OK;
        };
        const int n_tiles = (p.per + WV * kMTile - 1) / (WV * kMTile);      // per wavefront, at most
        auto by_tiles = [&](auto step_tag) -> keepkv_status {
          const bool solo = p.nsplit == 1, xcd = p.arrivals != nullptr;
          if (n_tiles == 1 && solo) return launch(step_tag, std::integral_constant<int, kOneSolo>{});
          if (n_tiles == 1 && xcd) return launch(step_tag, std::integral_constant<int, kOneXcd>{});
          if (n_tiles == 1) return launch(step_tag, std::integral_constant<int, kOneMem>{});
          if (n_tiles == 2 && solo) return launch(step_tag, std::integral_constant<int, kTwoSolo>{});
          if (n_tiles == 2 && xcd) return launch(step_tag, std::integral_constant<int, kTwoXcd>{});
          if (n_tiles == 2) return launch(step_tag, std::integral_constant<int, kTwoMem>{});
          if (solo) return launch(step_tag, std::integral_constant<int, kLoopSolo>{});
          return launch(step_tag, std::integral_constant<int, kLoopMem>{});
        };
        return step ? by_tiles(std::true_type{}) : by_tiles(std::false_type{});
      };
      if (p.waves == 8) return go(std::integral_constant<int, 8>{});
      return go(std::integral_constant<int, 4>{});
    }
  }
  constexpr int parts = kWavesPerBlock * (kWave / (LPS < 16 ? 16 : LPS));
  constexpr size_t smem = (size_t)parts * G * (D + 2) * sizeof(float);
  if constexpr (smem > 64 * 1024) {
    static const bool allowed =
        hipFuncSetAttribute((const void*)decode_attn_kernel<T, D, G, LPS, U, true>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) == hipSuccess &&
        hipFuncSetAttribute((const void*)decode_attn_kernel<T, D, G, LPS, U, false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) == hipSuccess;
    if (!allowed) return KEEPKV_ERR_DEVICE;
  }
  if (step) decode_attn_kernel<T, D, G, LPS, U, true><<<grid, block, smem, st>>>(p);
  else decode_attn_kernel<T, D, G, LPS, U, false><<<grid, block, smem, st>>>(p);
  return KEEPKV_OK;
}

}  // namespace
static DecodePlan kept_plan(const keepkv_layout* L, int capacity, int force_per, int force_waves, bool charge);
namespace {

template <typename T, int D>
keepkv_status dispatch_g(const DecodeParams& p, int units, int G, bool step, bool valu, hipStream_t st) {
  switch (G) {
    case 1: return launch_decode<T, D, 1>(p, units, step, valu, st);
    case 2: return launch_decode<T, D, 2>(p, units, step, valu, st);
    case 4: return launch_decode<T, D, 4>(p, units, step, valu, st);
    default: return launch_decode<T, D, 8>(p, units, step, valu, st);
  }
}

keepkv_status run_decode(const keepkv_layout* layout, const keepkv_cache* cache, const void* q, const void* k_t,
                         const void* v_t, void* out, float* logits_out, float* lse_out, float alpha, int32_t* overflow,
                         bool step, void* workspace, size_t workspace_bytes, void* stream) {
  if (!layout_ok(layout) || !cache_ok(cache) || !q || !out) return KEEPKV_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(out) || !aligned16(cache->k) || !aligned16(cache->v)) return KEEPKV_ERR_INVALID_ARG;
  if (step && (!k_t || !v_t || !aligned16(k_t) || !aligned16(v_t) || !(alpha >= 0.f && alpha < 1.f)))
    return KEEPKV_ERR_INVALID_ARG;
  if (!layout_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  const int units = layout->batch * layout->n_kv_heads;
  if (units > kMaxUnits) return KEEPKV_ERR_UNSUPPORTED;
  const int fw = cache->plan_wavefronts, fp = cache->plan_slots_per_split;
  if (!(fw == 0 || fw == 4 || fw == 8 || fw == -1) || fp < 0 || (fp > 0 && fp < 64)) return KEEPKV_ERR_INVALID_ARG;
  DecodePlan pl = plan_decode(layout, cache->capacity, fp, fw);
  if (pl.nsplit > 1 && (!workspace || workspace_bytes < pl.bytes || !aligned16(workspace))) {
    pl = kept_plan(layout, cache->capacity, fp, fw, false);        // heads split for the charge on whole ones alone need no workspace whole
    if (pl.nsplit > 1) return KEEPKV_ERR_WORKSPACE;
  }

  DecodeParams p;
  p.q = q; p.k = cache->k; p.v = cache->v; p.votes = cache->votes; p.log_s = cache->log_s; p.born = cache->born; p.t_obs = cache->t_obs;
  p.len = cache->len; p.k_t = k_t; p.v_t = v_t; p.overflow = overflow;
  p.out = out; p.logits_out = logits_out; p.lse_out = lse_out;
  char* const ws = reinterpret_cast<char*>(workspace);
  p.partial = reinterpret_cast<float*>(ws + pl.partial_off);
  p.ticket = reinterpret_cast<int32_t*>(ws);
  p.arrivals = nullptr;
  p.ticket_xcd = nullptr;
  p.split_stride = layout->n_q_heads / layout->n_kv_heads * (layout->head_dim + 2);
  // Of two splits of two tiles (D 128) the second must not be much shorter than the first, or its workgroup looks in vain: 128 heads x 751 of 884
  // slots 14.2 us through memory, 14.7 within the XCD; x 868 15.08 and 15.09, of eight query heads 15.9 and 15.8.
  const int bound = cache->len_hint > 0 && cache->len_hint < cache->capacity ? cache->len_hint : cache->capacity;
  const bool second_short = step && fp == 0 && pl.nsplit == 2 && layout->head_dim == 128 && pl.per > pl.waves * kMTile &&
                            4 * (bound - pl.per) < 3 * pl.per;
  if (pl.xcd_bytes != 0 && (step ? pl.xcd_step && !second_short : pl.xcd_attn) && workspace_bytes >= pl.xcd_bytes) {   // (a smaller workspace has room for partial results without lines of their own)
    p.arrivals = reinterpret_cast<uint64_t*>(ws + kArrivalsOff);
    p.ticket_xcd = reinterpret_cast<int32_t*>(ws + kXcdTicketsOff);
    p.split_stride = xcd_split_stride(layout);
    p.partial = reinterpret_cast<float*>(align_up(reinterpret_cast<uintptr_t>(p.partial), kLine));
  }
  p.n_kv_heads = layout->n_kv_heads; p.capacity = cache->capacity; p.nsplit = pl.nsplit; p.per = pl.per; p.waves = pl.waves; p.scale = layout->scale;
  p.len_hint = cache->len_hint > 0 ? cache->len_hint : 0;
  p.ln_alpha = (step && alpha > 0.f) ? logf(alpha) : -INFINITY;
  p.ln_1m_alpha = step ? log1pf(-alpha) : 0.f;

  const int G = layout->n_q_heads / layout->n_kv_heads;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  keepkv_status rc;
  if (layout->dtype == KEEPKV_BF16) {
    if (layout->head_dim == 128) rc = dispatch_g<uint16_t, 128>(p, units, G, step, pl.valu, st);
    else rc = dispatch_g<uint16_t, 64>(p, units, G, step, pl.valu, st);
  } else {
    if (layout->head_dim == 128) rc = dispatch_g<float, 128>(p, units, G, step, false, st);
    else rc = dispatch_g<float, 64>(p, units, G, step, false, st);
  }
  if (rc != KEEPKV_OK) return rc;
  return launch_status();
}

// ---- scratch for the entry point that takes no workspace --------------------------------------------------
// One array per GPU, held by the code object until the process ends.  In host code `scratch` is only a handle:
// the device address comes from hipGetSymbolAddress, once per device with that device current, and that address
// is what kernels receive.
constexpr size_t kStaticPartialBytes = (size_t)4 << 20;
constexpr size_t kStaticScratchBytes = kWorkspaceHead + kStaticPartialBytes;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];     // per device, filled on the first call there
std::mutex g_scratch_mutex;

__global__ void clear_words_kernel(int32_t* w, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = 0;
}

keepkv_status static_scratch(void** out, hipStream_t st) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KEEPKV_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return KEEPKV_ERR_DEVICE;
    // The control words (split tickets) must be zero when a call starts.  Every launch leaves them zero, so
    // they are cleared once, ahead of the first launch on this device (a kernel: it may be captured).
    const int n = (int)(kWorkspaceHead / sizeof(int32_t));
    clear_words_kernel<<<(n + 255) / 256, 256, 0, st>>>(reinterpret_cast<int32_t*>(ptr), n);
    if (hipGetLastError() != hipSuccess) return KEEPKV_ERR_DEVICE;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return KEEPKV_OK;
}

}  // namespace

// Workgroups of the matrix-core kernel that a compute unit holds: by its LDS (tile buffers, staging, static part), and by
// the 16 wavefronts that its registers allow.
static int resident_per_cu(int waves, int head_dim, int group) {
  const int lds = waves * (2 * kMTile * head_dim * 2 + mfma_stage_bytes(head_dim, group)) + 1024;
  const int by_lds = 160 * 1024 / lds, by_regs = 16 / waves;
  const int n = by_lds < by_regs ? by_lds : by_regs;
  return n > 0 ? n : 1;
}

// Slots per split and workgroup size of the matrix-core kernel, from a cost model.  A round of n workgroups takes the
// longer of what one workgroup needs for its rows (a compute unit pulls 34 GB/s, shared by its workgroups; a wavefront
// 10.2 GB/s with all its tiles requested at once, 7.5 in the tile loop) and of what memory needs for all of them
// (5.8 TB/s, less when the last workgroups leave compute units empty); further rounds cost 1.7 us each, smaller workgroups
// 0.5 us, and splits have to be combined, four, eight or sixteen at a time and, beyond sixteen, once more for every output
// element that a thread has.  At most kMaxSplitWorkgroups workgroups share
// heads: more of them never paid, and it bounds the workspace.
// The constants are a fit to 2000 measured (shape, plan) pairs on MI355X: batch 1 .. 128, 116 .. 32768 slots, head dims 64
// and 128.  Over those 55 shapes the plan chosen is 0.4 % slower than the best one (2.6 % at most); the model before, which
// rounded a split up to whole workgroup iterations and knew one price for combining, was 3.5 % (36 % at most) off: 8 heads
// x 32768 slots 43.5 us with 16 splits against 30.1 with 32, 128 heads x 2000 (D 64) 23.8 with one against 16.4 with two, 8
// heads x 852 7.1 with four against 6.7 with seven.  Over 30 more shapes of one to eight heads and up to 2^20 slots: 0.8 %
// slower than the best plan (8.6 % at most; 3.6 % and 20 % with one price for combining: one head of 8 query heads x 3405 slots
// 12.0 us with 27 splits against 9.9 with 16, x 50000 32.3 with 112 against 29.4 with 63).
// Combining came to cost less than that fit says; a head that would not be split although its wavefronts have more
// than one and a half tiles each is charged 0.35 us for that.  It moves shapes of 76 to 168 heads from one split to two or three, in bands, because
// splits are whole tiles.  In 362 shapes from all of those bands (every fourth number of heads, 1 and 8 query heads per head) splitting
// measured 11 % faster than the whole heads, 19 % at best and 0.3 % slower at worst: 96 heads x 460 slots (D 64) 7.4 us whole and 6.8 in two splits,
// 124 x 796 12.2 and 9.8, 140 x 1006 (D 128) 25.1 and 20.2, 156 x 874 20.3 and 20.4.  (A lower price for the combination itself
// also takes four splits for eight, 10 to 20 % slower at 8 heads x 1000.)  charge false: without it.
constexpr int kMaxSplitWorkgroups = 512;
constexpr int kMinSplit = 64;
static void choose_split(const keepkv_layout* L, int capacity, bool charge, long& per, int& waves) {
  const double units = (double)L->batch * L->n_kv_heads;
  const int group = L->n_q_heads / L->n_kv_heads;
  const double slot_bytes = 4.0 * L->head_dim + 24.0;
  const long max_ns = (capacity + kMinSplit - 1) / kMinSplit;
  double best = 1e300;
  for (int wv = 4; wv <= 8; wv += 4) {
    const double res_max = 256.0 * resident_per_cu(wv, L->head_dim, group);
    for (long ns = 1; ns <= max_ns && (ns == 1 || units * (double)ns <= kMaxSplitWorkgroups); ++ns) {
      long cand = ((capacity + ns - 1) / ns + kMTile - 1) / kMTile * kMTile;
      if (cand < kMinSplit) cand = kMinSplit;
      const double n_split = (double)((capacity + cand - 1) / cand);
      const double wgs = units * n_split;
      const long tiles = cand / kMTile;
      const double busy = (double)(tiles < wv ? tiles : wv);                           // wavefronts with a tile
      const double streams = (tiles <= 2 * wv ? 10.2 : 7.5) * busy;                   // GB/s
      auto round_of = [&](double n) {                                                  // us
        if (n <= 0.0) return 0.0;
        const double per_cu = (double)(long)((n + 255.0) / 256.0);
        const double rate = 33.7 / per_cu < streams ? 33.7 / per_cu : streams;
        const double alone = (double)cand * slot_bytes / (rate * 1e3);
        const double together = n * (units * capacity / wgs) * slot_bytes / (5.8e6 * pow(n / (256.0 * per_cu), 0.38));
        return alone > together ? alone : together;
      };
      const double full = (double)(long)(wgs / res_max), rest = wgs - full * res_max;
      const double rounds = full + (rest > 0.0 ? 1.0 : 0.0);
      const double elements = (double)((group * L->head_dim + wv * kWave - 1) / (wv * kWave));   // per thread
      double t = full * round_of(res_max) + round_of(rest) + 1.7 * (rounds - 1.0) + (wv == 4 ? 0.46 : 0.0);
      if (n_split > 1.0)
        t += (n_split <= 4.0 ? 1.85 : n_split <= 8.0 ? 2.7 : 4.3 + 1.3 * elements * (double)(long)((n_split - 1.0) / 16.0)) + 0.011 * n_split;
      else if (charge && 2 * tiles > 3 * wv)
        t += 0.35;
      if (t < best) {
        best = t;
        per = cand;
        waves = wv;
      }
    }
  }
}

// The vector-ALU kernel (4 wavefronts): a wavefront streams at no more than ~6.5 GB/s when all its tiles are requested at
// once and ~4.4 GB/s when it loops, all resident workgroups (512) together at ~5.1 TB/s when the chip is full; every round
// costs ~3 us, the combination ~2.3 / ~3.4 us per round trip of device-scope loads.  kMaxSplitWorkgroupsValu only bounds the
// workspace: the model's own choices stay below it (at most 1539 workgroups share heads, 513 heads of three splits).
constexpr int kMaxSplitWorkgroupsValu = 2048;
static void choose_split_valu(const keepkv_layout* L, int capacity, long& per) {
  const double units = (double)L->batch * L->n_kv_heads;
  const bool bf16 = L->dtype == KEEPKV_BF16;
  const double slot_bytes = 2.0 * L->head_dim * (bf16 ? 2 : 4) + 24.0;
  const int rv = L->head_dim * (bf16 ? 2 : 4) / 16;
  const long granule = bf16 ? 128 : (rv >= 32 ? 64 : 128);      // slots per loop iteration of a workgroup
  const double res_max = 512.0;
  const long max_ns = (capacity + 63) / 64 < 1024 ? (capacity + 63) / 64 : 1024;
  double best = 1e300;
  for (long ns = 1; ns <= max_ns && (ns == 1 || units * (double)ns <= kMaxSplitWorkgroupsValu); ++ns) {
    const long cand = ((capacity + ns - 1) / ns + 63) / 64 * 64;
    const double n_split = (double)((capacity + cand - 1) / cand);
    const double wgs = units * n_split;
    const double resident = wgs < res_max ? wgs : res_max;
    const double rounds = (double)(long)((wgs + res_max - 1.0) / res_max);
    const double wg_rate = (cand <= granule ? 6.5 : 4.4) * kWavesPerBlock;            // GB/s
    double together = 5100.0 * pow(resident / res_max, 0.15);                         // GB/s, all resident workgroups
    if (resident > 256.0) together *= (resident / 256.0) / (double)(long)((resident + 255.0) / 256.0);
    if (together > wg_rate * resident) together = wg_rate * resident;
    const double streamed = (double)((cand + granule - 1) / granule * granule);       // whole iterations
    const double t_one = streamed * slot_bytes / (wg_rate * 1e3);                     // us, a workgroup alone
    const double t_all = units * capacity * slot_bytes / rounds / (together * 1e3);   // us, one round of them
    const double t_stream = rounds * (3.0 + (t_one > t_all ? t_one : t_all));
    const double t_trips = n_split <= 8.0 ? 2.3 : 3.4 * (double)(long)((n_split + 15.0) / 16.0);
    const double t_combine = n_split > 1.0 ? 1.0 + t_trips + 0.02 * n_split : 0.0;
    if (t_stream + t_combine < best) {
      best = t_stream + t_combine;
      per = cand;
    }
  }
}

static size_t decode_bytes(const keepkv_layout* L, long nsplit) {
  return kWorkspaceHead + align_up((size_t)L->batch * L->n_q_heads * nsplit * (L->head_dim + 2) * sizeof(float), 256);
}

// Partial results with cache lines of their own, for heads that are combined within an XCD.
static size_t decode_xcd_bytes(const keepkv_layout* L, long nsplit) {
  return kWorkspaceHead + kLine + align_up((size_t)L->batch * L->n_kv_heads * nsplit * xcd_split_stride(L) * sizeof(float), 256);
}

// The heads have to divide evenly among the XCDs, or some would idle; with 4 heads, say, half of them.
static bool heads_fit_xcds(const keepkv_layout* L) {
  const long units = (long)L->batch * L->n_kv_heads;
  return units % 8 == 0 && units <= kMaxXcdUnits;
}

// Where combining within an XCD pays.  Measured through memory / within the XCD, us: with one tile a wavefront always, or it makes no
// difference (250 shapes, 4 % on average): 8 heads x 852 slots in seven splits 6.5 / 6.2, 64 x 852 in four 10.0 / 9.6, 32 x 1497 in eight 9.9 / 9.4.
// With two tiles the tail is a smaller share of the step, and how soon a head's workgroups have all arrived matters more.  D 128: 64 x 1487
// in four splits, which fill the chip, 15.4 / 14.8, 128 x 828 in two 14.6 / 14.55, but 48 x 1084 in four 10.0 / 10.3, 32 x 3284 in eight 15.0 / 15.5.  D 64,
// half the bytes beside the same tail: 64 x 1384 in four 9.15 / 8.97, 96 x 684 in two 8.5 / 8.3, but 32 x 1084 in four 7.56 / 7.72, 32 x 2584 in eight
// 9.1 / 9.3.  Attention alone has no wavefront that ends later for an appended token, and there it pays up to eight splits: 1 to 3 % (16 heads x
// 2300 to 5000 slots of D 64 in eight 1.5 %, 64 x 1044 to 1734 in four 2.5 %, partly filled ones of D 128 3 %), but 8 heads in sixteen and 128 x 420 of 600 slots of D 128 in two 3 % slower.  In the tile loop
// reading `arrivals` cost as much as it gave.
static bool xcd_pays(const keepkv_layout* L, long nsplit, long per, int waves, bool step) {
  const long workgroups = (long)L->batch * L->n_kv_heads * nsplit;
  if (per <= (long)waves * kMTile) return true;
  if (!step) return nsplit <= 8 && (L->head_dim == 64 || nsplit > 2);
  if (nsplit > 4) return false;
  return workgroups >= (L->head_dim == 64 ? 192 : 256);
}

static DecodePlan make_plan(const keepkv_layout* L, int capacity, int force_per, int force_waves, bool charge) {
  DecodePlan pl;
  const bool valu = L->dtype == KEEPKV_BF16 && force_waves == -1;
  const bool mfma = L->dtype == KEEPKV_BF16 && !valu;
  long per = 128;
  int waves = kWavesPerBlock;
  if (mfma) choose_split(L, capacity, charge, per, waves);
  else choose_split_valu(L, capacity, per);
  if (mfma && (force_waves == 4 || force_waves == 8)) waves = force_waves;
  pl.waves = waves;
  pl.valu = valu;
  if (force_per >= 64) per = mfma ? force_per / 32 * 32 : force_per / 64 * 64;
  long ns = (capacity + per - 1) / per;
  if (ns > 1024) { ns = 1024; per = ((capacity + ns - 1) / ns + 63) / 64 * 64; ns = (capacity + per - 1) / per; }   // (max_ns caps it already)
  pl.nsplit = (int)ns;
  pl.per = (int)per;
  pl.partial_off = kWorkspaceHead;
  pl.bytes = decode_bytes(L, ns);
  const bool may_share = mfma && ns > 1 && ns <= kMaxLocalSplits && per <= 2L * waves * kMTile && heads_fit_xcds(L);
  pl.xcd_bytes = may_share ? decode_xcd_bytes(L, ns) : 0;
  pl.xcd_step = force_per > 0 || xcd_pays(L, ns, per, waves, true);    // (the caller's splits wherever they can)
  pl.xcd_attn = force_per > 0 || xcd_pays(L, ns, per, waves, false);
  return pl;
}

// A workspace for caches of up to `capacity` slots: a smaller cache may be split finer than the largest.
size_t decode_workspace_bytes(const keepkv_layout* L, int capacity) {
  size_t bytes = plan_decode(L, capacity).bytes;
  const long units = (long)L->batch * L->n_kv_heads;
  const long most = (L->dtype == KEEPKV_BF16 ? kMaxSplitWorkgroups : kMaxSplitWorkgroupsValu) / units;
  long ns = (capacity + kMinSplit - 1) / kMinSplit;
  if (ns > most) ns = most;
  if (ns > 1 && decode_bytes(L, ns) > bytes) bytes = decode_bytes(L, ns);
  if (ns > 1 && L->dtype == KEEPKV_BF16 && heads_fit_xcds(L) && decode_xcd_bytes(L, ns) > bytes) bytes = decode_xcd_bytes(L, ns);
  return bytes;
}

// The cost model walks up to 1024 candidate plans, microseconds of host time, and a program asks for the same
// few plans again and again (one per layer shape and step): each thread keeps its last ones.  A plan is a pure function
// of the fields compared here.
static DecodePlan kept_plan(const keepkv_layout* L, int capacity, int force_per, int force_waves, bool charge) {
  struct Entry {
    int32_t key[9];
    DecodePlan plan;
  };
  static thread_local Entry kept[8] = {};          // (a zero batch is no valid key)
  const int32_t key[9] = {L->batch, L->n_q_heads, L->n_kv_heads, L->head_dim, L->dtype, capacity, force_per, force_waves, charge};
  uint32_t h = 0;
  for (int32_t k : key) h = h * 31u + (uint32_t)k;
  Entry& e = kept[(h ^ (h >> 15)) & 7u];
  if (memcmp(e.key, key, sizeof key) != 0) {
    e.plan = make_plan(L, capacity, force_per, force_waves, charge);
    memcpy(e.key, key, sizeof key);
  }
  return e.plan;
}
DecodePlan plan_decode(const keepkv_layout* L, int capacity, int force_per, int force_waves) {
  return kept_plan(L, capacity, force_per, force_waves, true);
}

}  // namespace kk

extern "C" keepkv_status keepkv_decode_attn(const keepkv_layout* layout, const keepkv_cache* cache,
                                            const void* q, void* out, float* logits_out, float* lse_out,
                                            void* workspace, size_t workspace_bytes, void* stream) {
  return kk::run_decode(layout, cache, q, nullptr, nullptr, out, logits_out, lse_out, 0.f, nullptr, false, workspace,
                        workspace_bytes, stream);
}

extern "C" keepkv_status keepkv_decode_step(const keepkv_layout* layout, keepkv_cache* cache, const void* q,
                                            const void* k_t, const void* v_t, void* out, float* logits_out,
                                            float alpha, int32_t* overflow, void* workspace, size_t workspace_bytes,
                                            void* stream) {
  return kk::run_decode(layout, cache, q, k_t, v_t, out, logits_out, nullptr, alpha, overflow, true, workspace,
                        workspace_bytes, stream);
}

extern "C" keepkv_status keepkv_decode_step_static(const keepkv_layout* layout, keepkv_cache* cache, const void* q,
                                                   const void* k_t, const void* v_t, void* out, float* logits_out,
                                                   float alpha, int32_t* overflow, void* stream) {
  using namespace kk;
  // validate first (nothing is launched, not even the one-time clear, on bad arguments), then size
  if (!layout_ok(layout) || !cache_ok(cache) || !q || !out || !k_t || !v_t) return KEEPKV_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(out) || !aligned16(cache->k) || !aligned16(cache->v) || !aligned16(k_t) ||
      !aligned16(v_t) || !(alpha >= 0.f && alpha < 1.f))
    return KEEPKV_ERR_INVALID_ARG;
  if (!layout_supported(layout) || !units_supported(layout)) return KEEPKV_ERR_UNSUPPORTED;
  const int fw = cache->plan_wavefronts, fp = cache->plan_slots_per_split;
  if (!(fw == 0 || fw == 4 || fw == 8 || fw == -1) || fp < 0 || (fp > 0 && fp < 64)) return KEEPKV_ERR_INVALID_ARG;
  const DecodePlan pl = plan_decode(layout, cache->capacity, fp, fw);
  if (pl.nsplit > 1 && pl.bytes > kStaticScratchBytes) return KEEPKV_ERR_UNSUPPORTED;   // partials beyond the static array
  void* ptr = nullptr;
  const keepkv_status rc = static_scratch(&ptr, reinterpret_cast<hipStream_t>(stream));
  if (rc != KEEPKV_OK) return rc;
  return run_decode(layout, cache, q, k_t, v_t, out, logits_out, nullptr, alpha, overflow, true, ptr,
                    kStaticScratchBytes, stream);
}

#ifdef KEEPKV_TRACE
extern "C" int keepkv_trace_read(long long* host, int n) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(kk::kk_trace), sizeof(long long) * n);
}
#endif
