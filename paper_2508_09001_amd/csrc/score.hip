// Page criticality score, eq. (quest_score), per (sequence, KV head, page), in
// the fixed fp32 order described in roles.h (score_role).  Digests are stored
// per logical page, so a KV head's digests form one contiguous stream; a
// workgroup scores a block of consecutive pages, four per wavefront.
//
// With a selection epilogue (PER > 0) the kernel also runs PageSelect and
// UpdateAndBuildMask: the last workgroup of each KV head to finish runs the
// head's selection (select_role, threshold.h) and clears the head's counters for
// the next launch.  With many heads most selections run beside other heads'
// scores.  Scores are written and read with device-coherent (agent-scope)
// atomic stores and loads, which bypass the per-XCD L2s; a workgroup counts
// itself out only after its score stores have completed, so the last one reads
// them all without any L2 write-back or invalidation (fences at device scope
// would write back and invalidate whole L2s, once per workgroup).
#include <algorithm>

#include "threshold.h"

namespace retro {
namespace {

// Workgroup shape: eight wavefronts of four pages a pass, up to four passes
// whose digests are all requested at once (64 KB in flight per workgroup, two
// workgroups per compute unit).  Bound by reading the digests: 67 MB (8
// sequences of 32K tokens, 8 KV heads) in 18.5 us, 3.6 TB/s; with a group of 8
// query heads, whose arithmetic took 19.0 us for 34 MB when every pass read the
// queries from LDS again, 15.8 us.  The selection in the last workgroup of each
// head (PER > 0) adds 7 to 10 us, the chain from the head's last score to its
// rows, against 4 to 6 us in front of the attention: a step selects there, and
// here only for retro_select_pages and RETRO_FLAG_SELECT_IN_SCORES.
constexpr int kScoreThreads = 512;
constexpr int kScoreWaves = kScoreThreads / 64;
constexpr int kScoreIters = 4;
constexpr int kPassPages = kScoreWaves * 4;              // pages of a pass
constexpr int kMaxPpb = kPassPages * kScoreIters;        // most pages a workgroup scores

// Workgroups per KV head and pages per workgroup: two workgroups for every
// compute unit while a pass each is left, at most kMaxPpb pages a workgroup.
void score_split(const Geometry& g, int* nbh, int* ppb) {
  const int heads = g.hk * g.batch;
  const int n_min = (g.max_pages + kMaxPpb - 1) / kMaxPpb;
  const int n_max = (g.max_pages + kPassPages - 1) / kPassPages;
  const int n = std::min(n_max, std::max(n_min, 2 * compute_units() / heads));
  *ppb = (g.max_pages + n - 1) / n;
  *nbh = (g.max_pages + *ppb - 1) / *ppb;
}

struct TokenArgs {
  const void* k_new;
  const void* v_new;
  void* kc;
  void* vc;
  const int32_t* pt;
};

struct SelectArgs {
  TopkArgs tk;
  // per KV head: a head counter, then one counter per group of `group`
  // workgroups, each in a 128-byte line of its own (kSelCounterInts apart);
  // zero between launches
  int32_t* count;
  int group;
};

template <typename T, int D, int PER>
__global__ void __launch_bounds__(kScoreThreads) score_kernel(
    Geometry g, const T* __restrict__ q, int64_t q_bstride, T* __restrict__ dg,
    const int32_t* __restrict__ seq_lens, float* __restrict__ scores, TokenArgs ta, SelectArgs sa,
    int ppb) {
  // [2][G][D] fp32 queries while scoring; the selection's histograms after
  extern __shared__ __attribute__((aligned(16))) float dyn_lds[];
  static_assert(ScoreShape<T, D>::PPW == 4, "four pages per wavefront and pass");
  const int page0 = blockIdx.x * ppb, page_end = min(page0 + ppb, g.max_pages);
  const int b = blockIdx.z, h = blockIdx.y;
  const int64_t bh = (int64_t)b * g.hk + h;
  // A workgroup whose pages all lie past the sequence (the step's token
  // included) has nothing to score: with sequences of mixed lengths the grid,
  // sized for the longest, would otherwise load their stale digests.
  // `active` workgroups are left (the first one always).
  const int pos0 = max(sload(seq_lens + b), 0);
  const int active = min((int)gridDim.x, pos0 / (g.P * ppb) + 1);
  if ((int)blockIdx.x >= active) return;  // uniform
  // the step's token and the sequence's pages (after the digest loads are issued)
  int n_pages = 0, tok_lp = -1, live_len = 0;
  auto tok_of = [&](int& np) {
    const int pos = seq_lens[b];
    StepToken<T> tk{-1, 0, nullptr, nullptr, nullptr, nullptr};
    int seq_len = pos;
    if (g.token_pending) {
      const int phys = token_phys(g, ta.pt, b, pos);
      if (phys >= 0) {
        seq_len = pos + 1;
        tk = make_step_token<T>(g, b, h, pos, phys, ta.k_new, ta.v_new, ta.kc, ta.vc);
      }
    }
    np = n_pages = min((seq_len + g.P - 1) / g.P, g.max_pages);
    tok_lp = tk.lp;
    live_len = seq_len;
    return tk;
  };
  float* srow = scores + bh * g.max_pages;
  score_role<T, D, kScoreIters, false, 0, kScoreThreads>(
      g, page0, page_end, q + b * q_bstride + (int64_t)h * g.G * D, dg + bh * g.max_pages * 2 * D,
      dyn_lds, tok_of, [] {},
      // device-coherent store: a later reader of the same launch (the selection)
      // may run on another XCD
      [&](int page, float v) {
        __hip_atomic_store(srow + page, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      });
  if constexpr (PER > 0) {
    __shared__ int s_last;
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's score stores have completed
    __syncthreads();
    // Count out in two levels (a group of workgroups, then the head), so that
    // no counter takes more than max(group, number of groups) updates; with a
    // single group its counter is the head's.
    if (threadIdx.x == 0) {
      const int ngroups = (active + sa.group - 1) / sa.group;
      int32_t* head = sa.count + bh * (int64_t)kSelCounterInts * (1 + kSelMaxGroups);
      const int grp = blockIdx.x / sa.group;
      const int in_grp = min(sa.group, active - grp * sa.group);
      int32_t* gc = head + kSelCounterInts * (1 + grp);
      bool last = false;
      if (__hip_atomic_fetch_add(gc, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == in_grp - 1) {
        __hip_atomic_store(gc, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = ngroups == 1 ||
               __hip_atomic_fetch_add(head, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   ngroups - 1;
        if (last && ngroups > 1) __hip_atomic_store(head, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      s_last = last;
    }
    __syncthreads();
    if (s_last)
      select_role<PER, kScoreWaves>(sa.tk, (int)bh, live_len, tok_lp,
                                    *reinterpret_cast<ThrLds<PER, kScoreWaves>*>(dyn_lds), true,
                                    [](int, int, int, int) {});
  }
}

template <typename T, int D, int PER>
hipError_t score_t(const Geometry& g, const void* q, int64_t qbs, const retro_kv_cache& c,
                   const void* k_new, const void* v_new, float* scores, const SelectArgs& sa,
                   int nbh, int ppb, hipStream_t s) {
  if (ppb < 1 || ppb > kMaxPpb || nbh < 1 || PER * kScoreThreads < (sa.count ? g.max_pages : 0))
    return hipErrorInvalidValue;
  dim3 grid(nbh, g.hk, g.batch);
  size_t lds = sizeof(float) * 2 * g.G * D;  // the queries' q+ and q- halves
  if constexpr (PER > 0) lds = std::max(lds, sizeof(ThrLds<PER, kScoreWaves>));
  const TokenArgs ta{k_new, v_new, c.k_cache, c.v_cache, c.page_table};
  score_kernel<T, D, PER><<<grid, kScoreThreads, lds, s>>>(g, (const T*)q, qbs, (T*)c.digest,
                                                          c.seq_lens, scores, ta, sa, ppb);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t score_d(const Geometry& g, const void* q, int64_t qbs, const retro_kv_cache& c,
                   const void* k_new, const void* v_new, float* scores, const SelectArgs& sa,
                   int nbh, int ppb, hipStream_t s) {
  auto go = [&](auto per) {
    return score_t<T, D, decltype(per)::value>(g, q, qbs, c, k_new, v_new, scores, sa, nbh, ppb, s);
  };
  if (!sa.count) return go(std::integral_constant<int, 0>{});
  return with_select_per(g.max_pages, go);
}

}  // namespace

int compute_units() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] <= 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

bool score_selects(const Geometry& g) { return g.max_pages <= kScoreThreads * kSelectPer; }

hipError_t launch_score(const Geometry& g, int step, const void* q_cur, int64_t q_batch_stride,
                        const retro_kv_cache& c, const void* k_new, const void* v_new,
                        float* scores, const retro_selection* sel, int32_t* sel_phys,
                        int32_t* counters, hipStream_t s) {
  SelectArgs sa{};
  int nbh, ppb;
  score_split(g, &nbh, &ppb);
  if (sel && counters && score_selects(g)) {
    sa.tk = TopkArgs{g, step, scores, c.page_table, c.last_loaded, sel->selected, sel->mask,
                     sel->num_selected, sel_phys, 1, nullptr};
    sa.count = counters;
    // one counter per head up to 32 workgroups, else groups of at least 16
    sa.group = nbh <= 32 ? nbh : std::max(16, (nbh + kSelMaxGroups - 1) / kSelMaxGroups);
  }
  auto go = [&](auto t, auto d) {
    using T = typename decltype(t)::type;
    return score_d<T, decltype(d)::value>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, sa,
                                          nbh, ppb, s);
  };
  struct BF { using type = bf16_t; };
  struct F32 { using type = float; };
  using D128 = std::integral_constant<int, 128>;
  using D64 = std::integral_constant<int, 64>;
  if (g.dtype == RETRO_BF16) return g.D == 128 ? go(BF{}, D128{}) : go(BF{}, D64{});
  return g.D == 128 ? go(F32{}, D128{}) : go(F32{}, D64{});
}

}  // namespace retro
