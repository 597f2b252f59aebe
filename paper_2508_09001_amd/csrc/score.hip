// Page criticality score, eq. (quest_score), per (sequence, KV head, page), in
// the fixed fp32 order described in roles.h (score_role).  Digests are stored
// per logical page, so a KV head's digests form one contiguous stream; a
// workgroup scores a block of consecutive pages, four per wavefront.
//
// With PER > 0 the last workgroup of each KV head to finish also makes the head's
// selection (select_role, threshold.h), for retro_select_pages on small tables
// (score_selects).  Scores are then written and read device-coherently, past the
// XCDs' L2s, and a workgroup counts itself out only after its score stores have
// completed, so that the last one reads them all.
#include <algorithm>

#include "threshold.h"

namespace retro {
namespace {

// Workgroup shape: eight wavefronts of four pages a pass, up to two passes whose
// digests are requested at once (32 KB in flight per workgroup, four workgroups
// per compute unit).  Bound by reading the digests: 67 MB (8 sequences of 32K
// tokens, 8 KV heads) in 17.3 us, 3.9 TB/s; 18.5 us with four passes in two
// workgroups, 17.8 with one.  With a group of 8 query heads, whose arithmetic took
// 19.0 us for 34 MB when every pass read the queries from LDS again, 13.1 us.
constexpr int kScoreThreads = 512;
constexpr int kScoreWaves = kScoreThreads / 64;
// A page of d 64 in bf16 is half as long: up to four passes (32 heads of 5386 pages
// 10.7 -> 9.6 us).
template <typename T, int D>
constexpr int score_iters = D * sizeof(T) <= 128 ? 4 : 2;
constexpr int kPassPages = kScoreWaves * 4;  // pages of a pass

// Workgroups per KV head and pages per workgroup: two workgroups for every
// compute unit while a pass each is left, at most `iters` passes a workgroup.  With
// the selection at the end, one for every compute unit where that is enough, of
// whole passes: 32 heads of 300 pages 8.7 us, 9.6 with two; 2 heads of 5900 pages
// 13.8, in workgroups of 47 pages 14.2, of 24 15.7.
void score_split(const Geometry& g, int iters, bool selects, int* nbh, int* ppb) {
  const int heads = g.hk * g.batch, cus = compute_units();
  const int n_min = (g.max_pages + iters * kPassPages - 1) / (iters * kPassPages);
  const int n_max = (g.max_pages + kPassPages - 1) / kPassPages;
  int n = std::min(n_max, std::max(n_min, 2 * cus / heads));
  if (selects && (int64_t)n_max * heads > cus && (int64_t)n_min * heads <= cus) n = n_min;
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
  int32_t* count;  // one counter per KV head, kSelCounterInts apart, zero between launches
};

template <typename T, int D, int PER>
__global__ void __launch_bounds__(kScoreThreads, PER ? 4 : 8) score_kernel(
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
  // (The first one always stays: pos0 >= 0.)
  const int pos0 = max(sload(seq_lens + b), 0);
  if (page0 * g.P > pos0) return;  // uniform
  // the step's token and the sequence's pages (after the digest loads are issued)
  auto tok_of = [&](int& np) {
    const int pos = seq_lens[b];
    StepToken<T> tk{-1, 0, nullptr, nullptr, nullptr, nullptr};
    int seq_len = pos;
    if (PER == 0 && g.token_pending) {  // (no step selects in its score launch)
      const int phys = token_phys(g, ta.pt, b, pos);
      if (phys >= 0) {
        seq_len = pos + 1;
        tk = make_step_token<T>(g, b, h, pos, phys, ta.k_new, ta.v_new, ta.kc, ta.vc);
      }
    }
    np = min((seq_len + g.P - 1) / g.P, g.max_pages);
    return tk;
  };
  float* srow = scores + bh * g.max_pages;
  score_role<T, D, score_iters<T, D>, false, 0, kScoreThreads>(
      g, page0, page_end, q + b * q_bstride + (int64_t)h * g.G * D, dg + bh * g.max_pages * 2 * D,
      dyn_lds, tok_of, [] {},
      [&](int page, float v) {
        if constexpr (PER > 0)
          __hip_atomic_store(srow + page, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          srow[page] = v;
      });
  if constexpr (PER > 0) {
    __shared__ int s_last;
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's score stores have completed
    __syncthreads();
    if (threadIdx.x == 0) {
      // workgroups of the head that score (the others have returned)
      const int active = min((int)gridDim.x, pos0 / (g.P * ppb) + 1);
      int32_t* n = sa.count + bh * kSelCounterInts;
      const bool last =
          __hip_atomic_fetch_add(n, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == active - 1;
      if (last) __hip_atomic_store(n, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last = last;
    }
    __syncthreads();
    if (s_last)
      select_role<PER, kScoreWaves, true>(
          sa.tk, (int)bh, [&](int& tok_lp) { return select_len(g, seq_lens, ta.pt, b, tok_lp); },
          *reinterpret_cast<ThrLds<PER, kScoreWaves>*>(dyn_lds), true, [](int, int, int, int) {});
  }
}

template <typename T, int D, int PER>
hipError_t score_t(const Geometry& g, const void* q, int64_t qbs, const retro_kv_cache& c,
                   const void* k_new, const void* v_new, float* scores, const SelectArgs& sa,
                   hipStream_t s) {
  int nbh, ppb;
  constexpr int IT = score_iters<T, D>;
  score_split(g, IT, PER > 0, &nbh, &ppb);
  if (ppb < 1 || ppb > IT * kPassPages || nbh < 1) return hipErrorInvalidValue;
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
                   hipStream_t s) {
  auto go = [&](auto per) {
    return score_t<T, D, decltype(per)::value>(g, q, qbs, c, k_new, v_new, scores, sa, s);
  };
  if (!sa.count) return go(std::integral_constant<int, 0>{});
  // (300 pages with two a thread: 8.4 us instead of 8.0)
  if (g.max_pages <= kScoreThreads) return go(std::integral_constant<int, 1>{});
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

// Up to here a call's host time, a launch fewer (15 heads of 1870 pages, separate
// calls of two layers 89 us a pass, 95 with it), is what the last workgroup's
// selection saves at about equal time on the GPU (128 heads of 250 pages 11.4 us
// both, 32 of 600 11.2 against 10.9 with a launch of its own, 16 of 2000 13.7
// against 13.1, 2 of 4100 12.2 against 12.4); past it the chain from a head's last
// score to its rows costs more (8 heads of 4090 pages 16.7 against 15.0, 33K pages
// 16.0 against 13.8, 131K 41 against 28).
bool score_selects(const Geometry& g) {
  const int64_t pages = (int64_t)g.batch * g.hk * g.max_pages;
  return pages <= (g.max_pages <= 3072 ? 1 << 15 : 1 << 14) && g.max_pages <= kScoreThreads * kSelectPer;
}

hipError_t launch_score(const Geometry& g, const void* q_cur, int64_t q_batch_stride,
                        const retro_kv_cache& c, const void* k_new, const void* v_new,
                        float* scores, hipStream_t s, int step, const retro_selection* sel,
                        int32_t* counters) {
  SelectArgs sa{};
  if (sel) {
    if (!counters || !score_selects(g) || g.token_pending) return hipErrorInvalidValue;
    sa.tk = TopkArgs{g, step, scores, c.page_table, c.last_loaded, sel->selected, sel->mask,
                     sel->num_selected, nullptr, 1, nullptr};
    sa.count = counters;
  }
  if (g.dtype == RETRO_BF16)
    return g.D == 128 ? score_d<bf16_t, 128>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, sa, s)
                      : score_d<bf16_t, 64>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, sa, s);
  return g.D == 128 ? score_d<float, 128>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, sa, s)
                    : score_d<float, 64>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, sa, s);
}

}  // namespace retro
