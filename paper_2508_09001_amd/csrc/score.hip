// Page criticality score, eq. (quest_score), per (sequence, KV head, page), in
// the fixed fp32 order described in roles.h (score_role).  Digests are stored
// per logical page, so a KV head's digests form one contiguous stream; a
// workgroup scores a block of consecutive pages, four per wavefront.
#include <algorithm>

#include "roles.h"

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
constexpr int kScoreIters = 2;
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

template <typename T, int D>
__global__ void __launch_bounds__(kScoreThreads, 8) score_kernel(
    Geometry g, const T* __restrict__ q, int64_t q_bstride, T* __restrict__ dg,
    const int32_t* __restrict__ seq_lens, float* __restrict__ scores, TokenArgs ta, int ppb) {
  // [2][G][D] fp32 queries
  extern __shared__ __attribute__((aligned(16))) float dyn_lds[];
  static_assert(ScoreShape<T, D>::PPW == 4, "four pages per wavefront and pass");
  const int page0 = blockIdx.x * ppb, page_end = min(page0 + ppb, g.max_pages);
  const int b = blockIdx.z, h = blockIdx.y;
  const int64_t bh = (int64_t)b * g.hk + h;
  // A workgroup whose pages all lie past the sequence (the step's token
  // included) has nothing to score: with sequences of mixed lengths the grid,
  // sized for the longest, would otherwise load their stale digests.
  if (page0 * g.P > sload(seq_lens + b)) return;  // uniform
  // the step's token and the sequence's pages (after the digest loads are issued)
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
    np = min((seq_len + g.P - 1) / g.P, g.max_pages);
    return tk;
  };
  float* srow = scores + bh * g.max_pages;
  score_role<T, D, kScoreIters, false, 0, kScoreThreads>(
      g, page0, page_end, q + b * q_bstride + (int64_t)h * g.G * D, dg + bh * g.max_pages * 2 * D,
      dyn_lds, tok_of, [] {},
      [&](int page, float v) { srow[page] = v; });
}

template <typename T, int D>
hipError_t score_t(const Geometry& g, const void* q, int64_t qbs, const retro_kv_cache& c,
                   const void* k_new, const void* v_new, float* scores, hipStream_t s) {
  int nbh, ppb;
  score_split(g, &nbh, &ppb);
  if (ppb < 1 || ppb > kMaxPpb || nbh < 1) return hipErrorInvalidValue;
  dim3 grid(nbh, g.hk, g.batch);
  const size_t lds = sizeof(float) * 2 * g.G * D;  // the queries' q+ and q- halves
  const TokenArgs ta{k_new, v_new, c.k_cache, c.v_cache, c.page_table};
  score_kernel<T, D><<<grid, kScoreThreads, lds, s>>>(g, (const T*)q, qbs, (T*)c.digest,
                                                     c.seq_lens, scores, ta, ppb);
  return hipGetLastError();
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

hipError_t launch_score(const Geometry& g, const void* q_cur, int64_t q_batch_stride,
                        const retro_kv_cache& c, const void* k_new, const void* v_new,
                        float* scores, hipStream_t s) {
  if (g.dtype == RETRO_BF16)
    return g.D == 128 ? score_t<bf16_t, 128>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, s)
                      : score_t<bf16_t, 64>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, s);
  return g.D == 128 ? score_t<float, 128>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, s)
                    : score_t<float, 64>(g, q_cur, q_batch_stride, c, k_new, v_new, scores, s);
}

}  // namespace retro
