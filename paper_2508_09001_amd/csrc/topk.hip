// PageSelect + UpdateAndBuildMask (Alg. 1, Alg. 2) as a launch of its own, one
// workgroup per (sequence, KV head): for retro_select_pages, for tables longer
// than the attention launch's own selection takes and for
// RETRO_FLAG_SELECT_IN_SCORES.  The selection is select_role (threshold.h).
#include "threshold.h"

namespace retro {
namespace {

template <int THREADS, int PER>
__global__ void __launch_bounds__(THREADS) topk_mask_kernel(TopkArgs ta,
                                                            const int32_t* __restrict__ seq_lens) {
  __shared__ __attribute__((aligned(16))) ThrLds<PER, THREADS / 64> L;
  const int bh = blockIdx.x;
  // a pending token (Geometry::token_pending) gets Alg. 2's current-page rule here
  select_role<PER, THREADS / 64>(
      ta, bh,
      [&](int& tok_lp) { return select_len(ta.g, seq_lens, ta.pt, bh / ta.g.hk, tok_lp); }, L, true,
      [](int, int, int, int) {});
}

// Alg. 2 on the kept selection of a top-k reuse step: one wavefront per
// (sequence, KV head); every mask value is read before any last_loaded entry
// of the head changes (the rows hold distinct pages).
__global__ void __launch_bounds__(64) reuse_mask_kernel(Geometry g, int step,
                                                        const int32_t* __restrict__ sel,
                                                        int32_t* __restrict__ msk,
                                                        const int32_t* __restrict__ nsel,
                                                        int32_t* __restrict__ A) {
  const int bh = blockIdx.x;
  const int k = min(max(nsel[bh], 0), g.k_max);
  const int32_t* row = sel + (int64_t)bh * g.k_max;
  int32_t* m = msk + (int64_t)bh * g.k_max;
  int32_t* a = A + (int64_t)bh * g.max_pages;
  for (int i = threadIdx.x; i < g.k_max; i += 64) {
    const int p = i < k ? row[i] : -1;
    m[i] = (p >= 0 && p < g.max_pages) ? a[p] : -1;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < k; i += 64) {
    const int p = row[i];
    if (p >= 0 && p < g.max_pages) a[p] = step;
  }
}

}  // namespace

bool reuse_step(const Geometry& g, int step) { return g.reuse >= 2 && step % g.reuse != 0; }

hipError_t launch_reuse_mask(const Geometry& g, int step, const retro_kv_cache& c,
                             const retro_selection& sel, hipStream_t s) {
  reuse_mask_kernel<<<(unsigned)(g.batch * g.hk), 64, 0, s>>>(g, step, sel.selected, sel.mask,
                                                             sel.num_selected, c.last_loaded);
  return hipGetLastError();
}

hipError_t launch_topk_mask(const Geometry& g, int step, const float* scores,
                            const retro_kv_cache& c, const retro_selection& sel,
                            int32_t* sel_phys, hipStream_t s) {
  TopkArgs ta{g, step, scores, c.page_table, c.last_loaded, sel.selected, sel.mask,
              sel.num_selected, sel_phys, 1, nullptr};
  const unsigned grid = (unsigned)(g.batch * g.hk);
  // one workgroup per head; select_pages at 4 sequences of 4096 pages takes 26.4
  // us with eight wavefronts of nine pages a thread (28.6 with the selection in
  // the score launch's last workgroup of each head, 42.7 when that one searched
  // by 11-bit digits and one scanning wavefront); at 5900 pages eight wavefronts
  // of twelve take 23.1 us, sixteen of six 22.0
  if (g.max_pages <= 512)
    topk_mask_kernel<512, 1><<<grid, 512, 0, s>>>(ta, c.seq_lens);
  else if (g.max_pages <= 512 * 9)
    with_select_per(g.max_pages, [&](auto per) {
      topk_mask_kernel<512, decltype(per)::value><<<grid, 512, 0, s>>>(ta, c.seq_lens);
    });
  else if (g.max_pages <= 1024 * 6)
    topk_mask_kernel<1024, 6><<<grid, 1024, 0, s>>>(ta, c.seq_lens);
  else
    topk_mask_kernel<1024, 16><<<grid, 1024, 0, s>>>(ta, c.seq_lens);
  return hipGetLastError();
}

}  // namespace retro
