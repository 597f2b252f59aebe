// One attention pass over the selected pages for the W+1 queries of the
// retrospective window (Alg. 1 "Attention"; eq. update-org for the current
// query, eq. update-sup for the past ones, masked as in the "Retrospective Mask"
// paragraph: row tau uses page p iff tau == t or M_p < tau).
//
// Work decomposition.  A workgroup owns one (sequence, KV head, split), a split
// being a run of consecutive entries of the selected-page list, processed as
// 32-token chunks (two 16-token tiles: two pages of 16, or one page of 32).
// Every chunk's keys and values are read from HBM once, staged in LDS, and used
// by all R = (W+1)*G rows of the KV head's group (row = window step r times G
// plus query head), so the gather is shared by the whole window and group.
// Rows are split into 16-row tiles; each wavefront owns RTW row tiles.
//
// Per chunk and row tile, on MFMA (gfx950):
//   S^T (16 tokens x 16 rows) = K (16 x d) . Q^T (d x 16), per 16-token tile
//       bf16: v_mfma_f32_16x16x32_bf16, d/32 steps;  f32: 16x16x4, d/4 steps
//   masking, online softmax in registers (exp2 domain, running max per row)
//   O^T (16 d x 16 rows) += V^T (16 d x 32 tokens) . P^T (32 tokens x 16 rows)
//       bf16: P is split into bf16 hi + lo parts (two MFMAs) so that rounding P
//             to bf16 does not cost accuracy; f32: 16x16x4.
// The S^T accumulator layout (lane l: row l%16, tokens 4*(l/16)..+3) is exactly
// the B operand layout of the PV product once the 32 chunk tokens are ordered
// as [tile 0: 4g..4g+3, tile 1: 4g..4g+3] for lane group g; V^T is read from LDS
// in the same token order, so no data moves between lanes.  The running max is
// per row, i.e. per lane column, and the O^T accumulator keeps the row in the
// lane column too, so rescaling needs no shuffles.
//
// Values live d-major in the cache (v_cache[page][h][d][P]), which is what makes
// the PV operand a contiguous LDS read.
//
// Output: per split and row, the normalised partial output and its natural-log
// normaliser, combined across splits by the merge kernel.
#include "threshold.h"

namespace retro {
namespace {

// Workgroups have eight wavefronts (the host checks); staging registers are
// sized for that: a chunk's 16-byte pieces spread over 512 threads.
constexpr int kAttendThreads = 512;

template <typename T, int D, int RTW>
__global__ void __launch_bounds__(kAttendThreads) attend_kernel(AttendArgs a) {
  using TL = Tiles<T, D>;
  constexpr int MAXP = (TL::PIECES + kAttendThreads - 1) / kAttendThreads;
  __shared__ __attribute__((aligned(16))) T lds[2 * TL::BUF_ELEMS];
  __shared__ int s_phys[kMaxSplitPages];
  __shared__ int s_page[kMaxSplitPages];
  __shared__ int s_mask[kMaxSplitPages];
  __shared__ int s_tok;
  const Geometry& g = a.g;
  // Work units are ordered (sequence, KV head, row group, split), split fastest,
  // and spread so that the units of one KV head share an XCD (workgroups go to
  // the 8 XCDs round-robin): its partial outputs then stay in that XCD's L2 for
  // the combine.
  int u = xcd_remap(blockIdx.x, gridDim.x);
  const int split = u % g.n_splits;
  u /= g.n_splits;
  const int rg = u % g.n_rgroups;
  u /= g.n_rgroups;
  const int h = u % g.hk, b = u / g.hk;
  attend_role<T, D, RTW, MAXP, RTW == 1, false>(
      a, b, h, rg, split, [&] { return live_seq_len(g, a.seq_lens, a.pt, b); }, lds, s_phys,
      s_page, s_mask, &s_tok, -1, [] {}, SelectionRows{});
}

template <typename T, int D, int RTW>
hipError_t attend_t(const AttendArgs& a, hipStream_t s) {
  const Geometry& g = a.g;
  const int64_t n = (int64_t)g.n_splits * g.n_rgroups * g.hk * g.batch;
  if (64 * g.waves != kAttendThreads) return hipErrorInvalidValue;
  attend_kernel<T, D, RTW><<<(unsigned)n, kAttendThreads, 0, s>>>(a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t attend_d(const AttendArgs& a, hipStream_t s) {
  return a.g.rtw == 1 ? attend_t<T, D, 1>(a, s) : attend_t<T, D, 2>(a, s);
}

// Attention with the page selection in front: every workgroup of a KV head makes
// the head's selection (the same computation on the same scores, so the same
// result) and takes its split's slots of it from LDS, instead of waiting for
// a selection launch and reading the rows back.  The workgroup of the last
// split, row group 0 writes the selection rows, the count and the token's page
// (TopkArgs::tok_out); last_loaded is left alone here (other workgroups of the
// head read it) and updated by the combine launch from those outputs.  The
// selection's histograms share LDS with the chunk staging, which is only used
// after the page list is in place.
template <typename T, int D, int RTW, int PER>
__global__ void __launch_bounds__(kAttendThreads) attend_select_kernel(AttendArgs a, TopkArgs ta) {
  using TL = Tiles<T, D>;
  constexpr int MAXP = (TL::PIECES + kAttendThreads - 1) / kAttendThreads;
  constexpr int kStageBytes = 2 * TL::BUF_ELEMS * (int)sizeof(T);
  using Thr = ThrLds<PER, kAttendThreads / 64>;
  __shared__ __attribute__((aligned(16))) char lds[std::max(kStageBytes, (int)sizeof(Thr))];
  __shared__ int s_phys[kMaxSplitPages];
  __shared__ int s_page[kMaxSplitPages];
  __shared__ int s_mask[kMaxSplitPages];
  __shared__ int l_lp[kMaxSplitPages], l_m[kMaxSplitPages], l_ph[kMaxSplitPages];
  __shared__ int s_tok;
  const Geometry& g = a.g;
  int u = xcd_remap(blockIdx.x, gridDim.x);
  const int split = u % g.n_splits;
  u /= g.n_splits;
  const int rg = u % g.n_rgroups;
  u /= g.n_rgroups;
  const int h = u % g.hk, b = u / g.hk;
  const bool writer = split == g.n_splits - 1 && rg == 0;
  const int first = split * g.pages_per_split;
  int seq_len = 0, k = 0;
  auto select = [&] {
    k = select_role(ta, b * g.hk + h,
                    [&](int& tok_lp) {
                      return seq_len = select_len(g, a.seq_lens, a.pt, b, tok_lp);
                    },
                    *reinterpret_cast<Thr*>(lds), writer,
                    [&](int q, int p, int m, int ph) {
                      if (q >= first && q < first + g.pages_per_split) {
                        l_lp[q - first] = p;
                        l_m[q - first] = m;
                        l_ph[q - first] = ph;
                      }
                    });
    __syncthreads();  // the split's page list is in LDS
  };
  attend_role<T, D, RTW, MAXP, RTW == 1, false>(
      a, b, h, rg, split, [&] { return seq_len; }, reinterpret_cast<T*>(lds), s_phys, s_page,
      s_mask, &s_tok, -1, select, [&](int t, int& lp, int& m, int& phys) {
        if (t < min(g.pages_per_split, k - first)) {
          lp = l_lp[t];
          m = l_m[t];
          phys = l_ph[t];
        }
        return k;
      });
}

template <typename T, int D>
hipError_t attend_select_d(const AttendArgs& a, const TopkArgs& ta, hipStream_t s) {
  const Geometry& g = a.g;
  const int64_t n = (int64_t)g.n_splits * g.n_rgroups * g.hk * g.batch;
  if (64 * g.waves != kAttendThreads) return hipErrorInvalidValue;
  return with_select_per(g.max_pages, [&](auto per) {
    constexpr int PER = decltype(per)::value;
    if (g.rtw == 1)
      attend_select_kernel<T, D, 1, PER><<<(unsigned)n, kAttendThreads, 0, s>>>(a, ta);
    else
      attend_select_kernel<T, D, 2, PER><<<(unsigned)n, kAttendThreads, 0, s>>>(a, ta);
    return hipGetLastError();
  });
}

}  // namespace

int attend_min_waves(int dtype, int D) {
  const int pieces = dtype == RETRO_BF16 ? (D == 128 ? Tiles<bf16_t, 128>::PIECES : Tiles<bf16_t, 64>::PIECES)
                                         : (D == 128 ? Tiles<float, 128>::PIECES : Tiles<float, 64>::PIECES);
  return (pieces + 64 * kMaxPieces - 1) / (64 * kMaxPieces);
}

AttendArgs make_attend_args(const Geometry& g, int step, const void* q_window,
                            const retro_kv_cache& c, const retro_selection& sel,
                            const int32_t* sel_phys, float* o_ws, float* l_ws, const void* dummy) {
  AttendArgs a;
  a.g = g;
  a.step = step;
  a.scale_log2 = g.sm_scale * kLog2e;
  a.q = q_window;
  a.kc = c.k_cache;
  a.vc = c.v_cache;
  a.pt = c.page_table;
  a.seq_lens = c.seq_lens;
  a.sel = sel.selected;
  a.msk = sel.mask;
  a.nsel = sel.num_selected;
  a.sel_phys = sel_phys;
  a.o_ws = o_ws;
  a.l_ws = l_ws;
  a.dummy = dummy;
  a.tok_k = nullptr;
  a.tok_v = nullptr;
  return a;
}

hipError_t launch_attend(const Geometry& g, int step, const void* q_window,
                         const retro_kv_cache& c, const retro_selection& sel,
                         const int32_t* sel_phys, float* o_ws, float* l_ws, const void* dummy,
                         hipStream_t s) {
  if (!dummy) return hipErrorInvalidValue;
  const AttendArgs a = make_attend_args(g, step, q_window, c, sel, sel_phys, o_ws, l_ws, dummy);
  if (g.stream) return launch_stream_attend(a, nullptr, s);
  if (g.dtype == RETRO_BF16) return g.D == 128 ? attend_d<bf16_t, 128>(a, s) : attend_d<bf16_t, 64>(a, s);
  return g.D == 128 ? attend_d<float, 128>(a, s) : attend_d<float, 64>(a, s);
}

bool attend_selects(const Geometry& g) { return g.max_pages <= kSelectPer * kAttendThreads; }

hipError_t launch_attend_select(const Geometry& g, int step, const void* q_window,
                                const retro_kv_cache& c, const retro_selection& sel,
                                const float* scores, float* o_ws, float* l_ws, int32_t* tok_out,
                                const void* dummy, hipStream_t s) {
  if (!attend_selects(g) || !tok_out || !dummy) return hipErrorInvalidValue;
  AttendArgs a = make_attend_args(g, step, q_window, c, sel, nullptr, o_ws, l_ws, dummy);
  a.sel_phys = tok_out;  // non-null: the page list carries physical pages (never read here)
  const TopkArgs ta{g, step, scores, c.page_table, c.last_loaded, sel.selected, sel.mask,
                    sel.num_selected, nullptr, 0, tok_out};
  if (g.stream) return launch_stream_attend(a, &ta, s);
  if (g.dtype == RETRO_BF16)
    return g.D == 128 ? attend_select_d<bf16_t, 128>(a, ta, s) : attend_select_d<bf16_t, 64>(a, ta, s);
  return g.D == 128 ? attend_select_d<float, 128>(a, ta, s) : attend_select_d<float, 64>(a, ta, s);
}

}  // namespace retro
