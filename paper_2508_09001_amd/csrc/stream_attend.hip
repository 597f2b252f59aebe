// Attention of the multi-launch plans for bf16 layers: the selected pages of one
// (sequence, KV head, split) streamed through the matrix cores by wavefronts
// that never wait for each other.
//
// Same products as attend_role (attend.hip): S^T = K Q^T per 16-token tile,
// masking and online softmax in registers, O^T += V^T P^T with P split into
// bf16 hi + lo.  What differs is who does what:
//
//   - A workgroup's eight wavefronts are NR side by side over its row tiles (RT
//     each) and NT = 8 / NR over the split's 32-token chunks (wt, wt + NT, ...).
//     No barrier in the loop: a wavefront reads its chunk's values straight into
//     MFMA operand registers, and its keys by whole rows through a piece of LDS
//     of its own (read in operand order, four consecutive lanes of a load would
//     touch four rows, four times the address work: 133 -> 118 us for 537 MB).
//     A layout with one row tile per wavefront, sharing each chunk through LDS
//     between barriers (attend_role), took 3.5 us per two chunks.
//   - Row i of S tile t is token 8 (i / 4) + 4 t + i % 4 of the chunk, so that
//     lane group g ends up with the chunk's tokens 8g .. 8g+7 of its row: the
//     PV product's operand in order, and V^T is read 16 bytes per lane.
//   - The keys of the next chunk are requested once this chunk's are in LDS, the
//     values once PV is done.
//   - With PER > 0 every workgroup makes the head's selection itself in front
//     (select_role, 4 to 6 us, the same result in each).
//   - At the end the NW states of a row are merged through LDS, tile by tile.
//
// Measured per launch, without the selection, attend_role's before: batch 16, 64
// pages and 36 rows per KV head (67 MB) 28 -> 22 us; batch 8, 307 pages, 32 rows
// (161 MB) 98 -> 38 us; 131K tokens dense, 68 rows (537 MB) 242 -> 110 us: bound
// by HBM, 4.9 TB/s.  Batch 4, 256 pages, 264 rows (67 MB) 75 -> 46 us; 131K tokens,
// 256 pages of 32, 260 rows (34 MB) 45 -> 25 us: bound by vector instructions (38 %
// of the cycles the matrix cores are busy, 54 % the vector units).  (The pairs of
// figures at single choices, here and below, were taken when each was made.)
#include <algorithm>

#include "threshold.h"

namespace retro {
namespace {

constexpr int kListPages = 1024;  // pages of a split (list in LDS)

constexpr int NW = 8;               // wavefronts of a workgroup

// two floats rounded to bf16 (nearest even): a low, b high
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  uint32_t w = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
  asm("" : "+v"(w));  // one conversion for the pair: its halves are taken from w
  return w;
}

// RT: row tiles per wavefront; NR: wavefronts side by side over the row tiles of
// the workgroup's row group, NW / NR over the chunks.
template <int D, int RT, int NR, int PER>
struct StreamLds {
  static constexpr int OROW = D + 4;  // padded row of the merge buffer
  static constexpr bool kQ = RT >= 3;  // query operands in LDS (registers are short)
  struct {
    int phys[kListPages], len[kListPages], mask[kListPages];
  } list;
  union {
    ThrLds<PER ? PER : 1, PER ? NW : 1> thr;
    bf16x8 k[NW][32 * D / 8];  // each wavefront's chunk of keys
    float o[NW][16][OROW];
  } u;
  bf16x8 q[kQ ? NR : 1][kQ ? RT * (D / 32) : 1][64];
  float m[NW][RT * 16], l[NW][RT * 16];
};

template <int D, int RT, int NR, int PER>
__global__ void __launch_bounds__(64 * NW) stream_attend_kernel(AttendArgs a, TopkArgs ta) {
  using L_t = StreamLds<D, RT, NR, PER>;
  constexpr int NT = NW / NR;  // wavefronts over the chunks
  __shared__ __attribute__((aligned(16))) L_t L;
  constexpr int KK = D / 32, DT = D / 16;
  const Geometry& g = a.g;
  const int tid = thread_index();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln16 = lane & 15, g4 = lane >> 4;
  // row tiles wr * RT ..., chunks wt, wt + NT, ...  (Two wavefronts on one chunk
  // stay together and share its lines in the L1: leaving out a tile without
  // rows, so that one runs ahead, takes 131K dense from 120 to 159 us.)
  const int wr = wave % NR, wt = wave / NR;
  // units (sequence, KV head, split, row group), row group fastest: the row
  // groups of a split run at the same time on one XCD and share its L2
  int u = xcd_remap(blockIdx.x, gridDim.x);
  const int rg = u % g.n_rgroups;
  u /= g.n_rgroups;
  const int split = u % g.n_splits;
  u /= g.n_splits;
  const int h = u % g.hk, b = u / g.hk;
  const int bh = b * g.hk + h;
  const int W = g.W, P = g.P;

  // ---- row state: query operands, and the mask value from which row r may
  // not use a page (mask < thr: past query tau uses pages with M_p < tau, the
  // current one every page, a row that does not exist none)
  bf16x8 q[RT][KK];
  f32x4 acc[RT][DT];
  float m_run[RT], l_run[RT];
  int thr[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int lt = wr * RT + j;
    const int rho = (rg * g.tiles_per_group + lt) * 16 + ln16;
    const bool live = lt < g.tiles_per_group && rho < g.R;
    const int r = live ? rho / g.G : 0;
    const int gq = live ? rho - r * g.G : 0;
    const int tau = a.step - W + r;
    thr[j] = (live && tau >= 0) ? (r == W ? 0x7fffffff : tau) : (int)0x80000000;
    m_run[j] = -INFINITY;
    l_run[j] = 0.f;
    const bf16_t* qrow = reinterpret_cast<const bf16_t*>(a.q) +
                         (((int64_t)b * (W + 1) + r) * g.hq + (int64_t)h * g.G + gq) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      bf16x8 v = *reinterpret_cast<const bf16x8*>(qrow + kk * 32 + 8 * g4);
      if (!live)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.f;
      q[j][kk] = v;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[j][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // ---- page list of the split: from the selection rows, or made here (PER > 0)
  const int first = split * g.pages_per_split;
  int np, nch;
  if constexpr (PER > 0) {
    int len = 0;
    // the head's writer: a workgroup of the last split, which has the fewest pages
    const bool writer = split == g.n_splits - 1 && rg == 0;
    const int k = select_role<PER, NW>(
        ta, bh,
        [&](int& tok_lp) { return len = select_len(g, a.seq_lens, a.pt, b, tok_lp); }, L.u.thr,
        writer, [&](int s, int p, int m, int ph) {
          if (s >= first && s < first + g.pages_per_split) {
            L.list.phys[s - first] = max(ph, 0);
            L.list.len[s - first] = ph >= 0 ? max(0, min(P, len - p * P)) : 0;
            L.list.mask[s - first] = m;
          }
        });
    np = max(0, min(g.pages_per_split, k - first));
    nch = (np + g.chunk_pages - 1) / g.chunk_pages;
    if (tid == 0 && np < nch * g.chunk_pages) {  // an odd list: an empty page fills its chunk
      L.list.phys[np] = 0;
      L.list.len[np] = 0;
      L.list.mask[np] = 0;
    }
  } else {
    const int k_sel = a.nsel[bh];
    const int seq_len = live_seq_len(g, a.seq_lens, a.pt, b);
    np = max(0, min(min(g.pages_per_split, k_sel - first), g.k_max - first));
    nch = (np + g.chunk_pages - 1) / g.chunk_pages;
    for (int i = tid; i < nch * g.chunk_pages; i += 64 * NW) {
      int lp = -1, m = 0, phys = -1;
      if (i < np) {
        const int64_t o = (int64_t)bh * g.k_max + first + i;
        lp = a.sel[o];
        m = a.msk[o];
        if (a.sel_phys)
          phys = a.sel_phys[o];
        else if (lp >= 0 && lp < g.max_pages)
          phys = a.pt[(int64_t)b * g.max_pages + lp];
      }
      const bool ok = lp >= 0 && lp < g.max_pages && phys >= 0 && phys < g.num_phys;
      // a page without stored tokens reads page 0 of the pool; none of it is used
      L.list.phys[i] = ok ? phys : 0;
      L.list.len[i] = ok ? max(0, min(P, seq_len - lp * P)) : 0;
      L.list.mask[i] = m;
    }
  }
  if constexpr (L_t::kQ) {  // only now: waiting for the queries would hold up the selection
    if (wt == 0)
#pragma unroll
      for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) L.q[wr][j * KK + kk][lane] = q[j][kk];
  }
  __syncthreads();  // page list ready, the selection's LDS free

  // ---- operands.  Values straight from the cache: V^T row dt * 16 + ln16,
  // tokens 8 g4 .. 8 g4 + 7 of the chunk.  Keys by whole rows (a wavefront's
  // load is 1 KB of consecutive rows), then through LDS into the lanes' order:
  // a row's 16-byte pieces are stored permuted by key_swizzle, so that the
  // sixteen rows of a tile read one piece without bank conflicts.
  const bool two = g.chunk_pages == 2;
  const int64_t blk = (int64_t)P * D;
  const int vtok = 8 * g4;
  const int vpg = two ? vtok >> 4 : 0;
  const int vslot = two ? vtok & 15 : vtok;
  const int voff = ln16 * P + vslot;
  const bf16_t* kc = reinterpret_cast<const bf16_t*>(a.kc);
  const bf16_t* vc = reinterpret_cast<const bf16_t*>(a.vc);
  constexpr int KP = D / 8;         // 16-byte pieces of a key row
  constexpr int RPL = 64 / KP;      // key rows of a load
  constexpr int NK = 32 / RPL;      // loads of a chunk's keys
  auto key_swizzle = [](int row) {
    return KP == 16 ? (row & 3) | (((row >> 3) & 3) << 2)
                    : ((row >> 1) & 1) | (((row >> 3) & 3) << 1);
  };
  bf16x8 kst[NK];
  bf16x8 vf[DT];
  bf16x8* klds = L.u.k[wave];
  auto load_k = [&](int c) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      // rows [i * RPL, (i + 1) * RPL) of the chunk lie in one page
      const int pg = two ? i * RPL >> 4 : 0;
      const int ph = __builtin_amdgcn_readfirstlane(L.list.phys[c * g.chunk_pages + pg]);
      const bf16x8* p = reinterpret_cast<const bf16x8*>(kc + ((int64_t)ph * g.hk + h) * blk);
      kst[i] = p[(i * RPL - 16 * pg) * KP + lane];
    }
  };
  // this chunk's keys from the staging registers into this wavefront's LDS
  auto stage_k = [&] {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int row = i * RPL + lane / KP;
      klds[row * KP + ((lane % KP) ^ key_swizzle(row))] = kst[i];
    }
  };
  auto load_v = [&](int c) {
    const int ph = L.list.phys[c * g.chunk_pages + vpg];
    const bf16_t* p = vc + ((int64_t)ph * g.hk + h) * blk + voff;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[dt] = *reinterpret_cast<const bf16x8*>(p + dt * 16 * P);
  };
  const bf16x8* ql = &L.q[L_t::kQ ? wr : 0][0][lane];
  // S tile t, lane row ln16: token 8 (ln16 / 4) + 4 t + ln16 % 4
  const int krow = 8 * (ln16 >> 2) + (ln16 & 3);
  // A weight's exponent is s * scale - m in one fused operation.  m is rounded, the
  // product in it is not: the difference can be 2^-25 |m| off either way, which
  // from 2^31 on overflows or empties a row.  Where a maximum turned out that large
  // the chunks are gone through once more with the scores scaled, and so
  // rounded like m, first: 264 rows 157.6 -> 158.2 us a pass, with the question
  // asked within the loop 160.0.
  float pre = 1.f, scale = a.scale_log2;  // factors of a score before and in the exponent
  int whole = 8;  // a lane with fewer stored tokens masks (and applies `pre`)
#pragma unroll 1
  for (;;) {
    asm volatile("" : "+s"(whole), "+s"(scale), "+s"(pre));  // one loop for both passes
    if (wt < nch) {
      load_k(wt);
      load_v(wt);
    }
#pragma unroll 1
    for (int c = wt; c < nch; c += NT) {
      const int slot = c * g.chunk_pages + vpg;
      const int tlen = L.list.len[slot] - vslot;  // stored ones of this lane's eight tokens
      const int mk = L.list.mask[slot];
      f32x4 s[RT][2];
#pragma unroll
      for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int t = 0; t < 2; ++t) s[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
      stage_k();
      const bool more = c + NT < nch;
      if (more) load_k(c + NT);
      // read again in every iteration: kept, they would take the registers of the
      // accumulators
      int qoff = 0;
      if constexpr (L_t::kQ) asm volatile("" : "+v"(qoff));
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        bf16x8 kf[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int row = krow + 4 * t;
          kf[t] = klds[row * KP + ((kk * 4 + g4) ^ key_swizzle(row))];
        }
#pragma unroll
        for (int j = 0; j < RT; ++j) {
          const bf16x8 qv = L_t::kQ ? ql[qoff + (j * KK + kk) * 64] : q[j][kk];
#pragma unroll
          for (int t = 0; t < 2; ++t)
            s[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t], qv, s[j][t], 0, 0, 0);
        }
      }
      if (wave_ballot(tlen < whole) != 0) {  // slots past the sequence: no score, and a zero value
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (4 * t + i >= tlen) s[j][t][i] = -INFINITY;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (e >= tlen) vf[dt][e] = (__bf16)0.f;
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
          for (int t = 0; t < 2; ++t) s[j][t] *= pre;
      }
      // running maxima (the token slots of one lane lie in one page), tile by tile
      // where a row's maximum grows; only then are the lanes' maxima combined and
      // the accumulators rescaled.  (Rescaling later, once a maximum has grown by
      // a margin, would be 10 % faster at 264 rows and costs accuracy: 2.4e-6
      // against 2.0e-6 relative.)
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        float mx = s[j][0][0];
#pragma unroll
        for (int i = 1; i < 8; ++i) mx = fmaxf(mx, s[j][i >> 2][i & 3]);
        if (wave_ballot(mk < thr[j] && mx * scale > m_run[j]) != 0) {
          const float m_new = fmaxf(m_run[j], col_max4(mk < thr[j] ? mx * scale : -INFINITY));
          const float alpha = __builtin_amdgcn_exp2f(m_run[j] - (m_new == -INFINITY ? 0.f : m_new));
          m_run[j] = m_new;
          l_run[j] *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) acc[j][dt] *= alpha;
        }
      }
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        const bool use = mk < thr[j];
        const float nm = m_run[j] == -INFINITY ? 0.f : -m_run[j];
        uint32_t ph[4], pl[4];  // the weights' bf16 upper parts and remainders, in pairs
        float psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          // the hardware exp2 (v_exp_f32): a weight under 2^-126 becomes 0
          const float x0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[j][e >> 2][e & 3], scale, nm));
          const float x1 =
              __builtin_amdgcn_exp2f(__builtin_fmaf(s[j][e >> 2][(e & 3) + 1], scale, nm));
          const float p0 = use ? x0 : 0.f, p1 = use ? x1 : 0.f;
          psum += p0 + p1;
          ph[e / 2] = pack_bf16(p0, p1);
          pl[e / 2] = pack_bf16(p0 - __uint_as_float(ph[e / 2] << 16),
                                p1 - __uint_as_float(ph[e / 2] & 0xFFFF0000u));
        }
        const bf16x8 phv = __builtin_bit_cast(bf16x8, u32x4v{ph[0], ph[1], ph[2], ph[3]});
        const bf16x8 plv = __builtin_bit_cast(bf16x8, u32x4v{pl[0], pl[1], pl[2], pl[3]});
        l_run[j] += psum;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          acc[j][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], phv, acc[j][dt], 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          acc[j][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], plv, acc[j][dt], 0, 0, 0);
      }
      if (more) load_v(c + NT);
    }
    bool large = false;
#pragma unroll
    for (int j = 0; j < RT; ++j)
      large = large || (fabsf(m_run[j]) > 0x1p20f && fabsf(m_run[j]) < INFINITY);
    if (whole == 8 && wave_ballot(large) != 0) {
      whole = 0x7fffffff;
      pre = scale;
      scale = 1.f;
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        m_run[j] = -INFINITY;
        l_run[j] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[j][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    } else {
      break;
    }
  }

  // ---- merge the wavefronts' states: factors per row, then the outputs tile by
  // tile through LDS
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const float l = col_sum4(l_run[j]);
    if (g4 == 0) {
      L.m[wave][j * 16 + ln16] = m_run[j];
      L.l[wave][j * 16 + ln16] = l;
    }
  }
  __syncthreads();  // states in LDS; the page list is no longer read
  const int64_t part0 = ((int64_t)bh * g.n_splits + split) * g.R;
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int lt = wr * RT + j;
    const int row = (rg * g.tiles_per_group + lt) * 16 + ln16;
    const int rr = j * 16 + ln16;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NT; ++w) M = fmaxf(M, L.m[w * NR + wr][rr]);
    const float Mu = M == -INFINITY ? 0.f : M;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NT; ++w)
      sum += L.l[w * NR + wr][rr] * __builtin_amdgcn_exp2f(L.m[w * NR + wr][rr] - Mu);
    const float f = sum > 0.f ? __builtin_amdgcn_exp2f(m_run[j] - Mu) / sum : 0.f;
    // -inf for an empty sum; +inf (fminf skips NaN) for a NaN one, from NaN or
    // infinite scores: the combine then makes the row NaN.  One rounding at the
    // normaliser's size, since with few splits none average out.
    if (wt == 0 && g4 == 0 && lt < g.tiles_per_group && row < g.R)
      __builtin_nontemporal_store(fminf(__builtin_fmaf(M, kLn2, __log2f(sum) * kLn2), INFINITY),
                                  a.l_ws + part0 + row);
    if (j > 0) __syncthreads();  // the previous tiles have been read
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      *reinterpret_cast<f32x4*>(&L.u.o[wave][ln16][dt * 16 + 4 * g4]) = acc[j][dt] * f;
    __syncthreads();
    constexpr int VPR = D / 4;  // 16-byte pieces per row
    // tile j of each of the NR row ranges: the NT wavefronts' rows added up
#pragma unroll
    for (int r0 = 0; r0 < NR; ++r0) {
      const int t0 = r0 * RT + j;
      if (t0 >= g.tiles_per_group) break;  // uniform
      const int row0 = (rg * g.tiles_per_group + t0) * 16;
      for (int e = tid; e < 16 * VPR; e += 64 * NW) {
        const int rw = e / VPR, c4 = (e - rw * VPR) * 4;
        f32x4 o = *reinterpret_cast<const f32x4*>(&L.u.o[r0][rw][c4]);
#pragma unroll
        for (int w = 1; w < NT; ++w) o += *reinterpret_cast<const f32x4*>(&L.u.o[w * NR + r0][rw][c4]);
        if (row0 + rw < g.R)
          __builtin_nontemporal_store(
              o, reinterpret_cast<f32x4*>(a.o_ws + (part0 + row0 + rw) * D + c4));
      }
    }
  }
}

template <int D, int RT, int NR>
hipError_t go(const AttendArgs& a, const TopkArgs* ta, hipStream_t s) {
  const Geometry& g = a.g;
  const unsigned n = (unsigned)((int64_t)g.n_splits * g.n_rgroups * g.hk * g.batch);
  if (!ta) {
    stream_attend_kernel<D, RT, NR, 0><<<n, 64 * NW, 0, s>>>(a, TopkArgs{});
    return hipGetLastError();
  }
  if (g.max_pages > kSelectPer * 64 * NW) return hipErrorInvalidValue;
  return with_select_per(g.max_pages, [&](auto per) {
    stream_attend_kernel<D, RT, NR, decltype(per)::value><<<n, 64 * NW, 0, s>>>(a, *ta);
    return hipGetLastError();
  });
}

template <int D>
hipError_t go_d(const AttendArgs& a, const TopkArgs* ta, hipStream_t s) {
  switch (a.g.tiles_per_group) {
    case 1: return go<D, 1, 1>(a, ta, s);
    case 2: return go<D, 2, 1>(a, ta, s);
    case 3: return go<D, 3, 1>(a, ta, s);
    case 4: return go<D, 2, 2>(a, ta, s);
    case 5:
    case 6: return go<D, 3, 2>(a, ta, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

namespace {
// Small calls go to attend_kernel (attend_select_kernel): a wavefront's merge of
// several row tiles here is long straight-line code that runs once per workgroup.
// The two times, in us, for g (attend_kernel's split) and x (the split here), each
// from rounds of workgroups over the compute units, the chunks that a wavefront
// goes through one after another, and the partial rows that are written and
// combined; the constants fit 1450 measured shapes (1 to 17 row tiles, 2 to 200 KV
// heads, 4 to 512 pages, d 64 and 128) to 5 to 10 %.  The choice costs 0.3 % more
// than the faster of the two in every shape, the streamed attention always 8 %,
// attend_kernel always 16 %.  Some on either side (attend_kernel / here, attention
// and combine): 8 heads of 36 rows, 128 pages 12.6 / 15.8, 512 pages 22.4 / 20.4; 16
// heads of 20 rows, 16 pages 9.3 / 12.2, 10 of 260, 16 pages 15.0 / 17.9, 200 of 16,
// 4 pages 14.0 / 11.2.  With the selection in front (4 us a round) three launches
// took: 8 heads of 36 rows, 64 pages 19.7 / 21.9, 32 x 36 x 64 24.4 / 25.2, 64 x 36 x
// 64 30.8 / 28.6.  Splits of more than four chunks there stay here.  So does one row
// tile (2 heads of 4 rows, 256 pages 14.6 / 10.4, 200 of 16, 4 pages 14.0 / 11.2),
// but for d 128 in 4 to 16 splits of one chunk without a selection: 8 heads of 16
// rows, 16 pages 9.0 / 9.9, 32 of 4, 16 pages 9.0 / 9.3.
bool attend_kernel_wins(const Geometry& g, const Geometry& x, bool selects) {
  const int cap = compute_units();
  const int64_t heads = (int64_t)g.batch * g.hk;
  if (x.tiles_per_group == 1)
    return !selects && g.D == 128 && g.chunks_per_split == 1 && g.n_splits >= 4 &&
           g.n_splits <= 16 && heads * g.n_splits <= cap;
  if (g.chunks_per_split > 4) return false;
  auto time = [&](const Geometry& y, int chunks, const float (&c)[5]) {
    const int64_t rounds = (heads * y.n_rgroups * y.n_splits + cap - 1) / cap;
    const float partials = 1e-6f * (float)(heads * y.n_splits * y.R) * (float)y.D;
    return c[0] + (float)rounds * (c[1] + (selects ? 4.f : 0.f) + c[2] * (float)(chunks * y.D) / 128.f) +
           c[3] * partials + c[4] * (float)((y.n_splits - 1) / 32);
  };
  // fixed, per round, per chunk of 32 tokens at d 128, per million partial
  // elements, per 32 splits after the first (another group of the combine)
  static constexpr float kHere[5][5] = {{4.0f, 4.0f, 3.9f, 6.4f, 0.f},   // 2 row tiles
                                        {4.7f, 4.7f, 5.2f, 4.8f, 0.f},   // 3
                                        {2.0f, 8.0f, 2.0f, 2.8f, 1.1f},  // 4
                                        {1.3f, 10.1f, 2.8f, 2.7f, 0.7f},
                                        {0.1f, 12.1f, 3.0f, 2.2f, 1.5f}};
  static constexpr float kThere[2][5] = {{8.0f, 0.f, 1.5f, 2.1f, 1.5f},  // 1 tile a wavefront
                                         {6.2f, 3.0f, 2.0f, 1.8f, 0.7f}};
  const int nw = x.tiles_per_group <= 3 ? NW : NW / 2;  // wavefronts over the chunks (go_d)
  return time(g, g.chunks_per_split, kThere[g.rtw - 1]) <
         time(x, (x.chunks_per_split + nw - 1) / nw, kHere[x.tiles_per_group - 2]);
}
}  // namespace

Geometry attend_geometry(const Geometry& g, bool selects) {
  if (g.dtype != RETRO_BF16) return g;
  Geometry x = g;
  constexpr int kMaxTiles = 6;  // two wavefronts side by side, three tiles each
  x.n_rgroups = (g.row_tiles + kMaxTiles - 1) / kMaxTiles;
  x.tiles_per_group = (g.row_tiles + x.n_rgroups - 1) / x.n_rgroups;
  const int nw = x.tiles_per_group <= 3 ? NW : NW / 2;  // wavefronts over the chunks (go_d)
  x.stream = 1;
  // One workgroup per compute unit (its registers); the split count with the
  // smallest time, counted in chunk iterations of a wavefront: rounds of
  // workgroups times the iterations of one, plus three for its start and merge.
  // (For a number of iterations, the fewest splits that reach it.)
  const int64_t heads = (int64_t)g.batch * g.hk * x.n_rgroups;
  const int cap = compute_units();
  const int cps_max = kListPages / g.chunk_pages;
  int best = 0;
  int64_t best_cost = 0;
  for (int it = (std::min(g.chunks_max, cps_max) + nw - 1) / nw; it >= 1; --it) {
    const int cps = std::min(it * nw, cps_max);
    const int ns = (g.chunks_max + cps - 1) / cps;
    if (ns > g.n_splits) break;
    const int64_t cost = (heads * ns + cap - 1) / cap * (it + 3);
    if (best == 0 || cost < best_cost) {
      best = ns;
      best_cost = cost;
    }
  }
  if (best == 0) best = g.n_splits;
  x.chunks_per_split = (g.chunks_max + best - 1) / best;
  x.n_splits = (g.chunks_max + x.chunks_per_split - 1) / x.chunks_per_split;
  x.pages_per_split = x.chunks_per_split * g.chunk_pages;
  return attend_kernel_wins(g, x, selects) ? g : x;
}

hipError_t launch_stream_attend(const AttendArgs& a, const TopkArgs* ta, hipStream_t s) {
  return a.g.D == 128 ? go_d<128>(a, ta, s) : go_d<64>(a, ta, s);
}

}  // namespace retro
