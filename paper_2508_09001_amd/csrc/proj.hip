// Dense projections of the multi-layer decode with re-embedding (Sec. 3.3): the
// W+1 window rows of every sequence, a few dozen at most, times a weight matrix.
// With so few rows the product is bound by reading the weight once from HBM
// (the paper's appendix on linear layers makes the same point), so each weight is
// stored pre-tiled for the MFMA operand layout: one wavefront load of 1 KB per
// 16 columns x 32 reduction elements, contiguous in memory.
//
// Packed layout of a [K][N] weight (y = x . w): [N/16][K/32][4][16][8] bf16;
// element (k, n) sits at tile n/16, step k/32, group (k%32)/8, column n%16,
// position k%8.  Lane l = 16 * group + column of a wavefront then holds exactly
// the B operand of v_mfma_f32_16x16x32_bf16 for its column.
//
// A workgroup owns 16 output columns; its PJ_WAVES wavefronts split the
// reduction, each accumulating all row tiles (16 rows each) of its share with
// MFMA, and the shares are summed in a fixed order through LDS.  Sixteen
// wavefronts of 512 reduction elements each load their whole share of a
// 4096-deep weight in one pass: the launch is a single round trip to HBM per
// wavefront, which is what a few-row product costs.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "proj.h"

namespace retro {
namespace {

constexpr int PJ_WAVES = 16;         // wavefronts per workgroup, each a slice of the reduction
constexpr int PJ_MIN_STEPS = 2;      // 32-element reduction steps per wavefront (at least)
constexpr int PJ_MAX_ROW_TILES = 7;  // up to 112 rows (more would spill registers)

__device__ __forceinline__ uint16_t bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN stays NaN
  return static_cast<uint16_t>((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Row operands.  A wavefront loads a 16-row x 32-element tile of x with four
// consecutive lanes on one row (64 bytes of bf16; in operand order, lane % 16
// being the row, four consecutive lanes would touch four rows and the load take
// four times as long), converts f32 rows to bf16, and turns it into operand
// order through 1 KB of LDS of its own; the pieces of a row are stored permuted
// so that neither access meets bank conflicts.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <bool F32IN>
struct RowRaw {
  u32x4 v[F32IN ? 2 : 1];
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}

// this lane's piece of a tile: row lane / 4 of the 16 from row0, elements
// [k + 8 * (lane % 4), + 8); zero past the last row.  OPER: in operand order at
// once, row lane % 16, elements [k + 8 * (lane / 16), + 8).
template <bool F32IN, bool OPER>
__device__ __forceinline__ RowRaw<F32IN> load_rows(const void* x, int rows, int K, int row0, int k,
                                                   int lane) {
  RowRaw<F32IN> r{};
  const int row = row0 + (OPER ? lane & 15 : lane >> 2);
  if (row < rows) {
    const int64_t e = (int64_t)row * K + k + 8 * (OPER ? lane >> 4 : lane & 3);
    if constexpr (F32IN) {
      const u32x4* p = reinterpret_cast<const u32x4*>(static_cast<const float*>(x) + e);
      r.v[0] = p[0];
      r.v[1] = p[1];
    } else {
      r.v[0] = *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(x) + e);
    }
  }
  return r;
}

// the tile in operand order: row lane % 16, elements [8 * (lane / 16), + 8)
template <bool F32IN>
__device__ __forceinline__ bf16x8 rows_to_operand(const RowRaw<F32IN>& r, u32x4* lds, int lane) {
  u32x4 w = r.v[0];
  if constexpr (F32IN) {
    const u32x4 a = r.v[0], b = r.v[1];
    w = u32x4{pack2(__uint_as_float(a[0]), __uint_as_float(a[1])),
              pack2(__uint_as_float(a[2]), __uint_as_float(a[3])),
              pack2(__uint_as_float(b[0]), __uint_as_float(b[1])),
              pack2(__uint_as_float(b[2]), __uint_as_float(b[3]))};
  }
  const int wrow = lane >> 2, row = lane & 15;
  lds[wrow * 4 + ((lane & 3) ^ (wrow >> 2))] = w;
  return __builtin_bit_cast(bf16x8, lds[row * 4 + ((lane >> 4) ^ (row >> 2))]);
}

struct ProjArgs {
  const void* x;          // [rows][K]: bf16 (QKV) or f32 (output projection)
  const uint4* w;         // packed weight, N columns
  int rows, K, N;
  // QKV: columns [0, nq) -> q, [nq, nq + nkv) -> k, the rest -> v (bf16 [rows][n])
  int nq, nkv;
  bf16_t *q, *k, *v;
  // output projection: h [rows][N] f32 += bf16(y); x_next = bf16(h)
  float* h;
  bf16_t* x_next;
  // QKV with UpdateKV (rows = batch * W1 window rows): row W1-1 of every
  // sequence goes to k / v ([batch][nkv]), the n_upd rows before it overwrite the
  // sequence's last n_upd stored tokens, whose pages' digests are recomputed
  int W1, n_upd, P, D, hk, max_pages, num_phys;
  bf16_t *kc, *vc, *dg;
  const int32_t* pt;
  const int32_t* seq_lens;
};

constexpr int PJ_MAX_BATCH = 16 * PJ_MAX_ROW_TILES;

// Row tiles whose loads are in flight together per reduction step group: what the
// registers leave beside the weight's.
constexpr int rows_unroll(int mt, bool f32, int ct) {
  if (ct > 1 && mt > 4) return 1;
  if (f32) return mt == 1 ? 4 : mt == 2 ? 2 : 1;
  return mt == 1 ? 8 : mt == 2 ? 4 : mt <= 5 ? 2 : 1;
}

// U: reduction steps of the weight requested together.  SH: shares of the reduction
// per wavefront, each summed up by itself and added to the others in LDS in order.
template <int MT, bool OUT, int U, bool UPD = false, int CT = 1, int NW = PJ_WAVES, int SH = 1>
__global__ void __launch_bounds__(64 * NW) proj_kernel(ProjArgs a) {
  // a single tile of bf16 rows is loaded in operand order: with few rows the
  // loads are short either way and the pass through LDS would be the longer one
  constexpr bool OPER = MT == 1 && !OUT;
  constexpr int UA = OPER || rows_unroll(MT, OUT, CT) > U ? U : rows_unroll(MT, OUT, CT);
  // output tiles summed per round, 256 threads each
  constexpr int TPR = NW * 64 / 256 < CT * MT ? NW * 64 / 256 : CT * MT;
  // each wavefront's row tiles in turn; the shares of TPR tiles afterwards
  __shared__ __attribute__((aligned(16))) union {
    u32x4 x[OPER ? 1 : NW][OPER ? 1 : MT][64];
    float red[TPR][NW * SH][4][64];
  } L;
  __shared__ int s_len[UPD ? PJ_MAX_BATCH : 1];
  __shared__ uint16_t s_val[UPD ? CT : 1][UPD ? MT * 16 : 1][16];
  if constexpr (UPD) {
    // sequence lengths before the step's append, loaded under the weight stream
    const int nb = a.rows / a.W1;
    if ((int)threadIdx.x < nb) s_len[threadIdx.x] = a.seq_lens[threadIdx.x];
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile0 = blockIdx.x * CT;  // CT column tiles share each load of the rows
  const int steps = a.K / 32, per_share = steps / (NW * SH);
  const int s0 = wave * SH * per_share;
  const u32x4* wp = reinterpret_cast<const u32x4*>(a.w) + ((int64_t)tile0 * steps + s0) * 64 + lane;
  f32x4 acc[SH][CT][MT];
  auto one_pass = [&](int s, f32x4 (&acc)[CT][MT]) {
    RowRaw<OUT> raw[UA][MT];
    auto rows_of = [&](int v) {
#pragma unroll
      for (int u = 0; u < UA; ++u)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          raw[u][mt] = load_rows<OUT, OPER>(a.x, a.rows, a.K, mt * 16, (s0 + s + v + u) * 32, lane);
    };
    // Loads complete in order.  The output projection's first rows (from the L2)
    // go ahead of the weight (19.7 us at 72 rows, 20.1 behind it); the query /
    // key / value rows behind it (22.9 us, 24.3 ahead), step by step with it for
    // a single tile in operand order.
    u32x4 b[U][CT];
    if constexpr (OUT) rows_of(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int c = 0; c < CT; ++c) b[u][c] = wp[((int64_t)c * steps + s + u) * 64];
      if constexpr (OPER)
        raw[u][0] = load_rows<OUT, OPER>(a.x, a.rows, a.K, 0, (s0 + s + u) * 32, lane);
    }
#pragma unroll
    for (int v = 0; v < U; v += UA) {
      if (!OPER && (!OUT || v > 0)) rows_of(v);
#pragma unroll
      for (int u = 0; u < UA; ++u)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          bf16x8 av;
          if constexpr (OPER) av = __builtin_bit_cast(bf16x8, raw[u][mt].v[0]);
          else av = rows_to_operand<OUT>(raw[u][mt], L.x[wave][mt], lane);
#pragma unroll
          for (int c = 0; c < CT; ++c)
            acc[c][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                av, __builtin_bit_cast(bf16x8, b[v + u][c]), acc[c][mt], 0, 0, 0);
        }
    }
  };
#pragma unroll
  for (int sh = 0; sh < SH; ++sh) {
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[sh][c][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s = 0; s < per_share; s += U) one_pass(sh * per_share + s, acc[sh]);
  }
  // TPR tiles at a time through LDS: output (i, l) of column tile c and row
  // tile mt is row mt*16 + 4*(l/16) + i, column (tile0 + c)*16 + l%16
#pragma unroll
  for (int p0 = 0; p0 < CT * MT; p0 += TPR) {
    if (!OPER || p0 > 0) __syncthreads();  // the row tiles (or the previous round's sums) are read
#pragma unroll
    for (int t = 0; t < TPR; ++t)
      if (p0 + t < CT * MT)
#pragma unroll
        for (int sh = 0; sh < SH; ++sh)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            L.red[t][wave * SH + sh][i][lane] = acc[sh][(p0 + t) / MT][(p0 + t) % MT][i];
    __syncthreads();
    const int pass = p0 + (int)(threadIdx.x >> 8), c = pass / MT, mt = pass % MT;
    const int o = threadIdx.x & 255;
    if (pass >= CT * MT || pass - p0 >= TPR) continue;
    const int i = o >> 6, l = o & 63;
    const int row = mt * 16 + 4 * (l >> 4) + i;
    if (row >= a.rows) continue;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW * SH; ++w) sum += L.red[threadIdx.x >> 8][w][i][l];
    const int col = (tile0 + c) * 16 + (l & 15);
    const uint16_t y = bf16_rne(sum);
    if constexpr (OUT) {
      const int64_t e = (int64_t)row * a.N + col;
      const float hv = a.h[e] + __uint_as_float(uint32_t(y) << 16);
      a.h[e] = hv;
      a.x_next[e].bits = bf16_rne(hv);
    } else if constexpr (UPD) {
      s_val[c][row][l & 15] = y;
      if (col < a.nq) {
        a.q[(int64_t)row * a.nq + col].bits = y;
        continue;
      }
      const bool is_k = col < a.nq + a.nkv;
      const int c = is_k ? col - a.nq : col - a.nq - a.nkv;
      const int b = row / a.W1, j = row % a.W1;
      if (j == a.W1 - 1) {  // the step's token: appended by the step itself
        (is_k ? a.k : a.v)[(int64_t)b * a.nkv + c].bits = y;
        continue;
      }
      const int len = s_len[b];
      const int pos = len - (a.W1 - 1) + j;  // row j of the window is token t-W+j
      if (j < a.W1 - 1 - a.n_upd || pos < 0) continue;
      const int lp = pos / a.P, slot = pos % a.P;
      if (lp >= a.max_pages) continue;
      const int phys = a.pt[(int64_t)b * a.max_pages + lp];
      if (phys < 0 || phys >= a.num_phys) continue;
      const int h = c / a.D, e = c % a.D;
      const int64_t ph = (int64_t)phys * a.hk + h;
      if (is_k)
        a.kc[(ph * a.P + slot) * a.D + e].bits = y;
      else
        a.vc[(ph * a.D + e) * a.P + slot].bits = y;
    } else {
      if (col < a.nq)
        a.q[(int64_t)row * a.nq + col].bits = y;
      else if (col < a.nq + a.nkv)
        a.k[(int64_t)row * a.nkv + (col - a.nq)].bits = y;
      else
        a.v[(int64_t)row * a.nkv + (col - a.nq - a.nkv)].bits = y;
    }
  }
  if constexpr (UPD) {
    // digests of the pages the update touched, for this workgroup's 16 key
    // columns: element-wise min / max over every stored key of the page, the
    // updated ones taken from s_val (a min / max cannot be narrowed in place)
    if (a.n_upd == 0) return;
    __syncthreads();
    const int nb = a.rows / a.W1;
    const int span = (a.n_upd + a.P - 1) / a.P + 1;  // pages a run of n_upd can touch
#pragma unroll
    for (int c = 0; c < CT; ++c) {
    const int col0 = (tile0 + c) * 16;
    if (col0 < a.nq || col0 >= a.nq + a.nkv) continue;
    const int c0 = col0 - a.nq, h = c0 / a.D;
    for (int o = threadIdx.x; o < nb * span * 16; o += blockDim.x) {
      const int cl = o & 15, pi = (o >> 4) % span, b = (o >> 4) / span;
      const int e = c0 % a.D + cl;
      const int len = s_len[b];
      const int start = max(len - a.n_upd, 0);
      const int lp = start / a.P + pi;
      if (lp >= a.max_pages || lp * a.P >= len) continue;
      const int phys = a.pt[(int64_t)b * a.max_pages + lp];
      if (phys < 0 || phys >= a.num_phys) continue;
      const int filled = min(a.P, len - lp * a.P);
      const int64_t ph = (int64_t)phys * a.hk + h;
      float lo = 0.f, hi = 0.f;
      for (int sl = 0; sl < filled; ++sl) {
        const int pos = lp * a.P + sl;
        float f;
        if (pos >= start)
          f = to_f32(bf16_t{s_val[c][b * a.W1 + (pos - len + a.W1 - 1)][cl]});
        else
          f = to_f32(a.kc[(ph * a.P + sl) * a.D + e]);
        if (sl == 0) {
          lo = f;
          hi = f;
        } else {
          if (f < lo) lo = f;
          if (hi < f) hi = f;
        }
      }
      bf16_t* drow = a.dg + (((int64_t)b * a.hk + h) * a.max_pages + lp) * 2 * a.D;
      drow[e].bits = static_cast<uint16_t>(__float_as_uint(lo) >> 16);
      drow[a.D + e].bits = static_cast<uint16_t>(__float_as_uint(hi) >> 16);
    }
    }
  }
}

template <int MT, bool OUT, bool UPD>
void launch_proj_mt(const ProjArgs& a, hipStream_t s) {
  // a wavefront's whole share of the weight requested at once where it is eight
  // steps (K = 4096; the share, K / 512 steps, is even)
  // query / key / value with three to five row tiles: two column tiles per
  // workgroup where N allows, halving the re-reads of the rows (every workgroup
  // reads all of them); not for the output projection, whose 4096 columns would
  // then leave half the compute units without a workgroup
  constexpr int CT = (!OUT && MT >= 3 && MT <= 5) ? 2 : 1;
  const int per_wave = a.K / 32 / PJ_WAVES;
  const dim3 block(64 * PJ_WAVES);
  if (CT == 2 && a.N % 32 == 0) {
    const dim3 grid(a.N / 32);
    if (per_wave % 4 == 0)
      proj_kernel<MT, OUT, 4, UPD, CT><<<grid, block, 0, s>>>(a);
    else
      proj_kernel<MT, OUT, 2, UPD, CT><<<grid, block, 0, s>>>(a);
    return;
  }
  const dim3 grid(a.N / 16);
  if constexpr (MT <= 2) {
    // one or two row tiles and more column tiles than compute units: eight
    // wavefronts per workgroup (two passes of eight steps), so that every
    // workgroup of the launch is resident at once instead of a second,
    // half-empty round.  Two tiles keep the sixteen shares of the other shapes:
    // the sums are formed in the same order whatever N is.
    constexpr int SH = MT == 2 ? 2 : 1;
    if ((int)grid.x > compute_units() && (a.K / 32 / (8 * SH)) % 8 == 0) {
      proj_kernel<MT, OUT, 8, UPD, 1, 8, SH><<<grid, dim3(64 * 8), 0, s>>>(a);
      return;
    }
  }
  constexpr int UM = OUT && MT == 7 ? 4 : 8;  // eight steps and seven f32 row tiles would spill
  if (per_wave % UM == 0)
    proj_kernel<MT, OUT, UM, UPD><<<grid, block, 0, s>>>(a);
  else if (per_wave % 4 == 0)
    proj_kernel<MT, OUT, 4, UPD><<<grid, block, 0, s>>>(a);
  else
    proj_kernel<MT, OUT, 2, UPD><<<grid, block, 0, s>>>(a);
}

template <bool OUT, bool UPD>
hipError_t launch_proj(const ProjArgs& a, hipStream_t s) {
  switch ((a.rows + 15) / 16) {
    case 1: launch_proj_mt<1, OUT, UPD>(a, s); break;
    case 2: launch_proj_mt<2, OUT, UPD>(a, s); break;
    case 3: launch_proj_mt<3, OUT, UPD>(a, s); break;
    case 4: launch_proj_mt<4, OUT, UPD>(a, s); break;
    case 5: launch_proj_mt<5, OUT, UPD>(a, s); break;
    case 6: launch_proj_mt<6, OUT, UPD>(a, s); break;
    default: launch_proj_mt<7, OUT, UPD>(a, s); break;
  }
  return hipGetLastError();
}

// [K][N] row-major -> packed tiles; one thread per 8-element group.
__global__ void pack_kernel(const bf16_t* __restrict__ w, int K, int N, uint4* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)K * N / 8;
  if (idx >= total) return;
  const int lane = (int)(idx & 63);
  const int64_t ts = idx >> 6;           // tile * steps + step
  const int steps = K / 32;
  const int tile = (int)(ts / steps), step = (int)(ts % steps);
  const int col = tile * 16 + (lane & 15);
  const int k0 = step * 32 + 8 * (lane >> 4);
  uint32_t h[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) h[j] = w[(int64_t)(k0 + j) * N + col].bits;
  out[idx] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                        h[6] | (h[7] << 16));
}

retro_status status_of(hipError_t e) { return e == hipSuccess ? RETRO_OK : RETRO_EHIP; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool proj_shape_ok(int rows, int K, int N) {
  return rows >= 1 && rows <= 16 * PJ_MAX_ROW_TILES && K > 0 &&
         K % (32 * PJ_WAVES * PJ_MIN_STEPS) == 0 &&
         N > 0 && N % 16 == 0;
}

}  // namespace

hipError_t launch_project_qkv_update(const Geometry& g, const retro_kv_cache& c, const void* x,
                                     int k, const void* w_packed, int n_upd, void* q,
                                     void* k_new, void* v_new, hipStream_t s) {
  ProjArgs a{};
  a.x = x;
  a.w = static_cast<const uint4*>(w_packed);
  a.W1 = g.W + 1;
  a.rows = g.batch * a.W1;
  a.K = k;
  a.nq = g.hq * g.D;
  a.nkv = g.hk * g.D;
  a.N = a.nq + 2 * a.nkv;
  a.q = static_cast<bf16_t*>(q);
  a.k = static_cast<bf16_t*>(k_new);
  a.v = static_cast<bf16_t*>(v_new);
  a.n_upd = n_upd;
  a.P = g.P;
  a.D = g.D;
  a.hk = g.hk;
  a.max_pages = g.max_pages;
  a.num_phys = g.num_phys;
  a.kc = static_cast<bf16_t*>(c.k_cache);
  a.vc = static_cast<bf16_t*>(c.v_cache);
  a.dg = static_cast<bf16_t*>(c.digest);
  a.pt = c.page_table;
  a.seq_lens = c.seq_lens;
  return launch_proj<false, true>(a, s);
}

bool project_qkv_update_supported(const Geometry& g, int k) {
  return g.dtype == RETRO_BF16 && proj_shape_ok(g.batch * (g.W + 1), k, (g.hq + 2 * g.hk) * g.D) &&
         g.batch <= PJ_MAX_BATCH && g.D % 16 == 0;
}

}  // namespace retro

namespace {

// fp32 projections (fp32 stacks): each output element is one in-order chain of
// fused multiply-adds over the k inputs, so the parallelism is that of the
// outputs alone: a workgroup owns 16 columns and up to RB rows, one chain per
// thread of its first wavefronts (column tid % 16, row tid / 16 of the block).
// Eight more wavefronts feed them: slabs of 256 inputs (16 columns of w, RB rows
// of x) are requested ahead into registers, w by kF32Depth slabs (64 KB in
// flight per workgroup), and go through two LDS buffers, w transposed, from
// which a chain reads four steps of its column and its row at a time, two
// batches of 16 steps ahead of the multiply-adds.  Column tiles that share
// 128-byte lines are numbered to the same XCD.  [5][4096] x [4096][4096] takes 24
// us (2.8 TB/s), [5][4096] x [4096][1024] 21 us, the chain's length, 17 rows 51 us
// (LDS reads); one thread per output reading w from memory step by step took 430,
// 315 and 430 us, the same wavefronts feeding and computing 26, 25 and 53 us.
constexpr int kF32Loaders = 512;
constexpr int kF32Cols = 16;
constexpr int kF32Slab = 256;
constexpr int kF32Depth = 4;   // slabs of w in flight
constexpr int kF32XDepth = 2;  // slabs of x in flight (from the L2)
constexpr int kF32Row = kF32Slab + 4;  // padded LDS row

// VEC: w is read 16 bytes at a time (w 16-byte aligned, N a multiple of 4).
template <int RB, bool VEC>
__global__ void __launch_bounds__(kF32Loaders + RB * kF32Cols) project_f32_kernel(
    const float* __restrict__ x, int rows, int K, const float* __restrict__ w, int N,
    float* __restrict__ y, int accumulate) {
  constexpr int NC = RB * kF32Cols;                           // chain threads
  constexpr int WPT = kF32Cols * kF32Slab / 4 / kF32Loaders;  // 4-column pieces per loader and slab
  constexpr int XPT = RB * kF32Slab / kF32Loaders;            // row elements per loader and slab
  static_assert(NC % 64 == 0 && kF32Depth % 2 == 0 && kF32Depth % kF32XDepth == 0, "slab buffers");
  typedef float f32x4v __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) float ws[2][kF32Cols][kF32Row];
  __shared__ __attribute__((aligned(16))) float xs[2][RB][kF32Row];
  const int j0 = retro::xcd_remap(blockIdx.x, gridDim.x) * kF32Cols, r0 = blockIdx.y * RB;
  const int nrows = min(RB, rows - r0);
  const int slabs = (K + kF32Slab - 1) / kF32Slab;
  // Slab s goes through buffer s & 1: written before barrier s, read before
  // barrier s + 1, and rewritten (slab s + 2) after it.  Every wavefront passes
  // `slabs` barriers.
  if ((int)threadIdx.x >= NC) {
    const int tid = threadIdx.x - NC;
    f32x4v wr[kF32Depth][WPT];
    float xr[kF32XDepth][XPT];
    auto load_w = [&](int s, f32x4v (&wv)[WPT]) {
      const int i0 = s * kF32Slab;
#pragma unroll
      for (int p = 0; p < WPT; ++p) {
        const int e = tid + p * kF32Loaders;
        const int i = i0 + e / 4, c = j0 + 4 * (e % 4);
        f32x4v v = f32x4v{0.f, 0.f, 0.f, 0.f};
        if constexpr (VEC) {
          if (i < K && c < N) v = *reinterpret_cast<const f32x4v*>(w + (int64_t)i * N + c);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (i < K && c + q < N) v[q] = w[(int64_t)i * N + c + q];
        }
        wv[p] = v;
      }
    };
    auto load_x = [&](int s, float (&xv)[XPT]) {
#pragma unroll
      for (int p = 0; p < XPT; ++p) {
        const int e = tid + p * kF32Loaders;
        const int r = e / kF32Slab, i = s * kF32Slab + e % kF32Slab;
        xv[p] = (r < nrows && i < K) ? x[(int64_t)(r0 + r) * K + i] : 0.f;
      }
    };
#pragma unroll
    for (int d = 0; d < kF32Depth; ++d) {
      if (d < kF32XDepth && d < slabs) load_x(d, xr[d % kF32XDepth]);
      if (d < slabs) load_w(d, wr[d]);
    }
    for (int s0 = 0; s0 < slabs; s0 += kF32Depth) {
#pragma unroll
      for (int d = 0; d < kF32Depth; ++d) {
        const int s = s0 + d;
        if (s >= slabs) break;  // uniform
        const int buf = d & 1;
#pragma unroll
        for (int p = 0; p < WPT; ++p) {
          const int e = tid + p * kF32Loaders;
#pragma unroll
          for (int q = 0; q < 4; ++q) ws[buf][4 * (e % 4) + q][e / 4] = wr[d][p][q];
        }
#pragma unroll
        for (int p = 0; p < XPT; ++p) {
          const int e = tid + p * kF32Loaders;
          xs[buf][e / kF32Slab][e % kF32Slab] = xr[d % kF32XDepth][p];
        }
        if (s + kF32XDepth < slabs) load_x(s + kF32XDepth, xr[d % kF32XDepth]);
        if (s + kF32Depth < slabs) load_w(s + kF32Depth, wr[d]);
        __syncthreads();
      }
    }
    return;
  }
  const int c = threadIdx.x % kF32Cols, r = threadIdx.x / kF32Cols;
  float acc = 0.f;
  for (int s = 0; s < slabs; ++s) {
    __syncthreads();
    const int cnt = min(kF32Slab, K - s * kF32Slab);
    const float* wc = ws[s & 1][c];
    const float* xc = xs[s & 1][r];
    if (cnt == kF32Slab) {  // uniform
      f32x4v a[3][4], b[3][4];
      auto fetch = [&](int t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[t % 3][q] = *reinterpret_cast<const f32x4v*>(xc + 16 * t + 4 * q);
          b[t % 3][q] = *reinterpret_cast<const f32x4v*>(wc + 16 * t + 4 * q);
        }
      };
      fetch(0);
      fetch(1);
#pragma unroll
      for (int t = 0; t < kF32Slab / 16; ++t) {
        if (t + 2 < kF32Slab / 16) fetch(t + 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 16; ++q) acc = fmaf(a[t % 3][q / 4][q % 4], b[t % 3][q / 4][q % 4], acc);
      }
    } else {
      for (int i = 0; i < cnt; ++i) acc = fmaf(xc[i], wc[i], acc);
    }
  }
  if (r < nrows && j0 + c < N) {
    float* yo = y + (int64_t)(r0 + r) * N + j0 + c;
    *yo = accumulate ? *yo + acc : acc;
  }
}

}  // namespace

extern "C" {

retro_status retro_pack_weight(const void* w, int32_t k, int32_t n, void* w_packed,
                               void* stream) {
  if (!w || !w_packed || k <= 0 || n <= 0) return RETRO_EINVAL;
  if (!retro::aligned16(w_packed)) return RETRO_EINVAL;
  if (k % 32 != 0 || n % 16 != 0) return RETRO_EUNSUPPORTED;
  const int64_t groups = (int64_t)k * n / 8;
  const int threads = 256;
  const int64_t blocks = (groups + threads - 1) / threads;
  if (blocks > 0x7fffffff) return RETRO_EUNSUPPORTED;
  retro::pack_kernel<<<(unsigned)blocks, threads, 0, (hipStream_t)stream>>>(
      static_cast<const retro::bf16_t*>(w), k, n, static_cast<uint4*>(w_packed));
  return retro::status_of(hipGetLastError());
}

retro_status retro_project_qkv(const void* x, int32_t rows, int32_t k, const void* w_packed,
                               int32_t n_q, int32_t n_kv, void* q, void* k_out, void* v,
                               void* stream) {
  if (!x || !w_packed || !q || !k_out || !v || rows < 0 || k <= 0 || n_q <= 0 || n_kv <= 0)
    return RETRO_EINVAL;
  if (rows == 0) return RETRO_OK;
  if (!retro::aligned16(x) || !retro::aligned16(w_packed)) return RETRO_EINVAL;
  const int n = n_q + 2 * n_kv;
  if (!retro::proj_shape_ok(rows, k, n) || n_q % 16 != 0 || n_kv % 16 != 0)
    return RETRO_EUNSUPPORTED;
  retro::ProjArgs a{};
  a.x = x;
  a.w = static_cast<const uint4*>(w_packed);
  a.rows = rows;
  a.K = k;
  a.N = n;
  a.nq = n_q;
  a.nkv = n_kv;
  a.q = static_cast<retro::bf16_t*>(q);
  a.k = static_cast<retro::bf16_t*>(k_out);
  a.v = static_cast<retro::bf16_t*>(v);
  return retro::status_of(retro::launch_proj<false, false>(a, (hipStream_t)stream));
}

retro_status retro_project_out(const float* o, int32_t rows, int32_t k, const void* w_packed,
                               int32_t n, float* h, void* x_next, void* stream) {
  if (!o || !w_packed || !h || !x_next || rows < 0 || k <= 0 || n <= 0) return RETRO_EINVAL;
  if (rows == 0) return RETRO_OK;
  if (!retro::aligned16(o) || !retro::aligned16(w_packed)) return RETRO_EINVAL;
  if (!retro::proj_shape_ok(rows, k, n)) return RETRO_EUNSUPPORTED;
  retro::ProjArgs a{};
  a.x = o;
  a.w = static_cast<const uint4*>(w_packed);
  a.rows = rows;
  a.K = k;
  a.N = n;
  a.h = h;
  a.x_next = static_cast<retro::bf16_t*>(x_next);
  return retro::status_of(retro::launch_proj<true, false>(a, (hipStream_t)stream));
}

retro_status retro_project_f32(const float* x, int32_t rows, int32_t k, const float* w,
                               int32_t n, float* y, int32_t accumulate, void* stream) {
  if (!x || !w || !y || rows < 0 || k <= 0 || n <= 0) return RETRO_EINVAL;
  if (rows == 0) return RETRO_OK;
  if (rows > 65535 || (int64_t)rows * n >= (int64_t(1) << 31)) return RETRO_EUNSUPPORTED;
  const bool vec = n % 4 == 0 && retro::aligned16(w);
  auto go = [&](auto rb) {
    constexpr int RB = decltype(rb)::value;
    const dim3 grid((unsigned)((n + kF32Cols - 1) / kF32Cols), (unsigned)((rows + RB - 1) / RB));
    if (vec)
      project_f32_kernel<RB, true><<<grid, kF32Loaders + RB * kF32Cols, 0, (hipStream_t)stream>>>(
          x, rows, k, w, n, y, accumulate ? 1 : 0);
    else
      project_f32_kernel<RB, false><<<grid, kF32Loaders + RB * kF32Cols, 0, (hipStream_t)stream>>>(
          x, rows, k, w, n, y, accumulate ? 1 : 0);
  };
  // Blocks of eight rows, a quarter of the LDS reads per workgroup, where a compute
  // unit is left for each: 33 rows, 64 x 64 5.2 -> 4.4 us, 17 rows, 4096 x 1024 45 ->
  // 21; with more workgroups the weight's second reading costs more (70 rows, 4096 x
  // 1024 46 -> 54).
  const int64_t eights = (int64_t)((n + kF32Cols - 1) / kF32Cols) * ((rows + 7) / 8);
  if (rows <= 8 || eights <= retro::compute_units()) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 32>{});
  return retro::status_of(hipGetLastError());
}

}  // extern "C"
