// Grouped GEMMs over few rows per expert (decode and short prefill calls).
//
// With a handful of rows per expert the layer is bound by reading the expert
// weights once; the 256 x 256 tiles of gemm_core.h then run one latency-bound
// k loop per CU (T = 1, d = 1536, n = 256, E = 128, K = 8: 16 workgroups of 24
// dependent 64-deep steps, 26 us for 12.6 MB), and their M side stages 256 rows
// for the few that exist.  Here the weights stream straight into registers, and
// nothing but the final sum is shared between waves:
//   - A workgroup computes 128 columns of one expert for 16 MB rows; its KW
//     waves split the reduction (wave w takes steps w, w + KW, ... of 32 k), so
//     every wave is an independent stream of loads without barriers, and even
//     one row's weights are requested by many waves at once.
//   - Weights with k outer in memory (W1 and W2 in the forward): a lane loads
//     16 bytes (8 columns) of 8 consecutive k rows, whole 128- or 256-byte runs
//     per row, and transposes its 8 x 8 block with 32 v_perm_b32.  MFMA j
//     (16x16x32) then takes column 8 l + j of lane l: the columns of one MFMA
//     are 8 apart, which only permutes the accumulators, so a lane ends with
//     eight consecutive columns of four rows.
//   - The rows (k contiguous) are MFMA fragments as they lie in memory: 16
//     bytes per lane of a gathered row, no LDS.
//   - NBUF steps of loads are in flight per wave (8 KB of weights each).
//   - At the end the waves' accumulators meet in LDS, 16 rows at a time, and are
//     added in wave order by the epilogue.
#include <algorithm>

#include "device_common.h"
#include "launch.h"

namespace smoe {

// 8 rows (k) x 8 columns of bf16, one row per register quad -> per column the
// 8 k values (an MFMA operand)
__device__ __forceinline__ bf16x8 column_of(const u32x4 (&w)[8], int j) {
  const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
  u32x4 f;
#pragma unroll
  for (int p = 0; p < 4; ++p) f[p] = __builtin_amdgcn_perm(w[2 * p + 1][j >> 1], w[2 * p][j >> 1], sel);
  return __builtin_bit_cast(bf16x8, f);
}

constexpr int kStreamCols = 128;  // columns of a workgroup
typedef f32x4 StreamPart[16][2][16];  // one wave's 16 x 128 partial: [row][half of 8 columns][lane column]

// the sum over the waves of four consecutive columns, 4 c4 .. 4 c4 + 3 of the tile
template <int KW>
__device__ __forceinline__ f32x4 stream_sum(const StreamPart* part, int row, int c4) {
  f32x4 s = part[0][row][c4 & 1][c4 >> 1];
#pragma unroll
  for (int w = 1; w < KW; ++w) {
    const f32x4 v = part[w][row][c4 & 1][c4 >> 1];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] += v[q];
  }
  return s;
}

// The i-th further group (of `rows` rows; each expert's first is not counted, the
// others follow in expert order): its expert and first row.  False where there are
// no more than i.  Called by every thread of a workgroup of NT; lds: 18 words.
template <int NT>
__device__ __forceinline__ bool find_group(const int32_t* __restrict__ offsets, int E, int rows, int i, int* lds,
                                           int* expert, int* first_row) {
  constexpr int kOwn = 8;  // consecutive experts of a thread (E is a multiple of 8)
  if (i >= offsets[E] / rows) return false;  // (c rows have at most c / rows further groups)
  int* found = lds + 16;
  int base = 0;
  for (int e0 = 0; e0 < E; e0 += kOwn * NT) {
    const int e = e0 + kOwn * threadIdx.x;
    int n[kOwn], sum = 0;
    if (e < E) {
      int o[kOwn + 1];
#pragma unroll
      for (int q = 0; q <= kOwn; ++q) o[q] = offsets[e + q];
#pragma unroll
      for (int q = 0; q < kOwn; ++q) {
        n[q] = o[q + 1] > o[q] ? (o[q + 1] - o[q] - 1) / rows : 0;
        sum += n[q];
      }
    }
    int total;
    int at = base + block_excl_scan<NT>(sum, &total, lds);
    if (base + total > i) {  // here: one thread holds it
      if (at <= i && i < at + sum)
#pragma unroll
        for (int q = 0; q < kOwn; ++q) {
          if (at <= i && i < at + n[q]) {
            found[0] = e + q;
            found[1] = (i - at + 1) * rows;
          }
          at += n[q];
        }
      __syncthreads();
      *expert = __builtin_amdgcn_readfirstlane(found[0]);
      *first_row = __builtin_amdgcn_readfirstlane(found[1]);
      return true;
    }
    base += total;
  }
  return false;
}

// grid: x column tiles.  Router: y k slices, z groups of 16 MB rows.  Experts: y
// < E the first group of expert y, y >= E the experts' other groups, in expert
// order.  Most experts have one group, but with a skewed router a hot one has up
// to T rows; a workgroup past E finds its group in the sums of the experts'
// further groups (find_group), about 2 us beside the first groups' loads.
// (Eight workgroups per expert and tile that looped over its groups, most of them
// empty, ran a hot expert's groups one after the other: T = 1024, d = 1536, n =
// 256, E = 512, K = 8, Zipf 2: 207 us a forward call, now 134; balanced 291, 284.)
// Op supplies
//   EXPERTS: rows and groups by expert,
//   void rows(p, y, off, cnt): the rows [off, off + cnt),
//   int k0(p, y), int k(p, y): the reduction, a multiple of 32,
//   const uint16_t* x_row(p, row) (k contiguous from 0),
//   const uint16_t* w(p, y) with leading dimension ldw(p),
//   int col(p, tile, l): first of the eight columns of lane column l
//   template <int KW> void finish(p, y, tile, row0, rows, part): 16 rows
template <class Op, int MB, int KW, int NBUF, int OCC>
__global__ __launch_bounds__(64 * KW, OCC) void stream_gemm_kernel(const typename Op::Params p) {
  __shared__ StreamPart part[KW];
  const int tile = blockIdx.x;
  int e = blockIdx.y, m0 = blockIdx.z * 16 * MB;
  if constexpr (Op::EXPERTS)
    if (e >= p.E && !find_group<64 * KW>(p.offsets, p.E, 16 * MB, e - p.E, (int*)part, &e, &m0)) return;
  int off, cnt;
  Op::rows(p, e, off, cnt);
  if (m0 >= cnt) return;
  const int kbeg = Op::k0(p, e);
  const int lane = lane_id(), g = lane >> 4, l = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ns = (Op::k(p, e) / 32 - wave + KW - 1) / KW;  // this wave's steps
  const uint16_t* wbase = Op::w(p, e);
  const uint32_t ldw = Op::ldw(p);
  const uint32_t wcol = Op::col(p, tile, l);
  const uint16_t* xp[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) xp[b] = Op::x_row(p, off + min(m0 + 16 * b + l, cnt - 1)) + 8 * g;
  f32x4 acc[MB][8];
#pragma unroll
  for (int b = 0; b < MB; ++b)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 wv[NBUF][8];
  bf16x8 xv[NBUF][MB];
  // step s of this wave; a step past the end reads the step 0 addresses (cached, unused)
  auto load = [&](int buf, int s) {
    const uint32_t k = kbeg + 32 * (s < ns ? wave + KW * s : wave);
    const uint32_t o = (k + 8 * g) * ldw + wcol;
#pragma unroll
    for (int i = 0; i < 8; ++i) wv[buf][i] = *(const u32x4*)(wbase + (size_t)(o + i * ldw));
#pragma unroll
    for (int b = 0; b < MB; ++b) xv[buf][b] = *(const bf16x8*)(xp[b] + k);
  };
  if (ns > 0) {
#pragma unroll
    for (int q = 0; q < NBUF; ++q) load(q, q);
    for (int s = 0;; s += NBUF) {
#pragma unroll
      for (int q = 0; q < NBUF; ++q) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bf16x8 wf = column_of(wv[q], j);
#pragma unroll
          for (int b = 0; b < MB; ++b)
            acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[q][b], wf, acc[b][j], 0, 0, 0);
        }
        if (s + q + 1 >= ns) goto done;
        load(q, s + q + NBUF);
      }
    }
  done:;
  }
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    if (m0 + 16 * b >= cnt) break;
    __syncthreads();  // the previous rows' sums have been read
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        part[wave][4 * g + r][h][l] =
            f32x4{acc[b][4 * h][r], acc[b][4 * h + 1][r], acc[b][4 * h + 2][r], acc[b][4 * h + 3][r]};
    __syncthreads();
    Op::template finish<KW>(p, e, tile, off + m0 + 16 * b, min(16, cnt - m0 - 16 * b), part);
  }
}

// rows of the routing: expert y's
template <class Params>
__device__ __forceinline__ void expert_rows(const Params& p, int y, int& off, int& cnt) {
  off = p.offsets[y];
  cnt = p.offsets[y + 1] - off;
}

// H = gather(X) W1_e (+ b1_e), A = SwiGLU(H): 64 gate columns (lane columns
// 0..7) and the matching up columns (8..15)
struct StreamUp {
  using Params = UpArgs;
  static constexpr bool EXPERTS = true;
  static __device__ void rows(const Params& p, int y, int& off, int& cnt) { expert_rows(p, y, off, cnt); }
  static __device__ int k0(const Params&, int) { return 0; }
  static __device__ int k(const Params& p, int) { return p.d; }
  static __device__ const uint16_t* x_row(const Params& p, int row) { return p.X + (size_t)p.row_token[row] * p.d; }
  static __device__ const uint16_t* w(const Params& p, int e) { return p.W1 + (size_t)e * p.d * (2 * p.n); }
  static __device__ uint32_t ldw(const Params& p) { return 2 * p.n; }
  static __device__ uint32_t col(const Params& p, int tile, int l) {
    return (l < 8 ? 0 : p.n) + 64 * tile + 8 * (l & 7);
  }
  template <int KW>
  static __device__ void finish(const Params& p, int e, int tile, int row0, int rows, const StreamPart* part) {
    for (int i = threadIdx.x; i < 256; i += 64 * KW) {
      const int row = i >> 4, c4 = i & 15;
      if (row >= rows) break;
      f32x4 hg = stream_sum<KW>(part, row, c4), hu = stream_sum<KW>(part, row, c4 + 16);
      const int c = 64 * tile + 4 * c4;
      if (p.b1) {
        const float* b = p.b1 + (size_t)e * 2 * p.n + c;
        const f32x4 bg = *(const f32x4*)b, bu = *(const f32x4*)(b + p.n);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          hg[q] += bg[q];
          hu[q] += bu[q];
        }
      }
      float a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float sg;
        a[q] = silu_sig(hg[q], &sg) * hu[q];
      }
      uint16_t* h = p.H + (size_t)(row0 + row) * (2 * p.n) + c;
      *(u32x2*)h = pack_bf16x4(hg[0], hg[1], hg[2], hg[3]);
      *(u32x2*)(h + p.n) = pack_bf16x4(hu[0], hu[1], hu[2], hu[3]);
      *(u32x2*)(p.A + (size_t)(row0 + row) * p.n + c) = pack_bf16x4(a[0], a[1], a[2], a[3]);
    }
  }
};

// Y = A W2_e (+ b2_e); AGG: how Y leaves (0: Y rows expert-major; 1 and 2: the
// aggregation ablation's scatter to p.dst[row] and fp32 atomics, as OpDown)
template <int AGG>
struct StreamDown {
  using Params = DownArgs;
  static constexpr bool EXPERTS = true;
  static __device__ void rows(const Params& p, int y, int& off, int& cnt) { expert_rows(p, y, off, cnt); }
  static __device__ int k0(const Params&, int) { return 0; }
  static __device__ int k(const Params& p, int) { return p.n; }
  static __device__ const uint16_t* x_row(const Params& p, int row) { return p.A + (size_t)row * p.n; }
  static __device__ const uint16_t* w(const Params& p, int e) { return p.W2 + (size_t)e * p.n * p.d; }
  static __device__ uint32_t ldw(const Params& p) { return p.d; }
  static __device__ uint32_t col(const Params& p, int tile, int l) { return kStreamCols * tile + 8 * l; }
  template <int KW>
  static __device__ void finish(const Params& p, int e, int tile, int row0, int rows, const StreamPart* part) {
    for (int i = threadIdx.x; i < 512; i += 64 * KW) {
      const int row = i >> 5, c4 = i & 31;
      if (row >= rows) break;
      f32x4 y = stream_sum<KW>(part, row, c4);
      const int c = kStreamCols * tile + 4 * c4;
      if (p.b2) {
        const f32x4 b = *(const f32x4*)(p.b2 + (size_t)e * p.d + c);
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] += b[q];
      }
      const u32x2 v = pack_bf16x4(y[0], y[1], y[2], y[3]);
      const int r = row0 + row;
      if constexpr (AGG == 2) {
        float* o = p.O32 + (size_t)p.row_token[r] * p.d + c;
        const float s = p.row_w[r];
        unsafeAtomicAdd(o, s * bf_lo(v[0]));
        unsafeAtomicAdd(o + 1, s * bf_hi(v[0]));
        unsafeAtomicAdd(o + 2, s * bf_lo(v[1]));
        unsafeAtomicAdd(o + 3, s * bf_hi(v[1]));
      } else {
        *(u32x2*)(p.Y + (size_t)(AGG == 1 ? p.dst[r] : r) * p.d + c) = v;
      }
    }
  }
};

// Row blocks per workgroup.  (up + down) streaming / tiled, with mb = 1 | mb = 2, for
// balanced experts and for a router skewed by Zipf exponents 0.5 to 2 (the worst):
//                                            mean 2       8            12           16
//   d = 1024, n = 256, E = 64, K = 8         .84|.83      .91|.89      1.12|.92     1.20|.95
//     skewed                                 .81|.80      1.15|1.01    1.15|1.10    1.16|1.08
//   d = 1536, n = 256, E = 256, K = 8        .78|.79      .91|.86      .97|.89      1.20|.90
//     skewed                                 .85|.81      1.08|.97     1.17|.99     1.42|1.11
//   d = 1024, n = 128, E = 1024, K = 8       .74|.75      .80|.78      .88|.80      1.11|.84
//     skewed                                 .76|.79      1.24|1.01    1.41|1.08    1.65|1.22
//   d = 4096, n = 512, E = 128, K = 8        .90|.90      1.03|.95     1.10|.95     1.36|.97
//     skewed                                 .89|.93      1.10|1.03    1.21|1.07    1.26|1.09
//   d = 1024, n = 256, E = 16, K = 8         .61|.63      .59|.63      .67|.69      .69|.70
//     skewed                                 .66|.67      .62|.68      .72|.71      .75|.72
// An expert with more rows than a group has its weights read again per group, so
// two row blocks are the better ones from a few rows per expert on, skewed or not
// (with at most 16 tokens no expert fills a second).  Up to 12 rows per expert
// streaming is the faster one and a skewed router costs it little; up to 20 it
// depends on the skew, more so the more tokens a hot expert can have (T = 2048 in
// the third line: 69 us against 57).  Beyond, and for more tokens, the tiled GEMMs
// are taken, except where they have too few tiles for the CUs:
//   d = 1536, n = 1024, E = 16, K = 2, T = 256, mean 32   up 29 / 41   down 18 / 25
// A rounded routing's experts have no rows or m_tile and more, whatever the mean:
//   T = 512, d = 1536, n = 256, E = 256, K = 8 (mean 16), rounded up to 256:
//   forward call 1088 us streaming, 350 tiled; d = 4096, n = 512, up to 128: 2923, 826
StreamShape stream_shape(const moe_dims& m, int capacity, int m_tile, int64_t tiles_per_expert) {
  const StreamShape tiled{0, 0};
  if ((int64_t)m.d * 2 * m.n > INT32_MAX) return tiled;  // 32-bit offsets within an expert's weights
  const int64_t mean = std::max<int64_t>(((int64_t)m.T * m.K + m.E - 1) / m.E, m_tile);
  const bool few_tiles = m.E * tiles_per_expert < 192;
  int mb;
  if (m.T <= 16 || mean <= 2)
    mb = 1;
  else if (mean <= (few_tiles || m.T <= 2048 ? 20 : 12))
    mb = 2;
  else if (mean <= 64 && few_tiles)
    mb = 4;
  else
    return tiled;
  // further groups of at most `capacity` rows over experts of at most T
  const int64_t rows = 16 * mb, further = std::min(capacity / rows, m.E * ((m.T - 1) / rows));
  return m.E + further <= 65535 ? StreamShape{mb, (int)further} : tiled;
}

// Partial router logits of k slice y: part[y][t][e] = sum over the slice of X W_r
struct StreamRouter {
  using Params = RouterPartArgs;
  static constexpr bool EXPERTS = false;
  static __device__ void rows(const Params& p, int, int& off, int& cnt) {
    off = 0;
    cnt = p.T;
  }
  static __device__ int k0(const Params& p, int y) { return y * p.slice; }
  static __device__ int k(const Params& p, int y) { return min(p.slice, p.d - y * p.slice); }
  static __device__ const uint16_t* x_row(const Params& p, int row) { return p.X + (size_t)row * p.d; }
  static __device__ const uint16_t* w(const Params& p, int) { return p.Wr; }
  static __device__ uint32_t ldw(const Params& p) { return p.E; }
  // (lane columns past E, a multiple of 8, re-read the last ones)
  static __device__ uint32_t col(const Params& p, int tile, int l) { return min(kStreamCols * tile + 8 * l, p.E - 8); }
  template <int KW>
  static __device__ void finish(const Params& p, int y, int tile, int row0, int rows, const StreamPart* part) {
    for (int i = threadIdx.x; i < 512; i += 64 * KW) {
      const int row = i >> 5, c4 = i & 31, c = kStreamCols * tile + 4 * c4;
      if (row >= rows) break;
      if (c < p.E) *(f32x4*)(p.part + ((size_t)y * p.T + row0 + row) * p.E + c) = stream_sum<KW>(part, row, c4);
    }
  }
};

// Waves and steps of loads in flight of the row blocks, within the registers (no
// spills): up to eight waves share the k / 32 steps.  From k = 768 on every wave has
// three or more; k = 256 is one step for each of eight waves, below 256 some of them
// have none, and a second buffer then re-reads the first step (cached, unused).  A
// short k (the down-projection of a narrow expert) has two waves with a step or two
// each (T = 65, d = 1664, n = 64, E = 312, K = 8: down 26 us with eight waves, six of
// them idle, 13 with two).
template <class Op>
static hipError_t run_stream(const typename Op::Params& p, dim3 grid, int mb, int k, hipStream_t s) {
  if (mb == 1 && k >= 768)
    stream_gemm_kernel<Op, 1, 8, 3, 2><<<grid, dim3(512), 0, s>>>(p);
  else if (mb == 1 && k > 128)
    stream_gemm_kernel<Op, 1, 8, 2, 4><<<grid, dim3(512), 0, s>>>(p);
  else if (mb == 1)
    stream_gemm_kernel<Op, 1, 2, 2, 3><<<grid, dim3(128), 0, s>>>(p);
  else if (mb == 2 && k <= 128)
    stream_gemm_kernel<Op, 2, 2, 1, 3><<<grid, dim3(128), 0, s>>>(p);
  else if (mb == 2)
    stream_gemm_kernel<Op, 2, 4, 2, 2><<<grid, dim3(256), 0, s>>>(p);
  else
    stream_gemm_kernel<Op, 4, 4, 1, 2><<<grid, dim3(256), 0, s>>>(p);
  return hipGetLastError();
}

static dim3 stream_grid(int tiles, int E, const StreamShape& t) { return dim3(tiles, E + t.further); }

hipError_t launch_stream_up(const UpArgs& a, const StreamShape& t, hipStream_t s) {
  return run_stream<StreamUp>(a, stream_grid(a.n / 64, a.E, t), t.mb, a.d, s);
}
hipError_t launch_stream_down(const DownArgs& a, int strategy, const StreamShape& t, hipStream_t s) {
  const dim3 grid = stream_grid(a.d / kStreamCols, a.E, t);
  if (strategy == MOE_AGG_SCATTER_SUM) return run_stream<StreamDown<1>>(a, grid, t.mb, a.n, s);
  if (strategy == MOE_AGG_ATOMIC_F32) return run_stream<StreamDown<2>>(a, grid, t.mb, a.n, s);
  return run_stream<StreamDown<0>>(a, grid, t.mb, a.n, s);
}

// Row blocks of the router's workgroups: one (16 tokens) while that gives up to
// two workgroups per CU, more as W_r would otherwise be re-read too often.
static int router_row_blocks(int T, int E, int* groups) {
  const int tiles = (E + kStreamCols - 1) / kStreamCols;
  for (int mb = 1;; mb *= 2) {
    *groups = (T + 16 * mb - 1) / (16 * mb);
    if (mb == 4 || tiles * *groups <= 512) return mb;
  }
}

int router_slices(int T, int d, int E, size_t part_bytes) {
  int groups;
  router_row_blocks(T, E, &groups);
  const int steps = d / 32, wgs = (E + kStreamCols - 1) / kStreamCols * groups;
  // about one workgroup per two CUs, two or more steps for each of eight waves
  const int64_t fit = part_bytes / ((size_t)T * E * 4);
  const int want = std::min({128 / wgs, steps / 16, (int)std::min<int64_t>(fit, 64)});
  if (want <= 1) return 1;
  const int per = (steps + want - 1) / want;  // steps of a slice
  return (steps + per - 1) / per;
}

hipError_t launch_router_part(const uint16_t* X, const uint16_t* Wr, float* part, int slices, int T, int d, int E,
                              hipStream_t s) {
  const int steps = d / 32, slice = 32 * ((steps + slices - 1) / slices);
  int groups;
  const int mb = router_row_blocks(T, E, &groups);
  const dim3 grid((E + kStreamCols - 1) / kStreamCols, slices, groups);
  return run_stream<StreamRouter>({X, Wr, part, T, d, E, slice}, grid, mb, slice, s);
}

}  // namespace smoe
