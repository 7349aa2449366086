// Expert aggregation (gather-and-sum) and the small helper kernels.
//
// Forward O kernel (Section 3, forward algorithm): every token gathers its
// experts' Y rows and sums them weighted by the routing scores.  Backward dX
// kernel (Appendix E, up-projection backward): the same gather-and-sum over
// dX~ rows, with the router's gradient term fused in.  Each token is owned by
// one wave, so the sum order is fixed and no atomics are used (the paper's
// gather-and-sum choice keeps the result deterministic).
#include "device_common.h"
#include "launch.h"

namespace smoe {

constexpr int kAggBatch = 8;  // rows whose loads are in flight together
constexpr int kDLPerLane = 4;  // router-gradient row entries per lane collected in registers (E <= 256)
static_assert(kAggBatch == 8, "lane & 7 picks a batch slot");

__device__ __forceinline__ int bcast_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float bcast_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// One wave per token; lanes cover 8 consecutive bf16 (16 bytes) of the row,
// in NC chunks of 512 columns of the workgroup's column slice (rows wider than
// 2048 columns are cut into slices; neighbouring workgroups take the slices of
// the same tokens, so a row's pieces are read at about the same time).  The
// token's rows are taken kAggBatch at a time
// without branches: lanes 0..7 fetch the batch's row indices and weights
// (padding slots clamped to the token's last row, weight 0) and broadcast
// them, then the row loads of every chunk are issued before any is
// accumulated, so a lane keeps NC * kAggBatch HBM reads in flight.  Every Y
// row is read exactly once and O is not read again here: both go through the
// caches as nontemporal accesses.
// CONTIG (the aggregation ablation's scatter + sum): Y holds the rows in
// token-major order, so the token's rows are Y[j0 .. j1) themselves.
template <int NC, bool CONTIG = false>
__global__ __launch_bounds__(256) void agg_o_kernel(const uint16_t* __restrict__ Y, const int32_t* __restrict__ tok_offsets,
                                                    const int32_t* __restrict__ tok_rows, const float* __restrict__ row_w,
                                                    uint16_t* __restrict__ O, int T, int d, int slices) {
  const int c0 = blockIdx.x % slices * (512 * NC);  // this workgroup's column slice
  // wave-uniform token: row indices and weights become scalar loads
  const int t = blockIdx.x / slices * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= T) return;
  const int lane = lane_id();
  const int j0 = tok_offsets[t], j1 = tok_offsets[t + 1];
  float acc[NC][8];
#pragma unroll
  for (int ci = 0; ci < NC; ++ci)
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[ci][q] = 0.f;
  for (int jb = j0; jb < j1; jb += kAggBatch) {
    const int slot = jb + (lane & 7);
    const int rl = tok_rows[min(slot, j1 - 1)];
    const float wl = slot < j1 ? row_w[rl] : 0.f;
    int r[kAggBatch];
    float w[kAggBatch];
#pragma unroll
    for (int u = 0; u < kAggBatch; ++u) {
      r[u] = CONTIG ? min(jb + u, j1 - 1) : bcast_i(rl, u);
      w[u] = bcast_f(wl, u);
    }
    u32x4 v[NC][kAggBatch];
#pragma unroll
    for (int ci = 0; ci < NC; ++ci) {
      const int c = min(c0 + lane * 8 + 512 * ci, d - 8);  // lanes past the row end re-read its last chunk
#pragma unroll
      for (int u = 0; u < kAggBatch; ++u) v[ci][u] = __builtin_nontemporal_load((const u32x4*)(Y + (size_t)r[u] * d + c));
    }
#pragma unroll
    for (int ci = 0; ci < NC; ++ci)
#pragma unroll
      for (int u = 0; u < kAggBatch; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[ci][2 * q] += w[u] * bf_lo(v[ci][u][q]);
          acc[ci][2 * q + 1] += w[u] * bf_hi(v[ci][u][q]);
        }
  }
#pragma unroll
  for (int ci = 0; ci < NC; ++ci) {
    const int c = c0 + lane * 8 + 512 * ci;
    if (c < d) {
      u32x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = pack_bf2(acc[ci][2 * q], acc[ci][2 * q + 1]);
      __builtin_nontemporal_store(o, (u32x4*)(O + (size_t)t * d + c));
    }
  }
}

// dX_t = sum over the token's rows of dX~ + sum_j dl_j W_r[:, e_j], with the
// router gradient on the token's selected set dl_j = s_j (dS_j - sum_k s_k dS_k).
// Also writes the dense router-logit gradient row dL[t, :] (bf16) for dW_r
// (when dL is given; the workgroups of column slice 0 do it).
// W_r^T [E][d] is a bf16 copy (exact: W_r is bf16), so each row term is one
// 16-byte load per lane.  As in the forward kernel, a batch's dX~ rows are
// requested for every column chunk before any is accumulated; the W_r^T rows
// (a few hundred KB, cache resident) follow chunk by chunk.
template <int NC>
__global__ __launch_bounds__(256) void agg_dx_kernel(const uint16_t* __restrict__ dXt, const float* __restrict__ dS, int ds_parts,
                                                     const uint16_t* __restrict__ WrT,
                                                     const int32_t* __restrict__ tok_offsets,
                                                     const int32_t* __restrict__ tok_rows,
                                                     const int32_t* __restrict__ row_expert,
                                                     const float* __restrict__ row_w, uint16_t* __restrict__ dX,
                                                     uint16_t* __restrict__ dL_, int T, int d, int E, int slices) {
  const int c0 = blockIdx.x % slices * (512 * NC);  // this workgroup's column slice
  uint16_t* const dL = c0 == 0 ? dL_ : nullptr;  // written by the first slice
  // wave-uniform token: row indices and weights become scalar loads
  const int t = blockIdx.x / slices * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= T) return;
  const int lane = lane_id();
  const int j0 = tok_offsets[t], j1 = tok_offsets[t + 1];
  auto ds_of = [&](int r) {  // dS of a row: its partial sums in order
    float v = dS[(size_t)r * ds_parts];
    for (int k = 1; k < ds_parts; ++k) v += dS[(size_t)r * ds_parts + k];
    return v;
  };
  // g = sum_k s_k dS_k in row order; lanes 0..7 fetch a batch's terms.  A
  // token whose rows fit one batch (every token-choice token with K <= 8,
  // most rounded ones) forms g in the main loop's only iteration instead, from
  // the weights and dS values that iteration loads anyway: one round trip of
  // dependent loads fewer before its dX~ rows are requested.
  const bool one_batch = j1 - j0 <= kAggBatch;
  float g = 0.f;
  if (WrT && !one_batch)
    for (int jb = j0; jb < j1; jb += kAggBatch) {
      const int slot = jb + (lane & 7);
      const int rl = tok_rows[min(slot, j1 - 1)];
      const float pl = slot < j1 ? row_w[rl] * ds_of(rl) : 0.f;
#pragma unroll
      for (int u = 0; u < kAggBatch; ++u) g += bcast_f(pl, u);
    }
  // dL[t, e] for e = lane + 64 q (q < kDLPerLane), collected from the batches
  const bool dl_fast = dL != nullptr && E <= 64 * kDLPerLane;
  float dlv[kDLPerLane] = {0.f, 0.f, 0.f, 0.f};
  float acc[NC][8];
#pragma unroll
  for (int ci = 0; ci < NC; ++ci)
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[ci][q] = 0.f;
  for (int jb = j0; jb < j1; jb += kAggBatch) {
    // slot lane&7 of the batch: one vector load per level, then broadcast
    const int slot = jb + (lane & 7);
    const int rl = tok_rows[min(slot, j1 - 1)];
    const int el = WrT ? row_expert[rl] : 0;
    if (WrT && one_batch) {
      const float pl = slot < j1 ? row_w[rl] * ds_of(rl) : 0.f;
#pragma unroll
      for (int u = 0; u < kAggBatch; ++u) g += bcast_f(pl, u);
    }
    const float dll = (WrT && slot < j1) ? row_w[rl] * (ds_of(rl) - g) : 0.f;
    int r[kAggBatch];
#pragma unroll
    for (int u = 0; u < kAggBatch; ++u) r[u] = bcast_i(rl, u);
    u32x4 v[NC][kAggBatch];
#pragma unroll
    for (int ci = 0; ci < NC; ++ci) {
      const int c = min(c0 + lane * 8 + 512 * ci, d - 8);  // lanes past the row end re-read its last chunk
#pragma unroll
      for (int u = 0; u < kAggBatch; ++u) v[ci][u] = __builtin_nontemporal_load((const u32x4*)(dXt + (size_t)r[u] * d + c));
    }
    float keep[kAggBatch];
#pragma unroll
    for (int u = 0; u < kAggBatch; ++u) keep[u] = jb + u < j1 ? 1.f : 0.f;  // padding slots re-read the last row
#pragma unroll
    for (int ci = 0; ci < NC; ++ci)
#pragma unroll
      for (int u = 0; u < kAggBatch; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[ci][2 * q] += keep[u] * bf_lo(v[ci][u][q]);
          acc[ci][2 * q + 1] += keep[u] * bf_hi(v[ci][u][q]);
        }
    if (WrT) {
#pragma unroll
      for (int ci = 0; ci < NC; ++ci) {
        const int c = min(c0 + lane * 8 + 512 * ci, d - 8);
        u32x4 wv[kAggBatch];
#pragma unroll
        for (int u = 0; u < kAggBatch; ++u) wv[u] = *(const u32x4*)(WrT + (size_t)bcast_i(el, u) * d + c);
#pragma unroll
        for (int u = 0; u < kAggBatch; ++u) {
          const float dl = bcast_f(dll, u);  // 0 for padding slots
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            acc[ci][2 * q] += dl * bf_lo(wv[u][q]);
            acc[ci][2 * q + 1] += dl * bf_hi(wv[u][q]);
          }
        }
      }
      if (dl_fast)
#pragma unroll
        for (int u = 0; u < kAggBatch; ++u) {
          const int e = bcast_i(el, u);
          const float dl = bcast_f(dll, u);
#pragma unroll
          for (int q = 0; q < kDLPerLane; ++q)
            if (jb + u < j1 && e == lane + 64 * q) dlv[q] = dl;
        }
    }
  }
#pragma unroll
  for (int ci = 0; ci < NC; ++ci) {
    const int c = c0 + lane * 8 + 512 * ci;
    if (c < d) {
      u32x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = pack_bf2(acc[ci][2 * q], acc[ci][2 * q + 1]);
      __builtin_nontemporal_store(o, (u32x4*)(dX + (size_t)t * d + c));
    }
  }
  if (dl_fast) {
#pragma unroll
    for (int q = 0; q < kDLPerLane; ++q)
      if (lane + 64 * q < E) dL[(size_t)t * E + lane + 64 * q] = f2bf(dlv[q]);
  } else if (dL) {
    for (int e = lane; e < E; e += 64) {
      float v = 0.f;
      for (int j = j0; j < j1; ++j) {
        const int r = tok_rows[j];
        if (row_expert[r] == e) v = row_w[r] * (ds_of(r) - g);
      }
      dL[(size_t)t * E + e] = f2bf(v);
    }
  }
}

// out[i] = sum_k part[i * parts + k] (fixed order)
__global__ __launch_bounds__(256) void reduce_rowparts_kernel(const float* __restrict__ part, float* __restrict__ out,
                                                              int n, int parts) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  for (int k = 0; k < parts; ++k) s += part[(size_t)i * parts + k];
  out[i] = s;
}

// ---------------------------------------------------------------- expert biases
// B2s[k][e] = hi(b2[e][k]) and B2s[k][E + e] = bf16(b2[e][k] - hi), hi = the
// round-to-nearest bf16 of b2[e][k]: the layout of W_r [d][E'] with E' = 2E,
// so the router GEMM forms dO B2s, i.e. <dO_t, hi_e> and <dO_t, lo_e>.
__global__ __launch_bounds__(256) void bias_split_kernel(const float* __restrict__ b2, int E, int d,
                                                         uint16_t* __restrict__ B2s) {
  const int i = blockIdx.x * 256 + threadIdx.x;  // over d x E, e fastest
  if (i >= d * E) return;
  const int k = i / E, e = i % E;
  const float v = b2[(size_t)e * d + k];
  const uint16_t hi = f2bf(v);
  B2s[(size_t)k * 2 * E + e] = hi;
  B2s[(size_t)k * 2 * E + E + e] = f2bf(v - bf2f(hi));
}

// The expert-bias gradients db1 (columns of dH) and db2 (columns of s * dO) in
// two launches.  They are bound by the latency of the row loads: a single
// workgroup that walks an expert's rows has one batch of loads in flight at a
// time (T = 5003, d = 896, n = 192, E = 40, K = 3, one workgroup of four waves
// per expert and 512 columns: 117 and 90 us for 17 MB).  So the rows are cut
// along the backward's m-tile list: one workgroup per m-tile and 512 columns,
// eight waves with eight rows each in flight, wave w on rows w, w + 8, ...;
// the waves' sums are added in wave order through LDS.  The second kernel adds
// an expert's tiles in row order, so nothing depends on timing.
constexpr int kColsumWaves = 8;
struct ColsumSrc {
  const uint16_t* src;
  int cols;               // columns summed, and the leading dimension of src; 0: not asked for
  const int32_t* token;   // gathered rows, or null
  const float* w;         // row weights, or null
};
__global__ __launch_bounds__(64 * kColsumWaves) void tile_colsum_kernel(const int32_t* __restrict__ mtiles, ColsumSrc s1,
                                                                       ColsumSrc s2, int ny1,
                                                                       float* __restrict__ part) {
  __shared__ float red[kColsumWaves][512];
  const int tile = blockIdx.x;
  if (tile >= mtiles[0]) return;
  const bool second = (int)blockIdx.y >= ny1;
  const ColsumSrc s = second ? s2 : s1;
  const int chunk = second ? blockIdx.y - ny1 : blockIdx.y;
  const int nrows = mtiles[4 + 4 * tile + 2], r0 = mtiles[4 + 4 * tile + 3], r1 = r0 + nrows;
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int c = chunk * 512 + lane * 8;
  const bool live = c < s.cols;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int kU = 8;
  for (int rb = r0 + wave; rb < r1; rb += kColsumWaves * kU) {
    u32x4 v[kU];
    float w[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int r = rb + u * kColsumWaves;
      const bool ok = r < r1 && live;
      const int g = ok ? (s.token ? s.token[r] : r) : 0;
      w[u] = ok ? (s.w ? s.w[r] : 1.f) : 0.f;
      v[u] = ok ? *(const u32x4*)(s.src + (size_t)g * s.cols + c) : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc[2 * q] += w[u] * bf_lo(v[u][q]);
        acc[2 * q + 1] += w[u] * bf_hi(v[u][q]);
      }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) red[wave][lane * 8 + q] = acc[q];
  __syncthreads();
  const int cc = chunk * 512 + threadIdx.x;  // one column per thread
  if (cc >= s.cols) return;
  float t = 0.f;
#pragma unroll
  for (int w2 = 0; w2 < kColsumWaves; ++w2) t += red[w2][threadIdx.x];
  part[(size_t)tile * (s1.cols + s2.cols) + (second ? s1.cols : 0) + cc] = t;
}

// out[e][c] = the sum of expert e's tiles: its full tiles, contiguous in the
// list, then its partial one (after every expert's full tiles).  Experts
// without rows get zeros.
__global__ __launch_bounds__(256) void colsum_reduce_kernel(const int32_t* __restrict__ mtiles,
                                                            const int32_t* __restrict__ offsets,
                                                            const float* __restrict__ part, int mtile, int cols1,
                                                            int cols2, float* __restrict__ out1,
                                                            float* __restrict__ out2) {
  __shared__ int red[2][4];
  const int e = blockIdx.x;
  int nf = 0, np = 0;  // tiles of the experts before e
  for (int i = threadIdx.x; i < e; i += 256) {
    const int cnt = offsets[i + 1] - offsets[i];
    nf += cnt / mtile;
    np += cnt % mtile != 0;
  }
  nf = wave_sum_i(nf);
  np = wave_sum_i(np);
  if (lane_id() == 0) {
    red[0][threadIdx.x >> 6] = nf;
    red[1][threadIdx.x >> 6] = np;
  }
  __syncthreads();
  const int first = red[0][0] + red[0][1] + red[0][2] + red[0][3];
  const int last = mtiles[0] - mtiles[1] + red[1][0] + red[1][1] + red[1][2] + red[1][3];
  const int c = blockIdx.y * 256 + threadIdx.x, cols = cols1 + cols2;
  if (c >= cols) return;
  const int cnt = offsets[e + 1] - offsets[e];
  const float* p = part + (size_t)first * cols + c;
  float t = 0.f;
#pragma unroll 8
  for (int i = 0; i < cnt / mtile; ++i) t += p[(size_t)i * cols];
  if (cnt % mtile) t += part[(size_t)last * cols + c];
  if (c < cols1)
    out1[(size_t)e * cols1 + c] = t;
  else
    out2[(size_t)e * cols2 + c - cols1] = t;
}

hipError_t launch_bias_split(const float* b2, int E, int d, uint16_t* B2s, hipStream_t s) {
  bias_split_kernel<<<dim3((d * E + 255) / 256), dim3(256), 0, s>>>(b2, E, d, B2s);
  return hipGetLastError();
}

hipError_t launch_expert_colsum(const ExpertColsumArgs& a, hipStream_t s) {
  const int c1 = a.db1 ? 2 * a.n : 0, c2 = a.db2 ? a.d : 0;
  const int ny1 = (c1 + 511) / 512, ny2 = (c2 + 511) / 512;
  const int tiles = a.capacity / kMTile + a.E;  // bound of the list's length
  tile_colsum_kernel<<<dim3(tiles, ny1 + ny2), dim3(64 * kColsumWaves), 0, s>>>(
      a.mtiles, {a.dH, c1, nullptr, nullptr}, {a.dO, c2, a.row_token, a.row_w}, ny1, a.part);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  colsum_reduce_kernel<<<dim3(a.E, (c1 + c2 + 255) / 256), dim3(256), 0, s>>>(a.mtiles, a.offsets, a.part, kMTile, c1,
                                                                              c2, a.db1, a.db2);
  return hipGetLastError();
}

// slices of at most four 512-column chunks, as equal as they go
static int agg_slices(int d) { return ((d + 511) / 512 + 3) / 4; }

template <bool CONTIG>
static hipError_t run_agg_o(const uint16_t* Y, const moe_routing& r, uint16_t* O, int T, int d, hipStream_t s) {
  const int slices = agg_slices(d), nc = ((d + 511) / 512 + slices - 1) / slices;
  const dim3 grid((unsigned)((T + 3) / 4) * slices), block(256);
#define SMOE_AGG(N) \
  if (nc == N) agg_o_kernel<N, CONTIG><<<grid, block, 0, s>>>(Y, r.tok_offsets, r.tok_rows, r.row_w, O, T, d, slices)
  SMOE_AGG(1);
  SMOE_AGG(2);
  SMOE_AGG(3);
  SMOE_AGG(4);
#undef SMOE_AGG
  return hipGetLastError();
}

hipError_t launch_agg_o(const uint16_t* Y, const moe_routing& r, uint16_t* O, int T, int d, hipStream_t s) {
  return run_agg_o<false>(Y, r, O, T, d, s);
}

hipError_t launch_agg_o_contig(const uint16_t* Yt, const moe_routing& r, uint16_t* O, int T, int d, hipStream_t s) {
  return run_agg_o<true>(Yt, r, O, T, d, s);
}

// dst[tok_rows[j]] = j for the j < tok_offsets[T] (token-major slot of each row)
__global__ __launch_bounds__(256) void tok_slots_kernel(const int32_t* __restrict__ tok_offsets,
                                                        const int32_t* __restrict__ tok_rows, int T, int n,
                                                        int32_t* __restrict__ dst) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j < n && j < tok_offsets[T]) dst[tok_rows[j]] = j;
}

__global__ __launch_bounds__(256) void fill_f32_kernel(float* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0.f;
}

__global__ __launch_bounds__(256) void f32_to_bf16_kernel(const float* __restrict__ in, uint16_t* __restrict__ out,
                                                          size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) out[i] = f2bf(in[i]);
}

hipError_t launch_tok_slots(const moe_routing& r, int T, int P_bound, int32_t* dst, hipStream_t s) {
  if (P_bound > 0) tok_slots_kernel<<<dim3((P_bound + 255) / 256), dim3(256), 0, s>>>(r.tok_offsets, r.tok_rows, T,
                                                                                     P_bound, dst);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, size_t n, hipStream_t s) {
  fill_f32_kernel<<<dim3(2048), dim3(256), 0, s>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_f32_to_bf16(const float* in, uint16_t* out, size_t n, hipStream_t s) {
  f32_to_bf16_kernel<<<dim3(2048), dim3(256), 0, s>>>(in, out, n);
  return hipGetLastError();
}

hipError_t launch_agg_dx(const uint16_t* dXt, const float* dS, int ds_parts, const uint16_t* WrT, const moe_routing& r, uint16_t* dX,
                         uint16_t* dL, int T, int d, int E, hipStream_t s) {
  const int slices = agg_slices(d), nc = ((d + 511) / 512 + slices - 1) / slices;
  const dim3 grid((unsigned)((T + 3) / 4) * slices), block(256);
#define SMOE_AGG(N)                                                                                                   \
  if (nc == N)                                                                                                        \
  agg_dx_kernel<N><<<grid, block, 0, s>>>(dXt, dS, ds_parts, WrT, r.tok_offsets, r.tok_rows, r.row_expert, r.row_w, dX, dL, T, \
                                          d, E, slices)
  SMOE_AGG(1);
  SMOE_AGG(2);
  SMOE_AGG(3);
  SMOE_AGG(4);
#undef SMOE_AGG
  return hipGetLastError();
}

hipError_t launch_reduce_rowparts(const float* part, float* out, int rows, int parts, hipStream_t s) {
  reduce_rowparts_kernel<<<dim3((rows + 255) / 256), dim3(256), 0, s>>>(part, out, rows, parts);
  return hipGetLastError();
}

}  // namespace smoe
