// Internal launchers of the HIP kernels (host side, C++).  The C ABI in
// moe_abi.cpp validates arguments, carves workspaces and calls these.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sonicmoe.h"

namespace smoe {

// routing
hipError_t launch_topk_route(const float* in, float* scores, float* scores_t, int32_t* topk_idx, float* topk_w,
                             uint64_t* mask, int T, int E, int K, int W, int do_softmax, hipStream_t s);
hipError_t launch_tc_metadata(const moe_routing& r, int T, int E, int K, bool counts_only, hipStream_t s);
// counted: r.mask_prefix and r.counts are already written (by launch_round)
hipError_t launch_metadata(const moe_routing& r, const float* scores_t, int T, int E, bool counted, hipStream_t s);
// list: round_scratch_bytes(T, E) bytes (8-byte aligned) for the selection's
// lists
size_t round_scratch_bytes(int T, int E);
hipError_t launch_round(const moe_routing& tc, moe_routing& tr, const float* u, int T, int E, int M, int mode,
                        uint64_t* list, bool* counted, hipStream_t s);

// GEMMs (all bf16 in, fp32 accumulation)
struct RouterGemmArgs {
  const uint16_t* X; const uint16_t* Wr; const float* bias; float* logits; int T, d, E;
};
hipError_t launch_router_gemm(const RouterGemmArgs& a, hipStream_t s);
// The router GEMM with softmax and top-K fused into its epilogue (one tile
// spans every expert): the outputs of launch_topk_route with do_softmax = 1,
// and the logits too when logits is not null.
struct RouterTopkArgs {
  const uint16_t* X; const uint16_t* Wr; const float* bias;
  float* logits; float* scores; float* scores_t; int32_t* topk_idx; float* topk_w; uint64_t* mask;
  int T, d, E, K, W;
};
bool router_topk_fusable(int E, int K);
hipError_t launch_router_topk(const RouterTopkArgs& a, hipStream_t s);

// Routing of few tokens (T <= kFewTokens, E <= kFewExperts, 32-bit offsets within
// W_r): the router GEMM's partial logits of `slices` k slices [slices][T][E], then a
// wave per token for softmax and top-K, then (T > kFewOneGroup) one launch of
// metadata, which every workgroup forms from all T K list entries.  us of moe_route,
// few-token form / other path:
//                                    T = 2048       4096        6144        8192       16384
//   d = 1024, E = 64, K = 8          17.7 / 28.7    20.6 / 29.2 29.4 / 29.3 32.4 / 29.6 50 / 31
//   d = 1536, E = 128, K = 8         21.3 / 38.9    24.4 / 39.4 37 / 40     41 / 41    62 / 42
//   d = 2048, E = 256, K = 8         27.9 / 64.7    39.5 / 65.7 51 / 68     55 / 69    89 / 73
//   d = 4096, E = 8, K = 2           23.4 / 38.6    24.9 / 39.5 39 / 40     41 / 40    55 / 41
//   d = 1536, E = 512, K = 8         40.6 / 101.5   48.8 / 104  69 / 105    73 / 106   130 / 113
// 4096 is below every crossing; with E >= 256 the form would pay to 8192.
constexpr int kFewTokens = 4096, kFewExperts = 1024;
constexpr int kFewOneGroup = 16;  // tokens whose top-K and metadata are one launch
// counts_only: its metadata counts the top-K entries in LDS, where the other path
// only sums bitmap words; with few experts and many entries that is the faster one
// (one_launch: router and top-K fuse there).  us, few-token form / other path:
//   E = 64, K = 8, d = 128   T = 1024 13.2 / 12.9   2048 14.9 / 13.3   4096 17.5 / 13.5
//   E = 64, K = 8, d = 768   T = 2048 16.2 / 17.2   3072 17.8 / 17.6   4096 18.9 / 17.4
//   E = 128, K = 8, d = 128  T = 2048 16.6 / 17.9   3072 18.4 / 18.0   4096 19.6 / 18.4
//   E = 64, K = 2, d = 128   T = 4096 11.5 / 13.0;  E = 256, K = 8 26.3 / 33.1
//   scores given, K = 8      E = 8 T = 256 6.6 / 6.3, 4096 11.5 / 6.4;  E = 64 T = 2048 11.5 / 11.4
inline bool route_few(const moe_dims& m, bool counts_only, bool scores_in, bool one_launch) {
  if (m.T > kFewTokens || m.E > kFewExperts || (int64_t)m.d * m.E > INT32_MAX) return false;
  if (!counts_only || m.T <= kFewOneGroup) return true;
  const int64_t entries = (int64_t)m.T * m.K;
  if (scores_in) return entries <= 256 * m.E;
  return !one_launch || m.E > 128 || entries <= 8192 + 18 * (int64_t)m.d + (m.E > 64 ? 16384 : 0);
}
struct RouterPartArgs {
  const uint16_t* X; const uint16_t* Wr; float* part; int T, d, E, slice;
};
// slices for part_bytes of partials (1 where two do not fit: the partial logits
// then go to a [T][E] array)
int router_slices(int T, int d, int E, size_t part_bytes);
hipError_t launch_router_part(const uint16_t* X, const uint16_t* Wr, float* part, int slices, int T, int d, int E,
                              hipStream_t s);
// in: `slices` slabs of logits (bias added here) or, with do_softmax = 0, the
// scores.  For T <= kFewOneGroup the launch also builds the metadata (counts_only as in
// launch_tc_metadata).
hipError_t launch_topk_few(const float* in, int slices, const float* bias, float* logits, float* scores_t,
                           const moe_routing& r, int T, int E, int K, int do_softmax, bool counts_only, hipStream_t s);
hipError_t launch_tc_metadata_few(const moe_routing& r, int T, int E, int K, bool counts_only, hipStream_t s);

// What built a routing, as moe_routing.reserved keeps it: 0 for token choice, else
// the rounding's m_tile and mode.  It guides the choice of kernels.
inline int rounding_word(int m_tile, int mode) { return m_tile | mode << 16; }
inline int rounding_tile(const moe_routing& r) { return r.reserved & 0xffff; }
inline int rounding_mode(const moe_routing& r) { return r.reserved >> 16; }

// The varlen-M m-tile list (mtiles_kernel): built from the expert offsets
// once per forward / backward call, read by the up, down, dH and dX~ GEMMs.
constexpr int kMTile = 256;  // rows of an m-tile
size_t mtiles_bytes(int64_t capacity, int E);
// about how many m-tiles a routing has
int64_t expected_mtiles(const moe_dims& m, const moe_routing& r);
hipError_t launch_mtiles(const int32_t* offsets, int E, int32_t* out, hipStream_t s);

// mt: the m-tiles to expect (expected_mtiles), for the choice of the tiles; capacity
// bounds the rows.
struct UpArgs {
  const uint16_t* X; const uint16_t* W1; const int32_t* offsets; const int32_t* row_token;
  uint16_t* H; uint16_t* A; int d, n, E, capacity; int64_t mt; const int32_t* mtiles;
  const float* b1;  // [E,2n] expert bias added to H, or null
};
hipError_t launch_up(const UpArgs& a, hipStream_t s);

struct DownArgs {
  const uint16_t* A; const uint16_t* W2; const int32_t* offsets; uint16_t* Y; int d, n, E, capacity;
  int64_t mt; const int32_t* mtiles;
  const float* b2;  // [E,d] expert bias added to Y, or null
  // aggregation ablation only: token-major destination row of each row
  // (scatter), or the fp32 output and the row tokens / weights (atomics)
  const int32_t* dst = nullptr; float* O32 = nullptr; const int32_t* row_token = nullptr;
  const float* row_w = nullptr;
};
hipError_t launch_down(const DownArgs& a, hipStream_t s);
// MOE_AGG_* strategy 0: as launch_down; 1: Y rows scattered to a.dst[row]; 2:
// fp32 atomic accumulation of s * Y into a.O32 (no Y stored)
hipError_t launch_down_ablation(const DownArgs& a, int strategy, hipStream_t s);

// The same for few rows per expert (stream_gemm.hip).  stream_shape: for a routing
// of at most `capacity` rows (m_tile: of the rounding that built it, else 0), or
// mb = 0 where the tiled GEMMs above (tiles_per_expert tiles of an expert with up to
// 256 rows) are the better ones.
struct StreamShape {
  int mb;       // row blocks per workgroup
  int further;  // workgroups (per column tile) for the experts' groups past the first
};
StreamShape stream_shape(const moe_dims& m, int capacity, int m_tile, int64_t tiles_per_expert);
hipError_t launch_stream_up(const UpArgs& a, const StreamShape& t, hipStream_t s);
hipError_t launch_stream_down(const DownArgs& a, int strategy, const StreamShape& t, hipStream_t s);  // MOE_AGG_*

struct DHArgs {
  const uint16_t* dO; const uint16_t* W2; const uint16_t* H; const int32_t* offsets; const int32_t* row_token;
  const float* row_w; uint16_t* dH; uint16_t* Ap; float* dS; float* dS_part; int d, n, E, capacity;
  int64_t mt; const int32_t* mtiles;
  // <dO_t, b2_e> of the expert-bias dS term as two fp32 halves [T][2E]
  // (columns e and E + e; see launch_bias_split), or null
  const float* bq;
};
int dh_n_tiles(int n, int64_t mt);  // dS partials per row
inline int dh_max_n_tiles(int n) { return (n + 63) / 64; }  // at the narrowest tile
hipError_t launch_dh(const DHArgs& a, hipStream_t s);

struct DXtArgs {
  const uint16_t* dH; const uint16_t* W1; const int32_t* offsets; uint16_t* dXt; int d, n, E, capacity;
  int64_t mt; const int32_t* mtiles;
};
hipError_t launch_dxt(const DXtArgs& a, hipStream_t s);

// Weight gradients (varlen K over each expert's rows).  klist: the GEMM's
// k-chunk list (kchunks_bytes(E) bytes, written by launch_bwd_lists); part:
// dw_part_bytes bytes of fp32 partials for experts split into row chunks, which
// launch_bwd_final_reduce sums.
constexpr int kDwSlabs = 128;                                // partial slabs per GEMM at most
constexpr int64_t kDwSlabBytes = (int64_t)256 << 20;         // and at most this many bytes
size_t kchunks_bytes(int E);
// slabs of a GEMM with mn outputs per expert (0: no expert is split)
int dw_slabs(int T, int64_t mn);
inline size_t dw_part_bytes(int T, int64_t mn) { return (size_t)dw_slabs(T, mn) * mn * 4; }
// the backward's m-tile list (as launch_mtiles) and the k-chunk lists of dW2
// and dW1, in one launch; with Wr non-null the same launch writes WrT[e][i] =
// Wr[i][e] (the dX aggregation's router term reads W_r by expert)
hipError_t launch_bwd_lists(const int32_t* offsets, int T, int64_t rows, int E, int d, int n, int32_t* mtiles, int32_t* klist2,
                            int32_t* klist1, const uint16_t* Wr, uint16_t* WrT, hipStream_t s);

struct DW2Args {
  const uint16_t* Ap; const uint16_t* dO; const int32_t* offsets; const int32_t* row_token; uint16_t* dW2;
  int T; int64_t rows; int d, n, E;
  int32_t* klist; float* part;
};
hipError_t launch_dw2(const DW2Args& a, hipStream_t s);

struct DW1Args {
  const uint16_t* X; const uint16_t* dH; const int32_t* offsets; const int32_t* row_token; uint16_t* dW1;
  int T; int64_t rows; int d, n, E;
  int32_t* klist; float* part;
};
hipError_t launch_dw1(const DW1Args& a, hipStream_t s);

// dW_r = X^T dL and dbias (column sums of dL), split over token chunks: partials
// part [splits][d][E] (null: no dW_r) and bias_part [splits][E] (null: no dbias),
// summed by launch_bwd_final_reduce
struct DWrArgs {
  const uint16_t* X; const uint16_t* dL; float* part; float* bias_part; int T, d, E, splits;
};
int dwr_splits(int T, int d, int E, bool dbias);  // (most without dbias)
hipError_t launch_dwr(const DWrArgs& a, hipStream_t s);

// Expert biases.  The down-projection bias term of dS, <dO_t, b2_e> for every
// (t, e), is one GEMM dO [T,d] x B2s [d,2E] on the router GEMM's path: B2s
// holds b2^T split into bf16 high and low parts (columns e and E + e), whose
// products with the bf16 dO are exact in the fp32 accumulation, so the term
// keeps about 16 bits of b2.  launch_bias_split writes B2s.
hipError_t launch_bias_split(const float* b2, int E, int d, uint16_t* B2s, hipStream_t s);
// The expert-bias gradients (either may be null): db1[e] = sum over expert e's
// rows of dH, db2[e] = sum of s * dO of the rows' tokens; fixed summation order,
// fp32.  part: colsum_part_bytes(capacity, E, d, n) bytes.
struct ExpertColsumArgs {
  const uint16_t* dH; const uint16_t* dO; const int32_t* offsets; const int32_t* row_token; const float* row_w;
  const int32_t* mtiles; float* part; float* db1; float* db2; int d, n, E, capacity;
};
inline size_t colsum_part_bytes(int64_t capacity, int E, int d, int n) {
  return (size_t)(capacity / kMTile + E) * (2 * n + d) * 4;
}
hipError_t launch_expert_colsum(const ExpertColsumArgs& a, hipStream_t s);

// aggregation and small kernels
hipError_t launch_agg_o(const uint16_t* Y, const moe_routing& r, uint16_t* O, int T, int d, hipStream_t s);
// aggregation ablation: dst[tok_rows[j]] = j (token-major slot of each row);
// O from token-major (contiguous) Y rows; fp32 buffer fill and fp32 -> bf16
hipError_t launch_tok_slots(const moe_routing& r, int T, int P_bound, int32_t* dst, hipStream_t s);
hipError_t launch_agg_o_contig(const uint16_t* Yt, const moe_routing& r, uint16_t* O, int T, int d, hipStream_t s);
hipError_t launch_fill_f32(float* p, size_t n, hipStream_t s);
hipError_t launch_f32_to_bf16(const float* in, uint16_t* out, size_t n, hipStream_t s);
// dS of row r: the sum of its ds_parts values at dS[r * ds_parts]
hipError_t launch_agg_dx(const uint16_t* dXt, const float* dS, int ds_parts, const uint16_t* WrT, const moe_routing& r, uint16_t* dX,
                         uint16_t* dL, int T, int d, int E, hipStream_t s);
hipError_t launch_reduce_rowparts(const float* part, float* out, int rows, int parts, hipStream_t s);
// The backward's last reductions: the chunk slabs of split experts in dW2 and
// dW1 (klist*, part*), the dW_r split-K partials and the dbias partials (dWr and
// dbias may be null).
struct FinalReduceArgs {
  const int32_t* klist2; const float* part2; uint16_t* dW2;
  const int32_t* klist1; const float* part1; uint16_t* dW1;
  const float* dwr_part; float* dWr; const float* dbias_part; float* dbias; int T, d, n, E, splits;
};
hipError_t launch_bwd_final_reduce(const FinalReduceArgs& a, hipStream_t s);

// timing hooks (moe_abi.cpp)
void prof_begin(int kernel_class, hipStream_t s);
void prof_end(int kernel_class, hipStream_t s);

}  // namespace smoe
