// Routing kernels: softmax + top-K selection, the per-expert membership
// bitmap, and the routing metadata built from it (counts, offsets,
// expert-major rows and the token-major CSR view).
//
// Top-K follows the token-choice rule of Section 2.3 with the stable order of
// the top-K kernel in Appendix D (equal scores go to the lower expert index).
// Unlike that kernel, the expert index is not packed into the low mantissa
// bits: the comparison uses the exact (score, index) pair, so no score is
// perturbed.  Three forms: a lane per token (topk_lane_kernel: E <= 256, many
// tokens), a wave per token over a workgroup of 64 consecutive tokens, i.e. one
// 64-bit word of every expert's membership bitmap, assembled in LDS
// (topk_route_kernel: more experts), and a wave per token with the metadata
// formed from the lists (topk_few_kernel: few tokens).  The waves select their
// token's K winners by arg-max rounds or over the key bits (wave_topk).
#include "device_common.h"
#include "launch.h"
#include "topk_net.h"

namespace smoe {

// The top K of one token, a wave per token (value j of lane l is expert 64 j +
// l), ordered by (value desc, expert asc): put(k, e, w) is called once for each
// of the K positions, by some lane, with w the value over the selected values'
// sum (added in ascending expert order).
//
// Small K: K rounds of a wave-wide arg-max (six dependent DPP steps each).
// Larger K, EPL <= 16 (beyond, the masks would not fit the scalar registers): a
// select over the bits of the 32-bit keys, most significant first, on ballots.  The
// candidates with the bit set replace the candidates if they are as many as still
// wanted, else they are selected and the others stay; it stops once the candidates
// are exactly as many as wanted, after about half of the bits.  Equal keys at the
// end go to the lowest experts (lowest j, then lowest lane).  Scalar masks and
// counts, one vector compare per bit, whatever K.  us of the top-K launch, rounds /
// bits:
//   T = 4096, E = 64     K = 1 6.7 / 7.3    4 7.5 / 7.9    6 8.2 / 8.5    8 9.3 / 8.7    16 12.0 / 9.3
//   T = 16, E = 64             7.3 / 8.8      9.0 / 8.5      9.7 / 8.6     11.1 / 9.2      14.1 / 10.2
//   T = 4096, E = 256          8.1 / 11.5     9.9 / 13.0    11.7 / 13.2    13.3 / 13.8     20.1 / 15.0
//   T = 4096, E = 1024        11.9 / 29.5    20.2 / 32.3    26.0 / 33.2    31.1 / 35.8     52.7 / 41.9
//   T = 16384, E = 512        19.4 / 47.4    36.6 / 55.3    48.0 / 57.7    58.8 / 61.2    103.5 / 67.1
template <int EPL>
constexpr int kBitSelectK = EPL == 1 ? 6 : EPL <= 4 ? 8 : EPL <= 16 ? 9 : 17;
template <int EPL, class Put>
__device__ __forceinline__ void wave_topk(const float (&v)[EPL], int E, int K, Put put) {
  static_assert(EPL >= 1 && EPL <= 64, "the taken mask holds one bit per value of a lane");
  const int lane = lane_id();
  float denom = 0.f;
  bool bits = false;
  if constexpr (kBitSelectK<EPL> <= 16) bits = K >= kBitSelectK<EPL>;
  if (bits) {
    uint32_t key[EPL];
    int rank[EPL];
    uint64_t alive[EPL], sel[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      key[j] = topk_key(v[j]);
      rank[j] = 0;
      alive[j] = __ballot(lane + 64 * j < E);
      sel[j] = 0;
    }
    int na = E, need = K;
    for (int b = 31; b >= 0 && na > need; --b) {
      const uint32_t bit = 1u << b;
      uint64_t one[EPL];
      int c = 0;
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        one[j] = __ballot((key[j] & bit) != 0) & alive[j];
        c += __popcll(one[j]);
      }
      const bool more = c >= need;
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        sel[j] |= more ? 0ull : one[j];
        alive[j] = more ? one[j] : alive[j] & ~one[j];
      }
      na = more ? c : na - c;
      need = more ? need : need - c;
    }
    const bool ties = na > need;  // equal keys: the lowest experts
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      uint64_t a = alive[j];
      if (ties) {
        for (int drop = __popcll(a) - need; drop > 0; --drop) a &= ~(1ull << (63 - __clzll(a)));
        need -= __popcll(a);
      }
      sel[j] |= a;
    }
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      for (uint64_t m = sel[j]; m; m &= m - 1) {
        const int l = __ffsll((unsigned long long)m) - 1;
        denom += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[j]), l));
        const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key[j], l);
        const int e = 64 * j + l;
#pragma unroll
        for (int i = 0; i < EPL; ++i) rank[i] += k > key[i] || (k == key[i] && e < lane + 64 * i);
      }
    }
#pragma unroll
    for (int j = 0; j < EPL; ++j)
      if ((sel[j] >> lane) & 1ull) put(rank[j], lane + 64 * j, topk_value(key[j]) / denom);
  } else {
    uint64_t taken = 0;  // bit j: value j of this lane is selected
    int sel_e[16];
    float sel_v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      sel_e[k] = 0;
      sel_v[k] = 0.f;
      if (k < K) {
        uint32_t best = 0;
        int bj = -1;  // j of this lane's best candidate (the lowest j on equal keys)
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
          const int e = lane + 64 * j;
          if (e < E && !((taken >> j) & 1ull)) {
            const uint32_t c = topk_key(v[j]);
            if (bj < 0 || c > best) {
              best = c;
              bj = j;
            }
          }
        }
        const uint32_t m = dpp_reduce(bj >= 0 ? best : 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
        int be = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
          const uint64_t hit = __ballot(bj == j && best == m);
          if (hit && be == 0x7fffffff) be = __ffsll((unsigned long long)hit) - 1 + 64 * j;
        }
        if (be != 0x7fffffff && (be & 63) == lane) taken |= 1ull << (be >> 6);
        sel_e[k] = be;
        sel_v[k] = topk_value(m);
      }
    }
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      uint64_t sel = __ballot((taken >> j) & 1ull);
      while (sel) {
        const int l = __ffsll((unsigned long long)sel) - 1;
        denom += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[j]), l));
        sel &= sel - 1;
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (k < K && lane == k) put(k, sel_e[k], sel_v[k] / denom);
  }
}

constexpr int kTopkWaves = 16;

// Workgroup = 64 tokens (one membership word).  `in` and `scores` may alias
// (logits overwritten in place by the scores).
template <int EPL>
__global__ __launch_bounds__(1024) void topk_route_kernel(const float* in, float* scores, float* __restrict__ scores_t,
                                                         int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                         uint64_t* __restrict__ mask, int T, int E, int K, int W,
                                                         int do_softmax) {
  extern __shared__ unsigned long long mword[];  // [E]
  const int w = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = lane_id();
  for (int e = threadIdx.x; e < E; e += kTopkWaves * 64) mword[e] = 0ull;
  __syncthreads();
  auto load_row = [&](int i, float (&v)[EPL]) {
    const int t = w * 64 + i;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + 64 * j;
      v[j] = (t < T && e < E) ? in[(size_t)t * E + e] : -INFINITY;
    }
  };
  float vn[EPL];
  load_row(wave, vn);
  for (int i = wave; i < 64; i += kTopkWaves) {
    const int t = w * 64 + i;
    if (t >= T) break;
    float v[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) v[j] = vn[j];
    if (i + kTopkWaves < 64) load_row(i + kTopkWaves, vn);  // the wave's next token, in flight meanwhile
    if (do_softmax) {
      float m = -INFINITY;
#pragma unroll
      for (int j = 0; j < EPL; ++j) m = fmaxf(m, v[j]);
      m = dpp_reduce(m, [](float a, float b) { return fmaxf(a, b); });
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        const int e = lane + 64 * j;
        v[j] = e < E ? expf(v[j] - m) : 0.f;
        s += v[j];
      }
      s = dpp_reduce(s, [](float a, float b) { return a + b; });
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        const int e = lane + 64 * j;
        if (e < E) {
          v[j] = v[j] / s;
          scores[(size_t)t * E + e] = v[j];
        }
      }
    }
    if (scores_t) {
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        const int e = lane + 64 * j;
        if (e < E) scores_t[(size_t)e * T + t] = v[j];
      }
    }
    wave_topk<EPL>(v, E, K, [&](int k, int e, float wt) {
      topk_idx[(size_t)t * K + k] = e;
      topk_w[(size_t)t * K + k] = wt;
      atomicOr(&mword[e], 1ull << i);
    });
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += kTopkWaves * 64) mask[(size_t)e * W + w] = mword[e];
}

// Lane-per-token selection (K <= KM <= 16; E a multiple of 4 * NW, E <= 256).
// A workgroup owns the 64 tokens of one membership word, lane l token 64w + l,
// and its NW waves split the experts into NW contiguous slices, so the
// per-token work is ordinary per-lane arithmetic instead of wave-wide
// reductions.  Each wave keeps its slice of the token's row in LDS as
// [slice/4][64] float4 (lane l's column: conflict-free in every pass):
//   1. row max (the row loads are issued 16 float4 at a time), combined
//      across the slices;
//   2. exp(x - max) and the slice sums, combined in slice order;
//   3. scores = exp * (1 / sum) (written token-major and, coalesced across lanes,
//      transposed), and a KM-slot insertion network over the (key, expert)
//      pairs of the slice: an element moves down past every slot whose pair
//      it exceeds; the network runs only when some lane's element beats its
//      last slot.  The slices' lists are then merged (top-KM of two sorted
//      lists: pairwise maxima of one list against the other reversed, then a
//      bitonic clean-up), every wave doing the same merge;
//   4. membership: expert e is selected iff its pair ranks at or above the
//      K-th slot; a ballot per expert is the membership word.  The selected
//      scores are summed in ascending expert order for the renormalisation
//      denominator (each slice lists its selected scores in order in LDS,
//      the first wave adds the lists slice by slice).
// The (score, index) pairs are compared exactly, as in the wave-per-token
// kernel above: equal keys order by the lower expert.
template <int KM, int NW>
__global__ __launch_bounds__(64 * NW) void topk_lane_kernel(const float* in, float* scores, float* __restrict__ scores_t,
                                                            int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                            uint64_t* __restrict__ mask, int T, int E, int K, int W,
                                                            int do_softmax) {
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  const int w = blockIdx.x;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = lane_id();
  const int t = w * 64 + lane;
  const bool live = t < T;
  const int Eq = E / NW, Gq = Eq >> 2, e0 = q * Eq;
  f32x4* cols = (f32x4*)dyn + (size_t)q * Gq * 64;      // [Gq][64]
  float* xmax = (float*)(dyn + (size_t)E * 256);           // [NW][64]
  float* xsum = xmax + NW * 64;                            // [NW][64]
  uint64_t* lists = (uint64_t*)(xsum + NW * 64);           // [NW][KM][64]
  int* nsel = (int*)(lists + NW * KM * 64);                // [NW][64]
  float* sv = (float*)lists;                               // [NW][KM][64] selected scores, expert order (lists read)
  // a lane past T reads token 0's row and discards it
  const f32x4* row = (const f32x4*)(in + (size_t)(live ? t : 0) * E + e0);
  const f32x4 ninf = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  float m = -INFINITY;
#pragma unroll 16
  for (int g = 0; g < Gq; ++g) {
    const f32x4 x0 = row[g];
    const f32x4 x = live ? x0 : ninf;
    cols[g * 64 + lane] = x;
    m = fmaxf(m, fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
  }
  float s = 1.f;
  if (do_softmax) {
    if constexpr (NW > 1) {
      xmax[q * 64 + lane] = m;
      __syncthreads();
#pragma unroll
      for (int p = 0; p < NW; ++p) m = fmaxf(m, xmax[p * 64 + lane]);
    }
    s = 0.f;
#pragma unroll 4
    for (int g = 0; g < Gq; ++g) {
      f32x4 x = cols[g * 64 + lane];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        x[c] = __expf(x[c] - m);  // v_exp_f32 of (x - m) log2(e): a few ulp for |x - m| < 100
        s += x[c];
      }
      cols[g * 64 + lane] = x;
    }
    if constexpr (NW > 1) {
      xsum[q * 64 + lane] = s;
      __syncthreads();
      s = xsum[lane];
#pragma unroll
      for (int p = 1; p < NW; ++p) s += xsum[p * 64 + lane];
    }
  }
  const float rs = 1.f / s;  // scores = exp * (1 / sum): within an ulp of the quotient
  uint64_t top[KM];
#pragma unroll
  for (int k = 0; k < KM; ++k) top[k] = 0;  // below every (key, ~expert) pair
  // Pairs are taken in groups of KM: each group is sorted by a bitonic network
  // and merged into the running top-KM list, i.e. independent compare-exchanges
  // instead of a serial insertion chain per pair.  One step covers G2 float4s
  // (KM = 8: two); slots past the slice and lanes past T hold 0, below every
  // real pair.
  constexpr int G2 = KM >= 4 ? KM / 4 : 1;
  for (int g0 = 0; g0 < Gq; g0 += G2) {
    uint64_t pr[4 * G2];
#pragma unroll
    for (int gg = 0; gg < G2; ++gg) {
      const int g = g0 + gg;
      if (g < Gq) {
        f32x4 p = cols[g * 64 + lane];
        const int eg = e0 + 4 * g;
        if (do_softmax) {
#pragma unroll
          for (int c = 0; c < 4; ++c) p[c] = p[c] * rs;
          cols[g * 64 + lane] = p;
          if (live) *(f32x4*)(scores + (size_t)t * E + eg) = p;
        }
        if (scores_t && live) {
#pragma unroll
          for (int c = 0; c < 4; ++c) scores_t[(size_t)(eg + c) * T + t] = p[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          pr[4 * gg + c] = live ? topk_pair(p[c], eg + c) : 0ull;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) pr[4 * gg + c] = 0ull;
      }
    }
#pragma unroll
    for (int h = 0; h < 4 * G2; h += KM) {
      uint64_t grp[KM];
#pragma unroll
      for (int k = 0; k < KM; ++k) grp[k] = pr[h + k];
      topk_sort<KM>(grp);
      topk_merge<KM>(top, grp);
    }
  }
  if constexpr (NW > 1) {
#pragma unroll
    for (int k = 0; k < KM; ++k) lists[(q * KM + k) * 64 + lane] = top[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KM; ++k) top[k] = lists[k * 64 + lane];
#pragma unroll
    for (int p = 1; p < NW; ++p) {
      uint64_t b[KM];
#pragma unroll
      for (int k = 0; k < KM; ++k) b[k] = lists[(p * KM + k) * 64 + lane];
      topk_merge<KM>(top, b);
    }
  }
  if constexpr (NW > 1) __syncthreads();  // the lists' space is reused for sv
  uint64_t thr = top[0];
#pragma unroll
  for (int k = 1; k < KM; ++k)
    if (k == K - 1) thr = top[k];
  // membership words of this wave's experts (expert e0 + 64 r + lane in mw[r])
  constexpr int kWords = NW > 1 ? 1 : 4;
  float den = 0.f;
  int ns = 0;
  uint64_t mw[kWords];
#pragma unroll
  for (int r = 0; r < kWords; ++r) mw[r] = 0ull;
#pragma unroll
  for (int r = 0; r < kWords; ++r) {
    const int g1 = min(Gq, 16 * r + 16);
    for (int g = 16 * r; g < g1; ++g) {
      const f32x4 p = cols[g * 64 + lane];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int el = 4 * g + c;  // expert e0 + el
        const uint64_t x = topk_pair(p[c], e0 + el);
        const bool sel = live && x >= thr;
        const uint64_t word = __ballot(sel);
        if (lane == (el & 63)) mw[r] = word;
        if constexpr (NW > 1) {
          if (sel) sv[(q * KM + ns) * 64 + lane] = p[c];
          ns += sel;
        } else {
          den += sel ? p[c] : 0.f;  // +0 for the others leaves the sum unchanged
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kWords; ++r)
    if (64 * r + lane < Eq) mask[(size_t)(e0 + 64 * r + lane) * W + w] = mw[r];
  if constexpr (NW > 1) {
    nsel[q * 64 + lane] = ns;
    __syncthreads();
    if (q != 0) return;
    // selected scores in ascending expert order: slice by slice
    for (int p = 0; p < NW; ++p) {
      const int np = nsel[p * 64 + lane];
      for (int j = 0; j < np; ++j) den += sv[(p * KM + j) * 64 + lane];
    }
  }
  if (live) {
#pragma unroll
    for (int k = 0; k < KM; ++k)
      if (k < K) {
        topk_idx[(size_t)t * K + k] = (int32_t)~(uint32_t)top[k];
        topk_w[(size_t)t * K + k] = topk_value((uint32_t)(top[k] >> 32)) / den;
      }
  }
}

static size_t topk_lane_lds(int E, int KM, int NW) {
  // E = 128, K = 8: 51 KB, three workgroups per CU (with sv in its own space two,
  // and T = 40960 ran two rounds: 32.5 -> 28 us)
  return (size_t)E * 256 + (NW > 1 ? (size_t)NW * 64 * (4 + 4 + 8 * KM + 4) : 0);
}

// ------------------------------------------------------------- few tokens
// Decode and short prefill calls (T <= kFewTokens).  The lane-per-token kernels
// above are built for many tokens: with few of them they run on a handful of
// CUs for the latency of a whole token's serial work (T = 1: the one-launch
// router 21 us, then three metadata launches 15 us).  Here a wave takes one
// token, and the routing metadata comes from the top-K lists instead of the
// bitmap: T K entries, counted in LDS.

// rows of one 64-token word from its top-K lists: row = first row of the expert
// + its tokens in earlier words + its earlier tokens in the word
__device__ __forceinline__ void place_word(const moe_routing& r, int w, int T, int K, const int* idx, const float* wt,
                                           const unsigned long long* word, const int* base) {
  const int nt = min(64, T - 64 * w);
  for (int i = threadIdx.x; i < nt * K; i += blockDim.x) {
    const int tl = i / K, t = 64 * w + tl, e = idx[i];
    int rank = 0;  // the token's selected experts below e
    for (int k = 0; k < K; ++k) rank += idx[tl * K + k] < e;
    const int row = base[e] + __popcll(word[e] & ((1ull << tl) - 1));
    r.tok_rows[(size_t)t * K + rank] = row;
    r.row_token[row] = t;
    r.row_expert[row] = e;
    r.row_w[row] = wt[i];
  }
  for (int tl = threadIdx.x; tl < nt; tl += blockDim.x) {
    r.tok_offsets[64 * w + tl] = (64 * w + tl) * K;
    r.tok_count[64 * w + tl] = K;
    if (64 * w + tl == T - 1) r.tok_offsets[T] = T * K;
  }
}

// A wave per token: softmax of the summed partial logits (or the scores as
// given), top-K.  WG16: a workgroup of 16 waves holds 16 tokens, whose
// transposed scores leave as 64-byte runs.  Else (META) one workgroup holds all
// T <= 16 tokens and goes on to the metadata.
constexpr int kFewWaves = kFewOneGroup;
template <int EPL, bool META>
__global__ __launch_bounds__(64 * kFewWaves) void topk_few_kernel(const float* in, int slices,
                                                                 const float* __restrict__ bias, float* logits,
                                                                 float* __restrict__ scores_t, const moe_routing r,
                                                                 int T, int E, int K, int do_softmax, int counts_only) {
  // META: words [E], bases [E], idx and weights [16][K]; else with scores_t: [E][17] scores
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  __shared__ int scan_lds[16];
  unsigned long long* word = (unsigned long long*)dyn;
  int* base = (int*)(dyn + 8 * (size_t)E);
  int* sidx = base + E;
  float* sw = (float*)(sidx + kFewWaves * K);
  float* st = (float*)dyn;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  if constexpr (META) {
    for (int e = threadIdx.x; e < E; e += 64 * kFewWaves) word[e] = 0ull;
    __syncthreads();
  }
  const size_t slab = (size_t)T * E;
  if (const int t = blockIdx.x * kFewWaves + wave; t < T) {
    float v[EPL];
    // slabs in slice order, four at a time (all their loads in flight together)
    for (int q0 = 0; q0 < slices; q0 += 4) {
      float x[4][EPL];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
          const int e = lane + 64 * j;
          x[q][j] = q0 + q < slices && e < E ? in[(q0 + q) * slab + (size_t)t * E + e] : 0.f;
        }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < EPL; ++j) v[j] = q0 + q == 0 ? x[0][j] : v[j] + x[q][j];
    }
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + 64 * j;
      if (e < E) {
        if (bias) v[j] += bias[e];
        if (logits) logits[(size_t)t * E + e] = v[j];
      } else {
        v[j] = -INFINITY;
      }
    }
    if (do_softmax) {
      float m = -INFINITY;
#pragma unroll
      for (int j = 0; j < EPL; ++j) m = fmaxf(m, v[j]);
      m = dpp_reduce(m, [](float a, float b) { return fmaxf(a, b); });
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        v[j] = lane + 64 * j < E ? expf(v[j] - m) : 0.f;
        s += v[j];
      }
      s = dpp_reduce(s, [](float a, float b) { return a + b; });
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        const int e = lane + 64 * j;
        if (e < E) r.scores[(size_t)t * E + e] = v[j] = v[j] / s;
      }
    }
    if (scores_t) {
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        const int e = lane + 64 * j;
        if (e >= E) continue;
        if constexpr (META)
          scores_t[(size_t)e * T + t] = v[j];
        else
          st[e * (kFewWaves + 1) + wave] = v[j];
      }
    }
    wave_topk<EPL>(v, E, K, [&](int k, int e, float wt) {
      r.topk_idx[(size_t)t * K + k] = e;
      r.topk_w[(size_t)t * K + k] = wt;
      if constexpr (META) {
        sidx[t * K + k] = e;
        sw[t * K + k] = wt;
        atomicOr(&word[e], 1ull << t);
      }
    });
  }
  if constexpr (META) {
    __syncthreads();
    int running = 0;
    for (int e0 = 0; e0 < E; e0 += 64 * kFewWaves) {
      const int e = e0 + threadIdx.x;
      const int c = e < E ? __popcll(word[e]) : 0;
      int total;
      const int off = running + block_excl_scan<64 * kFewWaves>(c, &total, scan_lds);
      if (e < E) {
        r.mask[e] = word[e];
        r.mask_prefix[e] = 0;
        r.counts[e] = c;
        if (!counts_only) r.offsets[e] = off;
        base[e] = off;
      }
      running += total;
    }
    if (counts_only) return;
    if (threadIdx.x == 0) {
      r.offsets[E] = running;
      *r.status = 0;
    }
    __syncthreads();
    place_word(r, 0, T, K, sidx, sw, word, base);
  } else if (scores_t) {
    __syncthreads();
    const int t0 = blockIdx.x * kFewWaves, nt = min(kFewWaves, T - t0);
    for (int i = threadIdx.x; i < E * kFewWaves; i += 64 * kFewWaves) {
      const int e = i / kFewWaves, tl = i % kFewWaves;
      if (tl < nt) scores_t[(size_t)e * T + t0 + tl] = st[e * (kFewWaves + 1) + tl];
    }
  }
}

// Bitmap, counts, offsets and rows in one launch: the workgroup of a 64-token
// word counts every expert's tokens, and those of the earlier words, from the
// top-K lists (at most kFewTokens x 16 entries, from L2) and places its own.
__global__ __launch_bounds__(1024) void tc_metadata_few_kernel(const moe_routing r, int T, int E, int K,
                                                               int counts_only) {
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  __shared__ int scan_lds[16];
  unsigned long long* word = (unsigned long long*)dyn;  // [E]
  int* total = (int*)(word + E);                        // [E] tokens of later words, then first rows of the word
  int* before = total + E;                              // [E] tokens of earlier words
  int* sidx = before + E;                               // [64][K]
  float* sw = (float*)(sidx + 64 * K);
  const int w = blockIdx.x, W = gridDim.x;
  for (int e = threadIdx.x; e < E; e += 1024) {
    word[e] = 0ull;
    total[e] = before[e] = 0;
  }
  __syncthreads();
  const int lo = 64 * w * K, hi = min(T, 64 * w + 64) * K;
  // one LDS count per entry outside the word: entries before it and after it
  for (int i0 = 0; i0 < T * K; i0 += 8192) {
    int e[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = i0 + 1024 * q + threadIdx.x;
      e[q] = i < T * K ? r.topk_idx[i] : -1;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = i0 + 1024 * q + threadIdx.x;
      if (e[q] < 0) continue;
      if (i < lo) {
        atomicAdd(&before[e[q]], 1);
      } else if (i >= hi) {
        atomicAdd(&total[e[q]], 1);
      } else {
        sidx[i - lo] = e[q];
        sw[i - lo] = r.topk_w[i];
        atomicOr(&word[e[q]], 1ull << (i / K - 64 * w));
      }
    }
  }
  __syncthreads();
  int running = 0;
  for (int e0 = 0; e0 < E; e0 += 1024) {
    const int e = e0 + threadIdx.x;
    const int c = e < E ? before[e] + __popcll(word[e]) + total[e] : 0;
    int sum;
    const int off = running + block_excl_scan<1024>(c, &sum, scan_lds);
    if (e < E) {
      r.mask[(size_t)e * W + w] = word[e];
      r.mask_prefix[(size_t)e * W + w] = before[e];
      if (w == 0) {
        r.counts[e] = c;
        if (!counts_only) r.offsets[e] = off;
      }
      total[e] = off + before[e];
    }
    running += sum;
  }
  if (counts_only) return;
  if (w == 0 && threadIdx.x == 0) {
    r.offsets[E] = running;
    *r.status = 0;
  }
  __syncthreads();
  place_word(r, w, T, K, sidx, sw, word, total);
}

// Per expert: popcount prefix over its mask words and its count f_e.  status
// (nullable) is cleared for a placement launch that may flag it.
__global__ __launch_bounds__(256) void expert_scan_kernel(const uint64_t* __restrict__ mask,
                                                          int32_t* __restrict__ prefix, int32_t* __restrict__ counts,
                                                          int W, int32_t* __restrict__ status) {
  __shared__ int lds[16];
  const int e = blockIdx.x;
  if (status && e == 0 && threadIdx.x == 0) *status = 0;
  const uint64_t* m = mask + (size_t)e * W;
  int32_t* p = prefix + (size_t)e * W;
  int running = 0;
  for (int c0 = 0; c0 < W; c0 += 256) {
    const int w = c0 + threadIdx.x;
    const int pc = w < W ? __popcll(m[w]) : 0;
    int total;
    const int ex = block_excl_scan<256>(pc, &total, lds);
    if (w < W) p[w] = running + ex;
    running += total;
  }
  if (threadIdx.x == 0) counts[e] = running;
}

// out[0..n] = exclusive scan of cnt[0..n-1] (one block of 1024 threads, four
// values per thread per pass).
__global__ __launch_bounds__(1024) void scan_kernel(const int32_t* __restrict__ cnt, int32_t* __restrict__ out,
                                                    int n) {
  __shared__ int lds[16];
  int running = 0;
  for (int c0 = 0; c0 < n; c0 += 4096) {
    const int i0 = c0 + threadIdx.x * 4;
    int v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = i0 + q < n ? cnt[i0 + q] : 0;
    const int sum = v[0] + v[1] + v[2] + v[3];
    int total;
    int ex = block_excl_scan<1024>(sum, &total, lds) + running;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (i0 + q < n) out[i0 + q] = ex;
      ex += v[q];
    }
    running += total;
  }
  if (threadIdx.x == 0) out[n] = running;
}

// Token-choice placement: every token has exactly K rows, so the token-major
// offsets are t*K.  Each token's experts are visited in ascending order.
// Every workgroup sums the experts' counts to their first rows itself, while
// its top-K lists load, and workgroup 0 writes them: as a launch of its own
// between the counts and the rows the scan was one workgroup's chain of latencies
// (T = 6000, d = 1024, n = 256, E = 64, K = 8 forward 185.9 -> 184.0 us; T = 4999,
// d = 1536, E = 128 253.3 -> 250.8; T = 8192, E = 512 480.5 -> 478.4).
__global__ __launch_bounds__(256) void tc_place_kernel(const int32_t* __restrict__ topk_idx,
                                                       const float* __restrict__ topk_w,
                                                       const uint64_t* __restrict__ mask,
                                                       const int32_t* __restrict__ prefix,
                                                       const int32_t* __restrict__ counts,
                                                       int32_t* __restrict__ offsets,
                                                       int32_t* __restrict__ tok_offsets, int32_t* __restrict__ tok_count,
                                                       int32_t* __restrict__ tok_rows, int32_t* __restrict__ row_token,
                                                       int32_t* __restrict__ row_expert, float* __restrict__ row_w, int T,
                                                       int E, int K, int W, int32_t* __restrict__ status) {
  extern __shared__ int first_row[];  // [E]
  __shared__ int scan_lds[16];
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int w = t >> 6, b = t & 63;
  const uint64_t below = b ? (~0ull >> (64 - b)) : 0ull;
  int ex[16];
  float wt[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    ex[k] = k < K && t < T ? topk_idx[(size_t)t * K + k] : 0x7fffffff;
    wt[k] = k < K && t < T ? topk_w[(size_t)t * K + k] : 0.f;
  }
  int running = 0;
  for (int e0 = 0; e0 < E; e0 += 1024) {
    const int e = e0 + 4 * threadIdx.x;
    int v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = e + q < E ? counts[e + q] : 0;
    int total;
    int row = running + block_excl_scan<256>(v[0] + v[1] + v[2] + v[3], &total, scan_lds);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (e + q < E) {
        first_row[e + q] = row;
        if (blockIdx.x == 0) offsets[e + q] = row;
      }
      row += v[q];
    }
    running += total;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) offsets[E] = running;
  __syncthreads();
  if (t >= T) return;
  int last = -1;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r < K) {
      int e = 0x7fffffff;
      float wv = 0.f;
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (ex[k] > last && ex[k] < e) {
          e = ex[k];
          wv = wt[k];
        }
      last = e;
      if (e == 0x7fffffff) {
        // Fewer than K distinct experts in topk_idx (never from moe_route's
        // top-K).  The mask then holds fewer rows than T*K: flag the routing
        // as invalid and point the token's remaining slots at row 0, so a
        // later kernel that ignores the flag still reads in bounds.
        atomicOr(status, MOE_STATUS_DUPLICATE_EXPERT);
        tok_rows[(size_t)t * K + r] = 0;
        continue;
      }
      const size_t ew = (size_t)e * W + w;
      const int row = first_row[e] + prefix[ew] + __popcll(mask[ew] & below);
      tok_rows[(size_t)t * K + r] = row;
      row_token[row] = t;
      row_expert[row] = e;
      row_w[row] = wv;
    }
  }
  tok_offsets[t] = t * K;
  tok_count[t] = K;
  if (t == T - 1) tok_offsets[T] = T * K;
}

// 64-bit value of lane (lane ^ s), and of lane src (any per-lane index).
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int s) {
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, s, kWave);
  const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), s, kWave);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, kWave);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src, kWave);
  return ((uint64_t)hi << 32) | lo;
}
// 64 x 64 bit transpose across a wave: lane i holds row i on entry; on exit
// lane j holds column j (bit i of lane j's result = bit j of lane i's input).
// Six butterfly stages, each exchanging the off-diagonal s x s blocks of
// every 2s x 2s block between lanes i and i ^ s.
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x, int lane) {
  constexpr uint64_t kLow[6] = {0x00000000FFFFFFFFull, 0x0000FFFF0000FFFFull, 0x00FF00FF00FF00FFull,
                                0x0F0F0F0F0F0F0F0Full, 0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int s = 32 >> k;
    const uint64_t m = kLow[k];  // bit positions j with (j & s) == 0
    const uint64_t y = shfl_xor_u64(x, s);
    x = (lane & s) ? (((y >> s) & m) | (x & ~m)) : ((x & m) | ((y & m) << s));
  }
  return x;
}

// General placement (any membership, e.g. after token rounding), one wave per
// 64-token word.  Pass 1: per-token expert count and renormalisation
// denominator (selected scores summed in ascending expert order, fp32).
// The wave loads the mask words of 64 experts (lane i: expert c0 + i) and
// transposes them, so that lane l holds token l's membership bits of those
// experts; it then walks its own set bits, lowest expert first, issuing the
// score loads of kMetaBatch experts before summing them.
constexpr int kMetaBatch = 8;
constexpr int kMetaChunks = 4;  // 64-expert chunks whose mask words are loaded together

__global__ __launch_bounds__(64) void token_count_kernel(const uint64_t* __restrict__ mask,
                                                         const float* __restrict__ scores_t, int32_t* __restrict__ cnt,
                                                         float* __restrict__ denom, int32_t* __restrict__ word_sum,
                                                         const int32_t* __restrict__ counts,
                                                         int32_t* __restrict__ offsets, int T, int E, int W,
                                                         int32_t* __restrict__ status) {
  const int w = blockIdx.x;
  const int lane = lane_id();
  if (w == W) {
    if (lane == 0) *status = 0;  // membership from the bitmap: always consistent
    // the extra workgroup: offsets = exclusive scan of the expert counts
    int running = 0;
    for (int e0 = 0; e0 < E; e0 += 64) {
      const int v = e0 + lane < E ? counts[e0 + lane] : 0;
      const int inc = wave_incl_scan(v);
      if (e0 + lane < E) offsets[e0 + lane] = running + inc - v;
      running += __shfl(inc, 63, kWave);
    }
    if (lane == 0) offsets[E] = running;
    return;
  }
  const int t = w * 64 + lane;
  const bool live = t < T;
  int c = 0;
  float s = 0.f;
  for (int cb = 0; cb < E; cb += 64 * kMetaChunks) {
    uint64_t words[kMetaChunks];
#pragma unroll
    for (int h = 0; h < kMetaChunks; ++h) {
      const int e = cb + 64 * h + lane;
      words[h] = e < E ? mask[(size_t)e * W + w] : 0ull;
    }
#pragma unroll
    for (int h = 0; h < kMetaChunks; ++h) {
      const int c0 = cb + 64 * h;
      if (c0 >= E) break;
      uint64_t bits = wave_transpose64(words[h], lane);
      if (!live) bits = 0;
      c += __popcll(bits);
      while (__ballot(bits != 0)) {
        float v[kMetaBatch];
#pragma unroll
        for (int u = 0; u < kMetaBatch; ++u) {
          const bool has = bits != 0;
          const int i = has ? __ffsll((unsigned long long)bits) - 1 : 0;
          v[u] = has ? scores_t[(size_t)(c0 + i) * T + t] : 0.f;
          bits &= bits - 1;
        }
        // adding +0 for a miss leaves the sum unchanged (it is never -0)
#pragma unroll
        for (int u = 0; u < kMetaBatch; ++u) s += v[u];
      }
    }
  }
  if (live) {
    cnt[t] = c;
    denom[t] = s;
  }
  const int total = wave_sum(live ? c : 0);
  if (lane == 0) word_sum[w] = total;  // rows of the word's 64 tokens
}

// Pass 2: rows of every token (expert ascending), renormalised weights.  The
// kPlaceWaves waves of a workgroup share one word: wave q places experts
// [q*Ew, (q+1)*Ew); it first counts its experts per token, and the counts of
// the lower ranges (exchanged through LDS) give each token's first slot.  As
// in pass 1, each lane walks its own token's set bits (from the transposed
// mask words); the expert's mask word and row base come from the lane that
// loaded them.
constexpr int kPlaceWaves = 4;
constexpr int kPlaceSumWords = 4096;  // T <= 262144

__global__ __launch_bounds__(64 * kPlaceWaves) void token_place_kernel(
    const uint64_t* __restrict__ mask, const int32_t* __restrict__ prefix, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ tok_count, const int32_t* __restrict__ word_base,
    const int32_t* __restrict__ word_sum, int32_t* __restrict__ tok_offsets,
    const float* __restrict__ scores_t, const float* __restrict__ denom, int32_t* __restrict__ tok_rows,
    int32_t* __restrict__ row_token, int32_t* __restrict__ row_expert, float* __restrict__ row_w, int T, int E,
    int W) {
  __shared__ int cnt[kPlaceWaves][64];
  const int w = blockIdx.x;
  const int lane = lane_id();
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = w * 64 + lane;
  const bool live = t < T;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  const int ew = (E + kPlaceWaves - 1) / kPlaceWaves;
  const int e_lo = min(E, q * ew), e_hi = min(E, e_lo + ew);
  // independent loads first: they overlap the count pass and the barrier
  const int ct = live ? tok_count[t] : 0;
  const float dn = live ? denom[t] : 1.f;
  // the first chunk's words and row bases stay in registers for pass 2
  const int el0 = e_lo + lane;
  const uint64_t words0 = el0 < e_hi ? mask[(size_t)el0 * W + w] : 0ull;
  const int bases0 = el0 < e_hi ? offsets[el0] + prefix[(size_t)el0 * W + w] : 0;
  uint64_t bits0 = wave_transpose64(words0, lane);
  if (!live) bits0 = 0;
  int c = __popcll(bits0);
  for (int c0 = e_lo + 64; c0 < e_hi; c0 += 64) {
    const int el = c0 + lane;
    const uint64_t words = el < e_hi ? mask[(size_t)el * W + w] : 0ull;
    const uint64_t bits = wave_transpose64(words, lane);
    c += live ? __popcll(bits) : 0;
  }
  cnt[q][lane] = c;
  // the word's base: given (word_base), or summed here from the word sums
  __shared__ int wsum[kPlaceWaves];
  int base;
  if (word_base) {
    base = word_base[w];
  } else {
    int part = 0;
    for (int i = threadIdx.x; i < w; i += 64 * kPlaceWaves) part += word_sum[i];
    part = wave_sum(part);
    if (lane == 0) wsum[q] = part;
  }
  __syncthreads();
  if (!word_base) {
    base = 0;
#pragma unroll
    for (int p = 0; p < kPlaceWaves; ++p) base += wsum[p];
  }
  // token t's first row: the word's base plus the rows of the word's earlier
  // tokens; wave 0 also writes tok_offsets
  const int tok_first = base + wave_incl_scan(ct) - ct;
  if (q == 0) {
    if (live) tok_offsets[t] = tok_first;
    if (w == W - 1 && lane == 63) tok_offsets[T] = tok_first + ct;
  }
  int j = tok_first;
  for (int p = 0; p < q; ++p) j += cnt[p][lane];
  for (int c0 = e_lo; c0 < e_hi; c0 += 64) {
    uint64_t words = words0, bits = bits0;
    int bases = bases0;
    if (c0 != e_lo) {
      const int el = c0 + lane;
      words = el < e_hi ? mask[(size_t)el * W + w] : 0ull;
      bases = el < e_hi ? offsets[el] + prefix[(size_t)el * W + w] : 0;
      bits = wave_transpose64(words, lane);
      if (!live) bits = 0;
    }
    while (__ballot(bits != 0)) {
      float v[kMetaBatch];
      int r[kMetaBatch], ex[kMetaBatch];
      bool hit[kMetaBatch];
#pragma unroll
      for (int u = 0; u < kMetaBatch; ++u) {
        hit[u] = bits != 0;
        const int i = hit[u] ? __ffsll((unsigned long long)bits) - 1 : 0;
        bits &= bits - 1;
        const uint64_t word = shfl_u64(words, i);  // expert c0 + i's mask word
        r[u] = __shfl(bases, i, kWave) + __popcll(word & below);
        ex[u] = c0 + i;
        v[u] = hit[u] ? scores_t[(size_t)(c0 + i) * T + t] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kMetaBatch; ++u) {
        if (hit[u]) {
          tok_rows[j++] = r[u];
          row_token[r[u]] = t;
          row_expert[r[u]] = ex[u];
          row_w[r[u]] = v[u] / dn;
        }
      }
    }
  }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_topk_route(const float* in, float* scores, float* scores_t, int32_t* topk_idx, float* topk_w,
                             uint64_t* mask, int T, int E, int K, int W, int do_softmax, hipStream_t s) {
  if (E <= 256) {
    // LDS beyond the default 64 KB of dynamic LDS is granted per kernel
#define SMOE_TOPK_LANE(KM, NW)                                                                                    \
  do {                                                                                                            \
    const size_t lds = topk_lane_lds(E, KM, NW);                                                                  \
    if (lds > 65536) {                                                                                            \
      const hipError_t e = hipFuncSetAttribute((const void*)topk_lane_kernel<KM, NW>,                             \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);            \
      if (e != hipSuccess) return e;                                                                              \
    }                                                                                                             \
    topk_lane_kernel<KM, NW><<<dim3(W), dim3(64 * NW), lds, s>>>(in, scores, scores_t, topk_idx, topk_w, mask, T, \
                                                                 E, K, W, do_softmax);                            \
  } while (0)
    // four waves per word when the experts split into four slices of whole float4s
    const bool four = E % 16 == 0;
    if (K <= 2) {
      if (four) SMOE_TOPK_LANE(2, 4); else SMOE_TOPK_LANE(2, 1);
    } else if (K <= 4) {
      if (four) SMOE_TOPK_LANE(4, 4); else SMOE_TOPK_LANE(4, 1);
    } else if (K <= 8) {
      if (four) SMOE_TOPK_LANE(8, 4); else SMOE_TOPK_LANE(8, 1);
    } else {
      if (four) SMOE_TOPK_LANE(16, 4); else SMOE_TOPK_LANE(16, 1);
    }
#undef SMOE_TOPK_LANE
    return hipGetLastError();
  }
  const dim3 grid(W), block(kTopkWaves * 64);
#define SMOE_TOPK(N)                                                                                               \
  if (E <= 64 * N) {                                                                                               \
    topk_route_kernel<N><<<grid, block, (size_t)E * 8, s>>>(in, scores, scores_t, topk_idx, topk_w, mask, T, E, K, \
                                                            W, do_softmax);                                        \
    return hipGetLastError();                                                                                      \
  }
  SMOE_TOPK(8)
  SMOE_TOPK(16)
  SMOE_TOPK(32)
  SMOE_TOPK(64)
#undef SMOE_TOPK
  return hipErrorInvalidValue;
}

hipError_t launch_topk_few(const float* in, int slices, const float* bias, float* logits, float* scores_t,
                           const moe_routing& r, int T, int E, int K, int do_softmax, bool counts_only, hipStream_t s) {
  const bool meta = T <= kFewOneGroup;
  const dim3 grid((T + kFewWaves - 1) / kFewWaves), block(64 * kFewWaves);
  // META: E * 12 + 16 K * 8 <= 14 KB; else the transposed scores: E * 68 <= 68 KB
  const size_t lds = meta ? (size_t)E * 12 + kFewWaves * K * 8 : scores_t ? (size_t)E * (kFewWaves + 1) * 4 : 16;
#define SMOE_FEW(N)                                                                                                  \
  if (E <= 64 * N) {                                                                                                 \
    if (meta) {                                                                                                      \
      topk_few_kernel<N, true><<<grid, block, lds, s>>>(in, slices, bias, logits, scores_t, r, T, E, K, do_softmax,  \
                                                        counts_only);                                                \
    } else {                                                                                                         \
      if (lds > 65536) {                                                                                             \
        const hipError_t e = hipFuncSetAttribute((const void*)topk_few_kernel<N, false>,                             \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);             \
        if (e != hipSuccess) return e;                                                                               \
      }                                                                                                              \
      topk_few_kernel<N, false><<<grid, block, lds, s>>>(in, slices, bias, logits, scores_t, r, T, E, K, do_softmax, \
                                                         counts_only);                                               \
    }                                                                                                                \
    return hipGetLastError();                                                                                        \
  }
  SMOE_FEW(1)
  SMOE_FEW(2)
  SMOE_FEW(4)
  SMOE_FEW(8)
  SMOE_FEW(16)
#undef SMOE_FEW
  return hipErrorInvalidValue;
}

hipError_t launch_tc_metadata_few(const moe_routing& r, int T, int E, int K, bool counts_only, hipStream_t s) {
  const size_t lds = (size_t)E * 16 + 64 * K * 8;  // <= 24 KB
  tc_metadata_few_kernel<<<dim3(r.words), dim3(1024), lds, s>>>(r, T, E, K, counts_only);
  return hipGetLastError();
}

hipError_t launch_tc_metadata(const moe_routing& r, int T, int E, int K, bool counts_only, hipStream_t s) {
  const int W = r.words;
  expert_scan_kernel<<<dim3(E), dim3(256), 0, s>>>(r.mask, r.mask_prefix, r.counts, W,
                                                   counts_only ? nullptr : r.status);
  if (counts_only) return hipGetLastError();
  tc_place_kernel<<<dim3((T + 255) / 256), dim3(256), (size_t)E * 4, s>>>(
      r.topk_idx, r.topk_w, r.mask, r.mask_prefix, r.counts, r.offsets, r.tok_offsets, r.tok_count, r.tok_rows,
      r.row_token, r.row_expert, r.row_w, T, E, K, W, r.status);
  return hipGetLastError();
}

hipError_t launch_metadata(const moe_routing& r, const float* scores_t, int T, int E, bool counted, hipStream_t s) {
  const int W = r.words;
  int32_t* word_sum = r.scratch + E + 64;  // [W]
  int32_t* word_base = word_sum + W + 1;   // [W + 1]
  if (!counted) expert_scan_kernel<<<dim3(E), dim3(256), 0, s>>>(r.mask, r.mask_prefix, r.counts, W, nullptr);
  // one extra workgroup turns the expert counts into offsets
  token_count_kernel<<<dim3(W + 1), dim3(64), 0, s>>>(r.mask, scores_t, r.tok_count, r.tok_denom, word_sum, r.counts,
                                                      r.offsets, T, E, W, r.status);
  // up to kPlaceSumWords words every placement workgroup sums the word sums
  // before it itself; beyond that a scan kernel provides the bases
  const bool scan_words = W > kPlaceSumWords;
  if (scan_words) scan_kernel<<<dim3(1), dim3(1024), 0, s>>>(word_sum, word_base, W);
  token_place_kernel<<<dim3(W), dim3(64 * kPlaceWaves), 0, s>>>(r.mask, r.mask_prefix, r.offsets, r.tok_count,
                                                                scan_words ? word_base : nullptr, word_sum,
                                                                r.tok_offsets, scores_t, r.tok_denom, r.tok_rows,
                                                                r.row_token, r.row_expert, r.row_w, T, E, W);
  return hipGetLastError();
}

}  // namespace smoe
