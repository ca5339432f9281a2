// Gating of single tokens: what the route kernels, the plan kernel (small batches) and the router kernel share.
#pragma once
#include "common.h"

namespace dsmoe {

struct RouteArgs {
  const float* logits;
  const float* tau;
  int32_t* idx;  // idx, w, keep: may be null (all three)
  float* w;
  uint8_t* keep;
  int32_t* bin_count;    // forward: [blocks][nbins] sort-bin histogram, one row per block (may be null)
  int bins;              // the sort bins are counted (in LDS, and from there to bin_count unless that is null)
  int32_t* group_count;  // stand-alone: [E*P] kept units per sub-expert (may be null)
  int32_t* sel;          // score histograms, or scores, in place of idx / w / keep (may be null); see launch_route_scores
  float* score;
  int T, E, K, P, lo, hi, renorm, nsub_bits, nsub, nhist;
};

// sort bin of a keep pattern inside its expert: patterns that keep the major partitions come first
__device__ __forceinline__ int sub_of_bits(int bits, int nsub_bits) {
  int rev = 0;
  for (int p = 0; p < nsub_bits; ++p) rev |= ((bits >> p) & 1) << (nsub_bits - 1 - p);
  return (1 << nsub_bits) - 1 - rev;
}

// tau: the [E][P] threshold table (in LDS)
__device__ __forceinline__ int keep_bits_of(float n, int e, const RouteArgs& a, const float* tau) {
  int bits = 0;
  if (e >= a.lo && e < a.hi) {
    if (!a.tau) return n >= 0.f ? (1 << a.P) - 1 : 0;
    for (int p = 0; p < a.P; ++p) bits |= (n >= tau[e * a.P + p] ? 1 : 0) << p;
  }
  return bits;
}

// histogram update of one pair into the block's LDS histogram
__device__ __forceinline__ void count_pair(int32_t* hist, int bits, int e, const RouteArgs& a) {
  if (bits == 0) return;
  if (a.bins) atomicAdd(&hist[(e - a.lo) * a.nsub + sub_of_bits(bits, a.nsub_bits)], 1);
  if (a.group_count) {
    int32_t* h2 = hist + (a.bins ? (a.hi - a.lo) * a.nsub : 0);
    for (int p = 0; p < a.P; ++p)
      if ((bits >> p) & 1) atomicAdd(&h2[e * a.P + p], 1);
  }
}

// One pair's results: routing outputs and sort-bin histogram, or its place in the score histograms.  There the bins are
// spread (two pairs of a wavefront rarely meet in one), while the pair counts of a few experts are not: those are
// collected in LDS.  (One global atomic per pair on them took 150 us for 32 k pairs over 8 experts.)
// MODE: what becomes of the pairs (decided outside the kernels: a branch per pair cost the large batches 1 us)
enum { kRoute, kScores, kRouteInLds };
// pairs (kRouteInLds; may be null): expert << 8 | keep pattern of every pair, in LDS
template <int MODE>
__device__ __forceinline__ void finish_pair(const RouteArgs& a, int32_t* hist, int32_t* pairs, const float* tau, int t, int k, int e, float n,
                                            float s) {
  if (MODE == kScores && a.sel) {
    int b = (int)floorf(n * (float)kSelBins);
    b = b < 0 ? 0 : (b > kSelBins ? kSelBins : b);
    atomicAdd(&a.sel[(size_t)e * kSelRow + b], 1);
    atomicAdd(&hist[e], 1);
    return;
  }
  if (MODE == kScores) {
    a.score[(size_t)t * a.K + k] = e >= a.lo && e < a.hi ? n : -1.f;
    return;
  }
  const int bits = keep_bits_of(n, e, a, tau);
  const size_t o = (size_t)t * a.K + k;
  if (MODE == kRoute || a.idx) {
    a.idx[o] = e;
    a.w[o] = a.renorm ? n : s;
    a.keep[o] = (uint8_t)bits;
  }
  if (MODE == kRouteInLds && pairs) pairs[o] = e << 8 | bits;
  count_pair(hist, bits, e, a);
}
// the block's LDS histogram leaves
__device__ __forceinline__ void flush_hist(const RouteArgs& a, const int32_t* hist, int threads) {
  const int nb = a.bins ? (a.hi - a.lo) * a.nsub : 0;
  for (int i = threadIdx.x; i < a.nhist; i += threads) {
    const int c = hist[i];
    if (i < nb) a.bin_count[(size_t)blockIdx.x * nb + i] = c;  // this block's row of the histogram: no atomics
    else if (c) atomicAdd(a.sel ? &a.sel[(size_t)i * kSelRow + kSelBins + 1] : &a.group_count[i - nb], c);
  }
}

// Sixteen lanes per token (one row of the wavefront), NCH * 4 logits per lane: lane r of the row
// holds experts 64c + 4r .. 64c + 4r + 3 of every chunk c of 64 experts (16-byte loads, 256
// contiguous bytes per row and chunk).  All reductions stay inside a row: four data-parallel
// steps (mirror, half mirror, two quad permutations) leave the result in every lane, with no
// scalar round trip, and the four rows of a wavefront work on four tokens at once.  U tokens per
// row are carried through every step together so that their dependency chains overlap.
// A block is WV wavefronts = WV * 4 * U tokens.
__device__ __forceinline__ int row_min(int v) {
  v = min(v, dpp_all<kRowMirror>(v));
  v = min(v, dpp_all<kRowHalfMirror>(v));
  v = min(v, dpp_all<kQuadSwap2>(v));
  v = min(v, dpp_all<kQuadSwap1>(v));
  return v;
}

// What route_row_tokens needs in LDS: hist cleared, and the threshold table fetched (together with the logits, not after the scores
// are known).  The barrier that publishes both sits right before their first use, after the scores.
__device__ __forceinline__ void route_row_setup(const RouteArgs& a, int32_t* hist, float* tau_l, int threads) {
  for (int i = threadIdx.x; i < a.nhist; i += threads) hist[i] = 0;
  if (a.tau)
    for (int i = threadIdx.x; i < a.E * a.P; i += threads) tau_l[i] = a.tau[i];
}
// The block's tokens [t_first, t_end), whose logits start at `logits`; ends with every thread past its own updates of hist (no barrier
// after them).
template <int NCH, int U, int WV, int MODE>
__device__ __forceinline__ void route_row_tokens(const RouteArgs& a, const float* logits, int t_first, int t_end, int32_t* hist, const float* tau_l,
                                                 int32_t* pairs) {
  constexpr int V = NCH * 4;
  const int r = threadIdx.x & 15, row = threadIdx.x >> 4;  // lane in its row; row in the block (WV * 4 of them)
  auto token = [&](int u) { return t_first + u * (WV * 4) + row; };
  auto expert = [&](int j) { return 64 * (j >> 2) + 4 * r + (j & 3); };
  int rank[U][V];
  float sc[U][V], ssum[U];
  // (a wavefront without a token leaves the units to the others: in a batch of one the sixteen of the small plan kernel shared them,
  // 1 token on 64 experts of 2048 x 1024 45.7 -> 43.9 us)
  if (t_first + (int)(threadIdx.x >> 6) * 4 < t_end) {
    float l[U][V];
    const bool vec = (a.E & 3) == 0;  // rows of the logits are 16-byte aligned
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = token(u);
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int e0 = 64 * c + 4 * r;
        float4 v = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        if (t < t_end) {
          const float* src = logits + (size_t)(t - t_first) * a.E + e0;
          if (vec) {
            if (e0 < a.E) v = *(const float4*)src;
          } else {
            if (e0 + 0 < a.E) v.x = src[0];
            if (e0 + 1 < a.E) v.y = src[1];
            if (e0 + 2 < a.E) v.z = src[2];
            if (e0 + 3 < a.E) v.w = src[3];
          }
        }
        // a NaN logit ranks last, so every round below finds a winner
        l[u][4 * c + 0] = v.x != v.x ? -INFINITY : v.x;
        l[u][4 * c + 1] = v.y != v.y ? -INFINITY : v.y;
        l[u][4 * c + 2] = v.z != v.z ? -INFINITY : v.z;
        l[u][4 * c + 3] = v.w != v.w ? -INFINITY : v.w;
      }
    }
    float m[U], z[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v = l[u][0];
#pragma unroll
      for (int j = 1; j < V; ++j) v = fmaxf(v, l[u][j]);
      m[u] = row_max(v);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v = 0.f;
#pragma unroll
      for (int j = 0; j < V; ++j)
        if (expert(j) < a.E) v += expf(l[u][j] - m[u]);
      z[u] = row_sum(v);
    }
    // Top-K in K rounds of "largest logit not yet taken, lowest expert id among equals" (Eq. 2): the
    // row's maximum, then the row's smallest expert id among the lanes that hold it; slot k of the
    // token is round k's winner.  rank = slot of a selected logit, a.K for the others.
    uint32_t taken[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      taken[u] = 0;
#pragma unroll
      for (int j = 0; j < V; ++j) {
        rank[u][j] = a.K;
        if (expert(j) >= a.E) taken[u] |= 1u << j;
      }
    }
    for (int k = 0; k < a.K; ++k) {
      float g[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float v = -INFINITY;
#pragma unroll
        for (int j = 0; j < V; ++j) v = fmaxf(v, (taken[u] >> j) & 1 ? -INFINITY : l[u][j]);
        g[u] = row_max(v);
      }
      int win[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int cand = 0x7fffffff;
#pragma unroll
        for (int j = V - 1; j >= 0; --j)  // expert ids grow with j: the last assignment is the smallest
          if (!((taken[u] >> j) & 1) && l[u][j] == g[u]) cand = expert(j);
        win[u] = row_min(cand);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int j = 0; j < V; ++j)
          if (expert(j) == win[u]) {
            rank[u][j] = k;
            taken[u] |= 1u << j;
          }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v = 0.f;
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const bool selq = expert(j) < a.E && rank[u][j] < a.K;
        sc[u][j] = selq ? expf(l[u][j] - m[u]) / z[u] : 0.f;  // Eq. 1
        v += sc[u][j];
      }
      ssum[u] = row_sum(v);
    }
  }
  __syncthreads();  // hist is cleared and tau_l is complete (route_row_setup)
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = token(u);
    if (t >= t_end) continue;
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int e = expert(j);
      if (e < a.E && rank[u][j] < a.K) {
        const float n = sc[u][j] / ssum[u];  // Sec. 4.1: normalise over the K selected
        finish_pair<MODE>(a, hist, pairs, tau_l, t, rank[u][j], e, n, sc[u][j]);
      }
    }
  }
}
inline void set_route_layer(const Layout& L, RouteArgs& a) {
  a.E = L.E;
  a.K = L.K;
  a.P = L.P;
  a.lo = L.lo;
  a.hi = L.hi;
  a.renorm = L.renorm;
  a.nsub = L.nsub;
  a.nsub_bits = L.P < kSubBits ? L.P : kSubBits;
  a.bins = a.bins || a.bin_count;
  a.nhist = a.sel ? L.E : (a.bins ? L.nbins : 0) + (a.group_count ? L.E * L.P : 0);
}

}  // namespace dsmoe
