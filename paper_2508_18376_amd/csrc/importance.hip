// Neuron importance profiling and reconstruction order (paper Sec. 4.2 b).
//
// GEMM-1 is run over the calibration tokens with every routed pair kept.  On the matrix-core path
// its epilogue sums the chosen metric over the rows of each tile and this file adds the tiles of an
// expert; on the full-precision path GEMM-1 stores the metric per (row, neuron) in fp32 and the rows of each
// expert are summed here (one thread per neuron, rows in order).  Both are deterministic.  An
// importance vector is turned into the permutation "neurons by descending importance, equal values
// by ascending id".
#include "common.h"

namespace dsmoe {

// importance[e][q] = sum over the rows of expert e of its column of H (the packed weights must have been
// made with the identity permutation, so neuron j of partition p is original neuron p * F/P + j)
// unscale: 2^-h_shift for the metrics that contain the up projection (the packed W3 carries 2^h_shift), else 1
__global__ __launch_bounds__(256) void colsum_kernel(Layout L, const char* ws, float* importance, float unscale) {
  const int e = blockIdx.y;
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= L.F) return;
  const int32_t* exp_nrows = (const int32_t*)(ws + L.o_exp_nrows);
  const int32_t* exp_row0 = (const int32_t*)(ws + L.o_exp_row0);
  const float* H = (const float*)(ws + L.o_H) + q / L.Fp * L.Fpk + q % L.Fp;
  const int n = exp_nrows[e];
  const size_t r0 = (size_t)(exp_row0[e] - L.sh_rows);
  // rows are added in order (deterministic); eight loads are in flight at a time
  float acc = 0.f;
  int r = 0;
  for (; r + 8 <= n; r += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = H[(r0 + r + u) * L.Fh];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; r < n; ++r) acc += H[(r0 + r) * L.Fh];
  importance[(size_t)e * L.F + q] = acc * unscale;
}

// MFMA path: the GEMM-1 profiling pass has left one row of F column sums per row tile where the layer
// keeps H; importance[e][q] = the sum of the rows of expert e's tiles, in tile order (deterministic).
__global__ __launch_bounds__(256) void colsum_tiles_kernel(Layout L, const char* ws, float* importance, float unscale) {
  const int e = blockIdx.y;
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= L.F) return;
  const int32_t* exp_nrows = (const int32_t*)(ws + L.o_exp_nrows);
  const int32_t* exp_row0 = (const int32_t*)(ws + L.o_exp_row0);
  const float* table = (const float*)(ws + L.o_H);
  const int nt = (exp_nrows[e] + L.BM - 1) / L.BM;
  const size_t t0 = (size_t)((exp_row0[e] - L.sh_rows) / L.BM);
  float acc = 0.f;
  for (int i = 0; i < nt; ++i) acc += table[(t0 + i) * L.F + q];
  importance[(size_t)e * L.F + q] = acc * unscale;
}

hipError_t launch_colsum(const Layout& L, const char* ws, int metric, float* importance, hipStream_t s) {
  dim3 grid((L.F + 255) / 256, L.E_res), block(256);
  const float unscale = metric >= 2 ? ldexpf(1.f, -L.h_shift) : 1.f;
  if (!L.mfma) colsum_kernel<<<grid, block, 0, s>>>(L, ws, importance, unscale);  // the full-precision path keeps H
  else colsum_tiles_kernel<<<grid, block, 0, s>>>(L, ws, importance, unscale);
  return hipGetLastError();
}

// perm[e][rank(q)] = q with rank(q) = #{q' : imp[q'] > imp[q], or equal and q' < q}.  A NaN importance
// counts as minus infinity (such neurons come last, by id), so the result is a permutation whatever the input.
// F^2 comparisons per expert, two vector operations each; what it costs beyond them is waiting for LDS, so four values come with
// each (broadcast) read, and the id only takes part next to the workgroup's own neurons: in front of them equal
// values rank higher, behind them lower.  A workgroup is twice its 256 neurons, each group of 256 threads with every other
// block of 256 values: one wavefront to a SIMD waited for each read and for the chain of its own additions.  One group -> two -> four,
// us a call: 64 experts of 1024 neurons 16.0 -> 10.9 -> 10.0, of 1408 22.5 -> 19.3 -> 23.7, 8 of 14336 156 -> 127 -> 135.
constexpr int kRankNeurons = 256, kRankParts = 2;
__global__ __launch_bounds__(kRankNeurons * kRankParts) void perm_rank_kernel(int F, const float* importance, int32_t* perm) {
  __shared__ float4 tile[kRankParts][kRankNeurons / 4];
  __shared__ int32_t others[kRankParts][kRankNeurons];
  const int e = blockIdx.y, part = __builtin_amdgcn_readfirstlane(threadIdx.x / kRankNeurons), own = threadIdx.x % kRankNeurons;
  const float* imp = importance + (size_t)e * F;
  const int q = blockIdx.x * kRankNeurons + own;
  auto key = [](float v) { return v != v ? -INFINITY : v; };
  const float mine = q < F ? key(imp[q]) : 0.f;
  int rank = 0, rank2 = 0;
  for (int base = 0; base < F; base += kRankNeurons * kRankParts) {
    __syncthreads();
    ((float*)tile)[threadIdx.x] = base + (int)threadIdx.x < F ? key(imp[base + threadIdx.x]) : -INFINITY;  // ranks above nothing
    __syncthreads();
    const int block = base / kRankNeurons + part;  // whose neurons this group's 256 values belong to
    const float4* v = tile[part];
    if (block * kRankNeurons >= F) {  // none
    } else if (block < (int)blockIdx.x) {
#pragma unroll 8
      for (int i = 0; i < kRankNeurons / 4; ++i) {
        const float4 o = v[i];
        rank += (o.x >= mine) + (o.y >= mine);
        rank2 += (o.z >= mine) + (o.w >= mine);
      }
    } else if (block == (int)blockIdx.x) {
#pragma unroll 4
      for (int i = 0; i < kRankNeurons / 4; ++i) {
        const float4 o = v[i];
        const int before = own - 4 * i;  // values of the group with a smaller id
        rank += (int)(o.x > mine) | ((int)(o.x == mine) & (int)(before > 0));
        rank2 += (int)(o.y > mine) | ((int)(o.y == mine) & (int)(before > 1));
        rank += (int)(o.z > mine) | ((int)(o.z == mine) & (int)(before > 2));
        rank2 += (int)(o.w > mine) | ((int)(o.w == mine) & (int)(before > 3));
      }
    } else {
#pragma unroll 8
      for (int i = 0; i < kRankNeurons / 4; ++i) {
        const float4 o = v[i];
        rank += (o.x > mine) + (o.y > mine);
        rank2 += (o.z > mine) + (o.w > mine);
      }
    }
  }
  others[part][own] = rank + rank2;
  __syncthreads();
  if (part || q >= F) return;
  rank = others[0][own];
  for (int i = 1; i < kRankParts; ++i) rank += others[i][own];
  perm[(size_t)e * F + rank] = q;
}

hipError_t launch_perm_from_importance(const Layout& L, const float* importance, int32_t* perm, hipStream_t s) {
  dim3 grid((L.F + kRankNeurons - 1) / kRankNeurons, L.E_res), block(kRankNeurons * kRankParts);
  perm_rank_kernel<<<grid, block, 0, s>>>(L.F, importance, perm);
  return hipGetLastError();
}

}  // namespace dsmoe
