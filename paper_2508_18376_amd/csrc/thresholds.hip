// Load-aware threshold selection on the device (Sec. 4.3 of the paper) and the map from a row
// budget to a threshold through the distribution of the normalised scores (Sec. 5.3.3 notes that
// the threshold <-> drop-rate relation is not linear).
//
// Input are histograms of the normalised scores n that a routing pass over the whole router, with nothing dropped,
// leaves: sel[e][0 .. kSelBins] counts floor(n * kSelBins) over the pairs of expert e (n = 1 falls
// into the last bin), sel[e][kSelBins+1] is the pair count of e.  Because kSelBins is a power of two, n * kSelBins is
// exact in fp32 and "n >= b / kSelBins" is the same decision as "bin(n) >= b": suffix sums of the histogram are the
// exact row counts the layer would keep at the grid thresholds.
//
// Both picks are latency: short scans over 4097 bins.  Wavefront scans and one pass of candidates per thread take
// the place of barriers per scan step and of a single thread's searches and stores (see the figures at the launchers).
#include "common.h"

namespace dsmoe {

// inclusive scan over the lanes of a wavefront
__device__ __forceinline__ int wave_incl(int v) {
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if ((int)(threadIdx.x & 63) >= o) v += u;
  }
  return v;
}

// One workgroup per expert.
__global__ __launch_bounds__(256) void tau_pick_kernel(const int32_t* __restrict__ sel, const float* __restrict__ tau_max, int T,
                                                       int E, int K, int P, int G, int row_cap, float* __restrict__ tau,
                                                       int32_t* __restrict__ pair_count) {
  __shared__ int32_t wtot[4], s_bin;
  __shared__ int32_t s_load;
  const int e = blockIdx.x, tid = threadIdx.x;
  const int32_t* h = sel + (int64_t)e * kSelRow;
  constexpr int per = kSelBins / 256;  // bins [tid*per, tid*per+per); the last bin (n = 1) belongs to thread 255
  if (tid == 0) s_bin = s_load = 0;
  int hb[per], sum = 0;
  if (row_cap > 0) {
#pragma unroll
    for (int j = 0; j < per; ++j) hb[j] = h[tid * per + j];
#pragma unroll
    for (int j = 0; j < per; ++j) sum += hb[j];
    if (tid == 255) sum += h[kSelBins];
  }
  const int incl = wave_incl(sum);
  if ((tid & 63) == 63) wtot[tid >> 6] = incl;
  __syncthreads();
  // load ratio of the device that holds this expert
  const int d0 = (e / G) * G;
  int load = 0;
  for (int j = tid; j < G; j += 256) load += sel[(int64_t)(d0 + j) * kSelRow + kSelBins + 1];
  if (load) atomicAdd(&s_load, load);
  if (row_cap > 0) {  // smallest b with (pairs of e whose bin >= b) <= row_cap
    int above = wtot[0] + wtot[1] + wtot[2] + wtot[3] - incl;  // pairs in the bins above this thread's
    for (int q = 0; q < (tid >> 6); ++q) above -= wtot[q];
    if (above <= row_cap && above + sum > row_cap) {  // the crossing lies among this thread's bins: exactly one thread
      int s = above, b = tid * per;
      bool past = false;  // the crossing has been met
      if (tid == 255) {
        const int last = h[kSelBins];
        if (s + last > row_cap) past = true, b = kSelBins + 1;
        s += last;
      }
#pragma unroll
      for (int j = per - 1; j >= 0; --j) {
        if (!past && s + hb[j] > row_cap) past = true, b = tid * per + j + 1;
        s += hb[j];
      }
      s_bin = b;
    }
  }
  __syncthreads();
  if (tid == 0) {
    // one rounding per operation (the multiply must not fuse with the subtraction below)
#pragma clang fp contract(off)
    const float ideal = (float)((int64_t)T * K * G) / (float)E;
    const float r = (float)s_load / ideal;
    const float scale = r < 1.f ? r : 1.f;
    float lowest = INFINITY;
    for (int p = 0; p < P; ++p) {
      const float v = tau_max[p] * scale;
      lowest = v < lowest ? v : lowest;
    }
    const float floor_e = (float)s_bin / (float)kSelBins;
    for (int p = 0; p < P; ++p) {
      float v = tau_max[p] * scale;
      if (floor_e > lowest) v = floor_e + (v - lowest);
      tau[e * P + p] = v;
    }
    if (pair_count) pair_count[e] = h[kSelBins + 1];
  }
}

// 8 experts, 16384 tokens, row cap: 170 us for the two clearing, routing, counting and picking launches before, now
// clear 5, route + count 9, pick 5 us
hipError_t launch_select_thresholds(const Layout& L, int T, const float* logits, const float* tau_max, int group_size, int row_cap, char* ws,
                                    float* tau, int32_t* pair_count, hipStream_t s) {
  int32_t* sel = (int32_t*)(ws + L.o_sel);
  hipError_t e = launch_fill_i32(sel, (int64_t)L.E * kSelRow, 0, s);
  if (e == hipSuccess) e = launch_route_scores(L, logits, T, sel, nullptr, s);
  if (e != hipSuccess) return e;
  tau_pick_kernel<<<dim3(L.E), dim3(256), 0, s>>>(sel, tau_max, T, L.E, L.K, L.P, group_size, row_cap, tau, pair_count);
  return hipGetLastError();
}

// Thresholds for a target drop rate (Sec. 5.3.3: the relation between threshold and drop rate is
// read off the batch's own score distribution; Sec. 4.2 c: the partitions keep fixed offsets).
// Histogram of floor(n * kSelBins) over the resident pairs, in kSelBlocks parts: each workgroup counts its share in LDS and
// writes one row.  (Global atomics of all pairs on the thousand bins they fall into took 15 us, from inside the
// routing kernel 23 us.)
__global__ __launch_bounds__(1024) void score_hist_kernel(const float* __restrict__ n, int64_t npairs, int32_t* __restrict__ rows) {
  __shared__ int32_t h[kSelBins + 1];
  const int tid = threadIdx.x;
  for (int i = tid; i <= kSelBins; i += 1024) h[i] = 0;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * 1024 + tid; i < npairs; i += (int64_t)gridDim.x * 1024) {
    const float v = n[i];
    if (v != -1.f) {
      const int b = (int)floorf(v * (float)kSelBins);
      atomicAdd(&h[b < 0 ? 0 : (b > kSelBins ? kSelBins : b)], 1);
    }
  }
  __syncthreads();
  for (int i = tid; i <= kSelBins; i += 1024) rows[(size_t)blockIdx.x * kSelRow + i] = h[i];
}

// h = histogram of floor(n * kSelBins) over the resident pairs.  Unit (pair, p) is dropped iff
// n < (b + off[p]) / kSelBins, i.e. iff bin(n) < b + off[p]: with C(x) = pairs whose bin is below x,
// the dropped units at centre b are sum_p C(b + off[p]).  One workgroup: prefix counts in LDS, then
// the smallest b with at least `need` dropped units (the count grows with b): every thread tries a few b.
struct DropRateArgs {
  int32_t off[kMaxPart];
  int P, E;
  double rate;
};
__global__ __launch_bounds__(1024) void drop_rate_pick_kernel(const int32_t* __restrict__ rows, int nrows, DropRateArgs a,
                                                              float* __restrict__ tau, int32_t* __restrict__ stats) {
  __shared__ int32_t below[kSelBins + 2];  // below[x] = pairs with bin < x, x = 0 .. kSelBins+1
  __shared__ int32_t wtot[16], s_b, s_last;
  const int tid = threadIdx.x, wv = tid >> 6;
  constexpr int per = 4;  // bins of a thread; thread 1023 also has the last one (n = 1)
  static_assert(per * 1024 == kSelBins, "bins per thread");
  // added up over the parts of the histogram, all of whose loads are in flight together
  int hb[per] = {}, last = tid < nrows ? rows[(size_t)tid * kSelRow + kSelBins] : 0, sum = 0;
  int4 v[kSelBlocks];
#pragma unroll
  for (int r = 0; r < kSelBlocks; ++r) v[r] = r < nrows ? *(const int4*)(rows + (size_t)r * kSelRow + tid * per) : make_int4(0, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < kSelBlocks; ++r) {
    hb[0] += v[r].x;
    hb[1] += v[r].y;
    hb[2] += v[r].z;
    hb[3] += v[r].w;
  }
  if (wv == 0) {
    for (int o = kSelBlocks / 2; o > 0; o >>= 1) last += __shfl_xor(last, o, 64);
    if (tid == 0) s_last = last;
  }
#pragma unroll
  for (int j = 0; j < per; ++j) sum += hb[j];
  const int incl = wave_incl(sum);
  if ((tid & 63) == 63) wtot[wv] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int q = 0; q < wv; ++q) run += wtot[q];
#pragma unroll
  for (int j = 0; j < per; ++j) {
    below[tid * per + j] = run;
    run += hb[j];
  }
  if (tid == 1023) {
    below[kSelBins] = run;
    below[kSelBins + 1] = run + s_last;
  }
  int omax = a.off[0], omin = a.off[0];
  for (int p = 1; p < a.P; ++p) {
    omax = max(omax, a.off[p]);
    omin = min(omin, a.off[p]);
  }
  const int b_lo = -omax, b_hi = kSelBins + 1 - omin;  // nothing dropped .. everything dropped
  if (tid == 0) s_b = b_hi;
  __syncthreads();
  const int pairs = below[kSelBins + 1];
  auto dropped = [&](int b) {
    int d = 0;
    for (int p = 0; p < a.P; ++p) {
      const int x = b + a.off[p];
      d += x <= 0 ? 0 : (x > kSelBins + 1 ? pairs : below[x]);
    }
    return d;
  };
  const double need = a.rate * ((double)pairs * a.P);
  for (int b = b_lo + tid; b < b_hi; b += 1024)
    if ((double)dropped(b) >= need) {  // a thread's first hit is its smallest
      atomicMin(&s_b, b);
      break;
    }
  __syncthreads();
  const int b = s_b;
  for (int i = tid; i < a.E * a.P; i += 1024) tau[i] = (float)(b + a.off[i % a.P]) / (float)kSelBins;
  if (tid == 0 && stats) {
    stats[0] = dropped(b);
    stats[1] = pairs * a.P;
  }
}

// 64 experts, 7001 tokens: 52 us in five launches before, now route 10, histogram 5, pick 11 us
hipError_t launch_drop_rate_thresholds(const Layout& L, int T, const float* logits, double rate, const int32_t* offset_bins, char* ws, float* tau,
                                       int32_t* stats, hipStream_t s) {
  int32_t* rows = (int32_t*)(ws + L.o_sel);
  float* n = (float*)(ws + L.o_w);
  const int64_t npairs = (int64_t)T * L.K;
  int nrows = 0;
  if (npairs > 0) {
    nrows = npairs > 1024 * kSelBlocks ? kSelBlocks : (int)((npairs + 1023) / 1024);
    hipError_t e = launch_route_scores(L, logits, T, nullptr, n, s);
    if (e != hipSuccess) return e;
    score_hist_kernel<<<dim3(nrows), dim3(1024), 0, s>>>(n, npairs, rows);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  DropRateArgs a;
  for (int p = 0; p < kMaxPart; ++p) a.off[p] = p < L.P ? offset_bins[p] : 0;
  a.P = L.P;
  a.E = L.E;
  a.rate = rate;
  drop_rate_pick_kernel<<<dim3(1), dim3(1024), 0, s>>>(rows, nrows, a, tau, stats);
  return hipGetLastError();
}

}  // namespace dsmoe
