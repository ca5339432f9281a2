// Gating + drop mask, row-list construction (histogram, scan, scatter) and the combine kernel.
//
// Gating follows Eq. 1-2 of the paper (softmax over all E logits, Top-K), the mask follows
// Sec. 4.1 / 4.2 c (normalise the K selected scores, keep unit (t,k,p) iff n >= tau[e][p]).
// The row lists realise the index remap of Sec. 3.2 without materialising K*P lists: the pairs of
// one expert are sorted by their keep pattern, so the rows that need sub-expert p are (for
// thresholds that grow with p) a prefix of the expert's list.
#include "route.h"

namespace dsmoe {

// ------------------------------------------------------------------------------------- fill
__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(p, n, v);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------- route
// One lane per token; all E logits of the token live in that lane's registers (E <= EPAD <= 32).
// tau: the threshold table in LDS.  All threads of the workgroup take part: the barrier that publishes it and the cleared histogram sits right
// before their first use, so that the table is fetched together with the logits.
template <int EPAD, int KMAX, int MODE>
__device__ __forceinline__ void route_lane_token(const RouteArgs& a, int t, int32_t* hist, int32_t* pairs, const float* tau) {
  float sk[KMAX], sel = 0.f;
  int ik[KMAX];
  if (t < a.T) {
    float l[EPAD];
#pragma unroll
    for (int e = 0; e < EPAD; ++e) l[e] = (e < a.E) ? a.logits[(size_t)t * a.E + e] : -INFINITY;
    float m = l[0];
#pragma unroll
    for (int e = 1; e < EPAD; ++e) m = (e < a.E && l[e] > m) ? l[e] : m;
    float z = 0.f;
#pragma unroll
    for (int e = 0; e < EPAD; ++e)
      if (e < a.E) z += expf(l[e] - m);
    // Top-K: K rounds of "largest not yet taken"; a later index wins only if strictly larger.
    unsigned long long taken = 0ull;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      sk[k] = 0.f;
      ik[k] = 0;
      if (k < a.K) {
        float bv = 0.f;
        int be = -1;
#pragma unroll
        for (int e = 0; e < EPAD; ++e) {
          bool free_e = (e < a.E) && !((taken >> e) & 1ull);
          if (free_e && (be < 0 || l[e] > bv)) {
            bv = l[e];
            be = e;
          }
        }
        taken |= 1ull << be;
        ik[k] = be;
        sk[k] = expf(bv - m) / z;  // Eq. 1
        sel += sk[k];
      }
    }
  }
  __syncthreads();
  if (t >= a.T) return;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    if (k < a.K) {
      const float n = sk[k] / sel;  // Sec. 4.1: normalise over the K selected
      finish_pair<MODE>(a, hist, pairs, tau, t, k, ik[k], n, sk[k]);
    }
  }
}
template <int EPAD, int KMAX, int MODE>
__global__ __launch_bounds__(64) void route_lane_kernel(RouteArgs a) {
  extern __shared__ int32_t hist[];
  float* tau_l = (float*)(hist + a.nhist);
  if (a.tau)
    for (int i = threadIdx.x; i < a.E * a.P; i += 64) tau_l[i] = a.tau[i];
  for (int i = threadIdx.x; i < a.nhist; i += 64) hist[i] = 0;
  route_lane_token<EPAD, KMAX, MODE>(a, blockIdx.x * 64 + threadIdx.x, hist, nullptr, tau_l);
  __syncthreads();
  flush_hist(a, hist, 64);
}

template <int NCH, int U, int WV, int MODE>
__global__ __launch_bounds__(WV * 64) void route_row_kernel(RouteArgs a) {
  extern __shared__ int32_t hist[];
  float* tau_l = (float*)(hist + a.nhist);
  const int t_first = (int)blockIdx.x * (WV * 4 * U);
  route_row_setup(a, hist, tau_l, WV * 64);
  route_row_tokens<NCH, U, WV, MODE>(a, a.logits + (size_t)t_first * a.E, t_first, min(a.T, t_first + WV * 4 * U), hist, tau_l, nullptr);
  __syncthreads();
  flush_hist(a, hist, WV * 64);
}

template <int MODE>
static hipError_t launch_route_kernel(const Layout& L, RouteArgs a, hipStream_t s) {
  const int T = a.T;
  if (T <= 0) return hipSuccess;
  set_route_layer(L, a);
  const size_t sh = sizeof(int32_t) * (size_t)(a.nhist + L.E * L.P);  // histogram + (row kernel) threshold table
  if (L.E <= 32) {  // few experts: a lane per token, no cross-lane traffic
    dim3 grid((T + 63) / 64), block(64);
    if (L.E <= 8) route_lane_kernel<8, 8, MODE><<<grid, block, sh, s>>>(a);
    else if (L.E <= 16) route_lane_kernel<16, 16, MODE><<<grid, block, sh, s>>>(a);
    else route_lane_kernel<32, 16, MODE><<<grid, block, sh, s>>>(a);
  } else if (T > kWaveSmallBatch) {  // many experts: sixteen lanes per token, 64 tokens per block
    dim3 grid((T + kRouteBlockTokens - 1) / kRouteBlockTokens);
    if (L.E <= 64) route_row_kernel<1, 1, 16, MODE><<<grid, dim3(1024), sh, s>>>(a);
    else if (L.E <= 128) route_row_kernel<2, 1, 16, MODE><<<grid, dim3(1024), sh, s>>>(a);
    else if (L.E <= 256) route_row_kernel<4, 1, 16, MODE><<<grid, dim3(1024), sh, s>>>(a);
    else route_row_kernel<8, 1, 16, MODE><<<grid, dim3(1024), sh, s>>>(a);
  } else {  // small batch: 16 tokens per block, one per row of four wavefronts
    dim3 grid((T + kWaveBlockTokens - 1) / kWaveBlockTokens), block(256);
    if (L.E <= 64) route_row_kernel<1, 1, 4, MODE><<<grid, block, sh, s>>>(a);
    else if (L.E <= 128) route_row_kernel<2, 1, 4, MODE><<<grid, block, sh, s>>>(a);
    else if (L.E <= 256) route_row_kernel<4, 1, 4, MODE><<<grid, block, sh, s>>>(a);
    else route_row_kernel<8, 1, 4, MODE><<<grid, block, sh, s>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_route(const Layout& L, const float* logits, int T, const float* tau, int32_t* idx, float* w,
                        uint8_t* keep, int32_t* bin_count, int32_t* group_count, hipStream_t s) {
  RouteArgs a = {};
  a.logits = logits;
  a.tau = tau;
  a.idx = idx;
  a.w = w;
  a.keep = keep;
  a.bin_count = bin_count;
  a.group_count = group_count;
  a.T = T;
  return launch_route_kernel<kRoute>(L, a, s);
}

hipError_t launch_route_scores(const Layout& L, const float* logits, int T, int32_t* sel, float* n, hipStream_t s) {
  RouteArgs a = {};
  a.logits = logits;
  a.sel = sel;
  a.score = n;
  a.T = T;
  return launch_route_kernel<kScores>(L, a, s);
}

// ------------------------------------------------------------------------------------- plan
// Turns the bin histogram into row offsets, the row lists and the two work lists of the grouped GEMMs, all in one launch: workgroup 0
// writes the GEMM-2 list, workgroup 1 the GEMM-1 list, the others the row lists; small batches are routed here as well.  Every workgroup
// works the tables that it needs out for itself.  Everything stays on the device: the GEMM grids are sized for the worst case and
// read their item count from the counters this kernel writes.
//
// The kernel is latency and nothing else: one workgroup's chain of memory and LDS round trips, barriers and instructions that a single compute unit
// issues.  So the chain is short: one wavefront makes the table of the experts (lane = expert, scans in registers) while the others
// count the tiles of the (expert, partition) groups, and whatever depends on an expert's sort bins (rows of a tile that keep a
// partition, a tile's place among those that do) is worked out from the bins' counts in one loop, by one thread.
constexpr int kPlanThreads = 1024;
constexpr int kPlanTilesLds = 2048;   // row tiles whose experts fit in the plan kernel's LDS (beyond: a search)
constexpr int kPlanRecords = kPlanThreads - 64;  // (row tile, partition) pairs that are looked at in one go
constexpr int kHalvedMost = kSplitItems / 2;  // GEMM-1 items of a last round that may be cut in two
constexpr int kLanePlanPairs = 2048;  // routed here with a lane per token: up to so many pairs (and tokens a workgroup has threads for)
constexpr int kRowPlanTokens = 64;    // with sixteen lanes per token: what one workgroup routes at once
constexpr int kListPairs = 4;         // pairs per thread of a workgroup that writes row lists

// the plan kernel's tables (in the order in which it lays them out)
__host__ __device__ inline int plan_lds_words(const Layout& L) {
  const int E_tot = L.E_res + (L.n_shared > 0 ? 1 : 0), NG = E_tot * L.P;
  const int groups = 2 * NG > L.nbins ? 2 * NG : L.nbins;  // (the workgroups with the row lists keep the next row of every bin there)
  return ((L.nbins + 3) & ~3) + ((3 * E_tot + 3) & ~3) + ((groups + 3) & ~3) + kPlanTilesLds / 2 + kPlanRecords * 4 + kHalvedMost * (int)(sizeof(Item1) / 4);
}
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
constexpr int kSumWords = 8192;  // partial column sums of the histograms (LANES == 0), behind the tables

// inclusive sum over the lanes of a wavefront, in registers
__device__ __forceinline__ int wave_incl_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // from 1, 2, 4, 8 lanes before, inside a row of sixteen
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // the last lane of rows 0 and 2 to the rows after them
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // the sum of the first half to the second
  return v;
}

// Orders LDS accesses only: the workgroups of the plan kernel hand each other nothing through global memory, and waiting for its
// stores at every barrier (as __syncthreads does) would cost a round trip to memory each time.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The sort bins of an expert: the rows are sorted by keep pattern, so every bin is a range of rows.  Loops over them stay loops: unrolled
// over sixteen bins at every use they were 10 KiB more instructions, which a launch fetches from memory, and slower.
template <int NSB>  // partitions in the sort key
struct Bins {
  static constexpr int N = 1 << NSB;
  // does bin sb keep partition p? (partitions outside the sort key: assumed kept)
  static __device__ __forceinline__ bool keeps(int sb, int p) { return p >= NSB || (((N - 1 - sb) >> (NSB - 1 - p)) & 1); }
  static __device__ __forceinline__ int pattern(int sb, int P) {
    return (int)(__brev((unsigned)(N - 1 - sb)) >> (32 - NSB)) | (((1 << P) - 1) & ~(N - 1));
  }
  // f(sb, first row, end) for every bin that has rows, in row order; returns the expert's rows
  template <class F>
  static __device__ __forceinline__ int each(const int32_t* bin_count, int e, F&& f) {
    int off = 0;
    const int32_t* src = bin_count + e * N;
    auto one = [&](int sb, int c) {
      if (c > 0) f(sb, off, off + c);
      off += c;
    };
    if constexpr (N >= 4) {
#pragma unroll 1
      for (int b = 0; b < N; b += 4) {
        const int4 v = *(const int4*)(src + b);
        one(b, v.x), one(b + 1, v.y), one(b + 2, v.z), one(b + 3, v.w);
      }
    } else {
      const int2 v = *(const int2*)src;
      one(0, v.x), one(1, v.y);
    }
    return off;
  }
  static __device__ __forceinline__ int rows(const int32_t* bin_count, int e) {
    return each(bin_count, e, [](int, int, int) {});
  }
  // partitions kept by some row of the rows [r0, r1), of [r1, r2)
  static __device__ __forceinline__ int2 kept(const int32_t* bin_count, int e, int r0, int r1, int r2, int P) {
    int2 bits = make_int2(0, 0);
    each(bin_count, e, [&](int sb, int off, int end) {
      const int pat = pattern(sb, P);
      bits.x |= off < r1 && end > r0 ? pat : 0;
      bits.y |= off < r2 && end > r1 ? pat : 0;
    });
    return bits;
  }
};
// Partition p in an expert's row tiles of 2^bm rows.  With thresholds that grow with p the rows that keep p are a prefix of the
// expert's rows; in general the counts bound them (rows in between that lack p are zeroed by the GEMM-1 epilogue).
struct TileUse {
  int rows;         // rows of the tile up to the last one that keeps p (0: none does)
  int next_rows;    // the same for the next tile
  int before;       // tiles before it of which some row keeps p
  bool full_before; // the last row of the tile before keeps p
};
template <int NSB>
__device__ __forceinline__ TileUse tile_use(const int32_t* bin_count, int e, int i, int bm, int p) {
  const int r0 = i << bm, r1 = r0 + (1 << bm), r2 = r1 + (1 << bm);
  TileUse u = {0, 0, 0, false};
  int next = 0;  // first tile that has not been looked at
  Bins<NSB>::each(bin_count, e, [&](int sb, int off, int end) {
    if (Bins<NSB>::keeps(sb, p)) {
      if (off < r1 && end > r0) u.rows = min(r1, end) - r0;
      if (off < r2 && end > r1) u.next_rows = min(r2, end) - r1;
      if (off < r0 && end >= r0) u.full_before = true;
      const int hi = min((end - 1) >> bm, i - 1), lo = max(off >> bm, next);
      if (hi >= lo) u.before += hi - lo + 1, next = hi + 1;
    }
  });
  return u;
}

// LANES: 0: the batch has been routed (its histograms are in the workspace).  Else every workgroup routes it, see
// launch_small_plan: 8 or 32: a lane per token and at most that many experts; 16: sixteen lanes per token, at most 64 experts.
// chunk: LANES == 0: route blocks whose pairs a workgroup of the row lists takes (0: no such workgroups, launch_scatter follows).
// MANY: more than 64 experts, or bins that are no multiple of four (in a kernel of their own: what these need slows the others down, as a
// launch fetches its instructions from memory: 333 tokens on 64 + 2 experts 9.5 us, with it 10.6)
template <int LANES, int NSB, bool MANY>
__global__ __launch_bounds__(kPlanThreads) void plan_kernel(Layout L, int T, char* ws, RouteArgs ra, int chunk) {
  extern __shared__ __attribute__((aligned(16))) int32_t sm[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int E_res = L.E_res, P = NSB < kSubBits ? NSB : L.P, BM = L.BM;
  const int units_log2 = 31 - __clz(max(L.split_items, 1));  // (powers of two)
  const int has_sh = L.n_shared > 0 ? 1 : 0;
  const int E_tot = E_res + has_sh, NG = E_tot * P;  // (expert, partition) groups; the shared pseudo-expert only uses p = 0
  const int bm = 31 - __clz(BM);                     // the tile heights are powers of two
  auto tiles_of = [&](int rows) { return (rows + BM - 1) >> bm; };
  auto short_rows = [&](int n) {  // rows of a last tile that the one before it can take along, else 0
    const int nt = tiles_of(n), last = n - (nt - 1) * BM;
    return nt >= 2 && last <= kTallExtra ? last : 0;
  };
  int32_t* bin_count = sm;                         // [nbins]
  int32_t* ne = sm + ((L.nbins + 3) & ~3);         // [E_tot] rows of each expert
  int32_t* ts = ne + E_tot;                        // [E_tot] first tile.  Order in the row space: the shared pseudo-expert (id E_res), then the others by id
  int32_t* ab = ts + E_tot;                        // [E_tot] 2 x (short last tiles of the experts before) + (this one's is short), see below
  int32_t* ga = ab + E_tot;                        // [NG] active tiles of each group
  int32_t* gb = ga + NG;                           // [NG] item base of each group
  int32_t* next = ga;                              // row lists: [nbins] next row of every bin
  int32_t* tail = sm + plan_lds_words(L) - kHalvedMost * (int)(sizeof(Item1) / 4);  // the items of a last round that may be cut
  int4* rec = (int4*)(tail - kPlanRecords * 4);    // what step 4 finds out about the (row tile, partition) pairs
  uint8_t* kmask_l = (uint8_t*)rec;                // GEMM-2: partitions of the first tiles
  uint16_t* texp = (uint16_t*)rec - kPlanTilesLds; // experts of the first kPlanTilesLds tiles
  int32_t* pairs = sm + plan_lds_words(L);         // LANES: see finish_pair; else partial sums
  __shared__ int total_tiles_l, total_short_l, multi_l[2], est[4], split_l[2], k_lo[2][kMaxSplit + 1];
  static_assert(kPlanRecords * 16 >= kPlanTilesLds && kMaxTailSplit <= kMaxSplit, "");
  const bool lists2 = blockIdx.x == 0, lists1 = blockIdx.x == 1, rows_list = blockIdx.x >= 2;

  // 0. rows of every sort bin
  int pr_keep[kListPairs], pr_e[kListPairs];  // row lists, LANES == 0: this thread's pairs, fetched with the histograms
  int64_t pr0 = 0, pr1 = 0;                   // the pairs of this workgroup
  if (tid < 4) est[tid] = 0;
  if constexpr (LANES != 0) {
    if (!rows_list) ra.idx = nullptr;  // one workgroup writes the routing results
    int32_t* mine = rows_list ? pairs : nullptr;
    if constexpr (LANES == 16) {
      float* tau_l = (float*)(pairs + T * L.K);
      route_row_setup(ra, bin_count, tau_l, kPlanThreads);
      route_row_tokens<1, 1, kPlanThreads / 64, kRouteInLds>(ra, ra.logits, 0, min(ra.T, kPlanThreads / 16), bin_count, tau_l, mine);
    } else {
      float* tau_l = (float*)(pairs + T * L.K);  // fetched now, together with the logits, not after the scores are known
      for (int i = tid; i < L.E * P; i += kPlanThreads) tau_l[i] = ra.tau[i];
      for (int i = tid; i < L.nbins; i += kPlanThreads) bin_count[i] = 0;
      route_lane_token<LANES, (LANES < 16 ? LANES : 16), kRouteInLds>(ra, tid, bin_count, mine, tau_l);
    }
    pr1 = (int64_t)T * L.K;
  } else {
    // column sums of the route kernel's per-block histograms; for the row lists also of the blocks before this workgroup's
    const int32_t* blk_hist = (const int32_t*)(ws + L.o_bin_count);
    const int bt = route_block_tokens(L.E, T), nblk = (T + bt - 1) / bt;
    const int blk0 = rows_list ? ((int)blockIdx.x - 2) * chunk : 0;
    if (rows_list) {
      const uint8_t* keep = (const uint8_t*)(ws + L.o_keep);
      const int32_t* idx = (const int32_t*)(ws + L.o_idx);
      pr0 = (int64_t)blk0 * bt * L.K;
      pr1 = min((int64_t)T * L.K, pr0 + (int64_t)chunk * bt * L.K);
#pragma unroll
      for (int u = 0; u < kListPairs; ++u) {
        const int64_t pr = min(pr0 + u * kPlanThreads + tid, pr1 - 1);
        pr_keep[u] = keep[pr];
        pr_e[u] = idx[pr];
      }
    }
    // Four columns to a thread (two where an odd number of experts has two bins each), up to sixteen threads to a column, up to sixteen rows
    // in flight each; where a column has several threads the partial sums meet in LDS.  (One load after the other for the bins that are no
    // multiple of four, or more than 4096: 16384 tokens on 512 experts in 8 parts 603 us instead of 121, on 257 in one 85 instead of 26.)
    const int nb = L.nbins;
    if constexpr (!MANY) {
      const int cols = nb >> 2, G = min(16, kPlanThreads / cols);
      const int g = tid / cols, c4 = tid - g * cols;
      int4 sum = make_int4(0, 0, 0, 0), before = sum;
      if (g < G) {
        for (int r = 0; r < nblk; r += 16 * G) {
          int4 v[16];
#pragma unroll
          for (int u = 0; u < 16; ++u)
            if (r + u * G < nblk) v[u] = *(const int4*)(blk_hist + (size_t)min(r + u * G + g, nblk - 1) * nb + c4 * 4);
#pragma unroll
          for (int u = 0; u < 16; ++u)
            if (r + u * G < nblk) {
              const int row = r + u * G + g, in = row < nblk ? -1 : 0, pre = row < blk0 ? -1 : 0;
              sum.x += v[u].x & in, sum.y += v[u].y & in, sum.z += v[u].z & in, sum.w += v[u].w & in;
              before.x += v[u].x & pre, before.y += v[u].y & pre, before.z += v[u].z & pre, before.w += v[u].w & pre;
            }
        }
        *(int4*)(pairs + g * nb + c4 * 4) = sum;
        if (rows_list) *(int4*)(pairs + kSumWords / 2 + g * nb + c4 * 4) = before;
      }
      lds_barrier();
      for (int c = tid; c < nb; c += kPlanThreads) {
        int n = 0, m = 0;
        for (int q = 0; q < G; ++q) {
          n += pairs[q * nb + c];
          if (rows_list) m += pairs[kSumWords / 2 + q * nb + c];
        }
        bin_count[c] = n;
        if (rows_list) next[c] = m;
      }
    } else {
      auto sums = [&](auto zero) {
        using V = decltype(zero);
        constexpr int N = sizeof(V) / 4;
        const int cols = nb / N, G = max(min(16, kPlanThreads / cols), 1);
        const bool direct = G == 1;  // the sums need no others
        for (int at = tid; at < cols * G; at += kPlanThreads) {  // (more than once only for G == 1)
          const int g = at / cols, c = at - g * cols;
          V sum = zero, before = zero;
          for (int r = 0; r < nblk; r += 16 * G) {
            V v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u)
              if (r + u * G < nblk) v[u] = *(const V*)(blk_hist + (size_t)min(r + u * G + g, nblk - 1) * nb + c * N);
#pragma unroll
            for (int u = 0; u < 16; ++u)
              if (r + u * G < nblk) {
                const int row = r + u * G + g, in = row < nblk ? -1 : 0, pre = row < blk0 ? -1 : 0;
                sum += v[u] & in;
                before += v[u] & pre;
              }
          }
          *(V*)(direct ? bin_count + c * N : pairs + g * nb + c * N) = sum;
          if (!rows_list) continue;
          if (!direct) *(V*)(pairs + kSumWords / 2 + g * nb + c * N) = before;
          else
            for (int i = 0; i < N; ++i) next[c * N + i] = before[i];  // (not at a multiple of 16 bytes)
        }
        if (direct) return;
        lds_barrier();
        for (int c = tid; c < nb; c += kPlanThreads) {
          int n = 0, m = 0;
          for (int q = 0; q < G; ++q) {
            n += pairs[q * nb + c];
            if (rows_list) m += pairs[kSumWords / 2 + q * nb + c];
          }
          bin_count[c] = n;
          if (rows_list) next[c] = m;
        }
      };
      if constexpr (NSB == 1) {
        if (nb & 3) sums(i32x2{0, 0});
        else sums(i32x4{0, 0, 0, 0});
      } else {
        sums(i32x4{0, 0, 0, 0});
      }
    }
  }
  lds_barrier();

  // 1. The experts' table, by the first wavefront.
  // A short last tile of an expert (at most kTallExtra rows) has no GEMM-2 items of its own: the items of the tile before it are
  // tall and compute its rows too.  Only if the short tile keeps no partition that the tile before it drops: the tall items run over
  // the partitions of the full tile, and where the short tile lacks one of them its rows of H are zeros (written by the
  // GEMM-1 item of the full tile, see step 4).
  // Beyond 64 experts it takes several turns, and what an expert's bins need goes over all threads: 512 experts in 4 parts (16 bins), one
  // token 29 -> 17 us.
  const bool makes_starts = rows_list || (lists2 && LANES == 0 && chunk == 0);
  auto starts = [&](int e, int off) {  // first row of every bin of expert e, whose first row is off
    int32_t* cursor = (int32_t*)(ws + L.o_cursor);  // where the scatter kernel starts
    for (int bin = e * Bins<NSB>::N; bin < (e + 1) * Bins<NSB>::N; ++bin) {
      if (!rows_list) cursor[bin] = off;
      else next[bin] = (LANES == 0 ? next[bin] : 0) + off;  // (behind the rows of the blocks before this workgroup's)
      off += bin_count[bin];
    }
  };
  if constexpr (MANY) {
    for (int e = tid; e < E_res; e += kPlanThreads) ne[e] = Bins<NSB>::rows(bin_count, e);
    lds_barrier();
  }
  if (wv == 0) {
    int tiles = 0, shorts = 0;
    uint64_t multi = 0;  // bit e & 63: some expert e has more than one row tile
    if (has_sh) {
      const int nt = tiles_of(T), s = L.tall_tiles && short_rows(T) ? 1 : 0;
      if (lane == 0) ne[E_res] = T, ts[E_res] = 0, ab[E_res] = s;
      if (!rows_list)
        for (int i = lane; i < min(nt, kPlanTilesLds); i += 64) texp[i] = (uint16_t)E_res;
      tiles = nt, shorts = s;
    }
    for (int e0 = 0; e0 < E_res; e0 += 64) {
      const int e = e0 + lane;
      const int n = e >= E_res ? 0 : MANY ? ne[e] : Bins<NSB>::rows(bin_count, e), nt = tiles_of(n);
      int s = 0;
      if (!rows_list && L.tall_tiles && short_rows(n)) {
        const int2 bits = Bins<NSB>::kept(bin_count, e, (nt - 2) * BM, (nt - 1) * BM, n, P);
        s = (bits.y & ~bits.x) == 0 ? 1 : 0;
      }
      const int incl = wave_incl_sum(nt), t0 = tiles + incl - nt;
      const uint64_t short_m = __ballot(s);
      multi |= __ballot(nt > 1);
      if (e < E_res) {
        ne[e] = n;
        ts[e] = t0;
        ab[e] = 2 * (shorts + __popcll(short_m & ((1ull << lane) - 1))) + s;
        if (!MANY && makes_starts) starts(e, t0 * BM);
        if (!rows_list)
          for (int i = t0; i < min(t0 + nt, kPlanTilesLds); ++i) texp[i] = (uint16_t)e;
        if (lists2) {
          ((int32_t*)(ws + L.o_exp_nrows))[e] = n;
          ((int32_t*)(ws + L.o_exp_row0))[e] = t0 * BM;
        }
      }
      tiles += __builtin_amdgcn_readlane(incl, 63);
      shorts += __popcll(short_m);
    }
    if (lane == 0) {
      total_tiles_l = tiles;
      total_short_l = shorts;
      multi_l[0] = (int)(uint32_t)multi, multi_l[1] = (int)(uint32_t)(multi >> 32);
    }
  }
  if (MANY && makes_starts) {
    lds_barrier();
    for (int e = tid; e < E_res; e += kPlanThreads) starts(e, ts[e] * BM);
  }

  // 2. The row lists.  The order inside a bin is arbitrary (it is decided by atomics); the layer output does not depend on it because
  // every row is computed independently of its tile neighbours.
  if (rows_list) {
    int32_t* pair_row = (int32_t*)(ws + L.o_pair_row);
    int32_t* row_token = (int32_t*)(ws + L.o_row_token);
    uint8_t* row_bits = (uint8_t*)(ws + L.o_row_bits);
    lds_barrier();
    auto place = [&](int64_t pr, int bits, int e) {
      int row = -1;
      if (bits) {
        row = atomicAdd(&next[(e - L.lo) * Bins<NSB>::N + sub_of_bits(bits, NSB)], 1);
        row_token[row] = (int32_t)(pr / L.K);
        row_bits[row] = (uint8_t)bits;
      }
      pair_row[pr] = row;
    };
    if constexpr (LANES != 0) {
      for (int pr = tid; pr < (int)pr1; pr += kPlanThreads) place(pr, pairs[pr] & 255, pairs[pr] >> 8);
    } else {
#pragma unroll
      for (int u = 0; u < kListPairs; ++u)
        if (pr0 + u * kPlanThreads + tid < pr1) place(pr0 + u * kPlanThreads + tid, pr_keep[u], pr_e[u]);
    }
    if (has_sh)  // the shared pseudo-expert's rows are the tokens themselves, at the start of the row space
      for (int t = (int)(pr0 / L.K) + tid; t < (int)(pr1 / L.K); t += kPlanThreads) {
        row_token[t] = t;
        row_bits[t] = 1;
      }
    return;
  }

  // Tall GEMM-1 items: when an expert's last row tile has at most kTallExtra rows, the item of the tile
  // before it (if that is full for the partition) computes them too, and the last tile gets no item of
  // its own: a few rows would otherwise pull the whole weight tile through another compute unit.
  // Groups in the order of the experts; the shared pseudo-expert's go first once it has several row tiles: its full tiles are the
  // longest items of a batch with a few rows per expert, and last they started last and ended long after the others
  // (333 tokens on 64 + 2 experts of 2048 x 1408: the layer 267 -> 252 us).
  const int sh_first = has_sh && T > BM ? 1 : 0;
  const bool price_lists = L.tall_tiles == 1 && (int64_t)T * L.K > BM;  // (no expert of a smaller batch has a second tile)
  if (lists1 && wv > 0) {
    // Whether the batch gets them is decided by pricing both lists.  Items in 1/256 of a full one: a ragged
    // item of r rows 128 + r / 2 (half of every stage is its weight tile), a tall one 256 + 33 with up to 32
    // extra rows and 256 + 56 beyond (measured).  A list of N items of mean cost c is taken to last
    // ceil(N / units) * c, whole rounds of one item per compute unit: removing a tenth of the items is worth
    // a round or nothing, and the longer items of a list that still needs the same rounds make it slower.
    // est[]: items and summed cost of the list without / with tall items
    int n0 = 0, w0 = 0, n1 = 0, w1 = 0;
    for (int gi = tid - 64; gi < NG; gi += kPlanThreads - 64) {
      const int pos = gi / P, p = gi - pos * P, e = sh_first ? (pos == 0 ? E_res : pos - 1) : pos;
      int n_e = p == 0 ? T : 0, rows = n_e, tiles = tiles_of(n_e), merged = short_rows(n_e) > 0;
      if (e < E_res) {
        rows = 0;
        n_e = Bins<NSB>::each(bin_count, e, [&](int sb, int, int end) { rows = Bins<NSB>::keeps(sb, p) ? end : rows; });
        const int nt = tiles_of(n_e);
        tiles = rows > 0, merged = 0;  // (as long as there is one tile)
        if (nt > 1) {
          const TileUse u = tile_use<NSB>(bin_count, e, nt - 1, bm, p);
          tiles = u.before + (u.rows > 0);
          merged = short_rows(n_e) && u.rows > 0 && u.full_before;
        }
      }
      ga[gi] = 2 * tiles + merged;  // the tiles that have an item, and whether the last one's goes into a tall one
      if (price_lists && rows > 0) {
        // (the rows that need p are taken to be a prefix of the expert's rows: exactly so with thresholds that grow with p)
        const int nt1 = e < E_res ? L.NT1 : L.NT1_sh;
        const int full = rows >> bm, rem = rows & (BM - 1);
        const int n = full + (rem ? 1 : 0), w = full * 256 + (rem ? 128 + rem / 2 : 0);
        const bool tall = short_rows(n_e) && rows > (tiles_of(n_e) - 1) * BM;  // the last tile's item goes into the one before
        n0 += nt1 * n;
        w0 += nt1 * w;
        n1 += nt1 * (tall ? n - 1 : n);
        w1 += nt1 * (tall ? full * 256 + (rem <= 32 ? 33 : 56) : w);
      }
    }
    if (price_lists) {
      n0 = wave_incl_sum(n0), w0 = wave_incl_sum(w0), n1 = wave_incl_sum(n1), w1 = wave_incl_sum(w1);
      if (lane == 63 && n0 > 0) {  // integer sums: the same in any order
        atomicAdd(&est[0], n0);
        atomicAdd(&est[1], w0);
        atomicAdd(&est[2], n1);
        atomicAdd(&est[3], w1);
      }
    }
  }
  lds_barrier();
  const int total_tiles = total_tiles_l, total_short = total_short_l;
  int32_t* counters = (int32_t*)(ws + L.o_counters);
  // tile g belongs to the expert at the last position whose first tile is <= g (and which has a tile)
  auto tile_expert = [&](int g) {
    if (g < kPlanTilesLds) return (int)texp[g];
    if (has_sh && g < tiles_of(T)) return E_res;
    int lo_i = 0, hi_i = E_res;  // first expert with ts > g
    while (lo_i < hi_i) {
      const int mid = (lo_i + hi_i) >> 1;
      if (ts[mid] > g) hi_i = mid;
      else lo_i = mid + 1;
    }
    return lo_i - 1;
  };

  if (lists2) {
    // 3. GEMM-2 items: every tile x every output column tile.  The compute units take the items in
    //    list order, one each.  Where that leaves units idle, items are split along K: every extra K
    //    range is an item of its own that writes a partial-output tile into a pool, and the combine
    //    kernel adds those tiles to the item's rows of Yp in a fixed order.
    //    (a) few row tiles (decode-sized batches): fewer items than units, each streaming a whole
    //        column tile of W2 alone -> all items are split, into as many ranges as keep the list
    //        within one item per unit;
    //    (b) the last round of a longer list is only partly full -> its items are split where the shorter
    //        pieces fill the units better (see below).
    Item2* items2 = (Item2*)(ws + L.o_items2);
    const int W2n = (total_tiles - total_short) * L.ND2;
    if (wv == 0) {  // items first_split .. W2n-1 (in list order) are split nsplit ways
      int nsplit = 1, first_split = W2n;
      if (L.split_items > 0 && W2n > 0) {
        int ksp = L.Fpk / kBK;
        if (has_sh) ksp = min(ksp, L.Fsk / kBK);
        if (W2n * 2 <= L.split_items) {
          while (nsplit < kMaxSplit && W2n * nsplit * 2 <= L.split_items && nsplit * 2 <= ksp && W2n * (nsplit * 2 - 1) <= L.pool_tiles) nsplit *= 2;
          first_split = 0;
        } else {
          // The last round holds `rest` items for split_items compute units.  Cut n ways they are rest * n
          // shorter items, which take ceil(rest * n / units) turns of 1/n of a round each (plus a fill and a
          // write-out per piece, worth about eight K stages): 192 items cut in four are three turns of a
          // quarter instead of a whole round at three quarters of the units.  The cheapest n that the pool
          // of partial tiles can hold wins; n = 1 (cost: one round) if none is cheaper.  (Lane n prices n pieces.)
          const int rest = W2n & (L.split_items - 1);
          const int item_stages = E_res > 0 ? P * (L.Fpk / kBK) : L.Fsk / kBK;   // K stages of a long item
          const float piece = 8.0f / (float)max(item_stages, 1);                  // per-piece overhead in units of such an item
          const int n = max(lane, 1), turns = (rest * n + L.split_items - 1) >> units_log2;
          const float cost = (float)turns * (1.0f / (float)n + piece);
          float best = 1.0f;
          for (int m = 2; m <= kMaxTailSplit && m <= ksp && rest > 0 && rest * (m - 1) <= L.pool_tiles; ++m) {
            const float cm = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cost), m));
            if (cm < best - 0.04f) {  // a clear gain only: every extra range costs a partial tile written and read
              best = cm;
              nsplit = m;
            }
          }
          if (nsplit > 1) first_split = W2n - rest;
        }
        if (nsplit == 1) first_split = W2n;
      }
      if (lane <= nsplit) {  // (at most a few thousand stages times 8)
        k_lo[0][lane] = L.Fpk / kBK * lane / nsplit;
        k_lo[1][lane] = L.Fsk / kBK * lane / nsplit;
      }
      if (lane == 0) split_l[0] = nsplit, split_l[1] = first_split;
    } else {  // the partitions that some row of a tile keeps
      for (int g = tid - 64; g < min(total_tiles, kPlanTilesLds); g += kPlanThreads - 64) {
        const int e = tile_expert(g), i = g - ts[e], r1 = (i + 1) * BM;
        const int2 bits = e < E_res ? Bins<NSB>::kept(bin_count, e, i * BM, r1, r1 + BM, P) : make_int2(1, 1);
        kmask_l[g] = (uint8_t)(bits.x | ((ab[e] & 1) && i + 2 == tiles_of(ne[e]) ? bits.y : 0));  // a tall item's: of both tiles
      }
    }
    lds_barrier();
    const int nsplit = split_l[0], first_split = split_l[1];
    int32_t* split_of = (int32_t*)(ws + L.o_split_of);
    // threads that share the column tiles of a row tile: a power of two
    int ls = 0;
    while ((1 << ls) < L.ND2 && total_tiles << (ls + 1) <= kPlanThreads) ++ls;
    const int S = 1 << ls;
    for (int qs = tid; qs < total_tiles << ls; qs += kPlanThreads) {
      const int g = qs >> ls, jd0 = qs & (S - 1);
      const int e = tile_expert(g);
      const int n = ne[e], i = g - ts[e], nt_all = tiles_of(n), sl = ab[e] & 1, shorts = ab[e] >> 1;
      if (sl && i == nt_all - 1) continue;         // the short last tile: computed by the items of the tile before
      const bool tall = sl && i == nt_all - 2;
      const int ksp = (e < E_res ? L.Fpk : L.Fsk) / kBK;
      Item2 v;
      v.row0 = g * BM;
      v.nrows = min(n - i * BM, BM) + (tall ? n - (i + 1) * BM : 0);
      v.e = e;
      if (g < kPlanTilesLds) {
        v.kmask = kmask_l[g];
      } else {
        const int2 bits = e < E_res ? Bins<NSB>::kept(bin_count, e, i * BM, (i + 1) * BM, (i + 2) * BM, P) : make_int2(1, 1);
        v.kmask = bits.x | (tall ? bits.y : 0);
      }
      // list order (expert, column tile, row tile) if g2_rows_inner: the row tiles that share one column
      // tile of W2 are adjacent, run at the same time on one XCD and fetch the weights once;
      // else (row tile, column tile)
      const int nt_e = nt_all - sl;        // tiles of the expert that have items
      const int ts_e = ts[e] - shorts;     // and of the experts before it
      if (jd0 == 0) {
        // The first row tile that has a split item (the combine kernel looks no tile before it up): later tiles have later last items.
        // (By comparison: an LDS minimum over all the split items took 2 us.)
        const int last = L.g2_rows_inner ? (ts_e + nt_e) * L.ND2 - nt_e + i : (ts_e + i + 1) * L.ND2 - 1;
        const int last_before = L.g2_rows_inner ? (i > 0 ? last - 1 : ts_e * L.ND2 - 1) : last - L.ND2;
        if (last >= first_split && last_before < first_split) counters[4] = g;
      }
      for (int jd = jd0; jd < L.ND2; jd += S) {
        v.jd = jd;
        const int gj = g * L.ND2 + jd;
        const int slot = L.g2_rows_inner ? ts_e * L.ND2 + jd * nt_e + i : (ts_e + i) * L.ND2 + jd;
        if (slot < first_split) {
          v.ks_lo = 0;
          v.ks_n = ksp;
          v.split = 0;
          items2[slot] = v;
          if (L.pool_tiles > 0) {  // (without a pool there is no table either, and nothing looks it up)
            split_of[gj] = -1;
            if (tall) split_of[gj + L.ND2] = -1;
          }
        } else {
          const int q = slot - first_split;  // q-th split item: its extra ranges use pool tiles q*(nsplit-1) ..
          for (int sp = 0; sp < nsplit; ++sp) {
            v.ks_lo = k_lo[e < E_res ? 0 : 1][sp];
            v.ks_n = k_lo[e < E_res ? 0 : 1][sp + 1] - v.ks_lo;
            v.split = sp == 0 ? 0 : 1 + q * (nsplit - 1) + (sp - 1);
            items2[first_split + q * nsplit + sp] = v;
          }
          split_of[gj] = q * (nsplit - 1);
          if (tall) split_of[gj + L.ND2] = q * (nsplit - 1) | kSplitRowsOffset;  // rows of the short tile: BM further down the pool tiles
        }
      }
    }
    if (tid == 0) {
      counters[9] = 0;  // see take_piece
      counters[1] = first_split + (W2n - first_split) * nsplit;
      counters[2] = total_tiles - total_short;  // row tiles that have GEMM-2 items
      counters[3] = nsplit;
      if (first_split == W2n) counters[4] = total_tiles;
      counters[5] = multi_l[0];
      counters[6] = multi_l[1];
      counters[7] = L.BN2 / 2;  // neurons of a neuron tile; an output column tile is twice as wide
    }
    return;
  }

  // 4. GEMM-1 items in the order (expert, partition, neuron tile, row tile): the row tiles that
  //    share one weight tile are adjacent.
  bool use_tall1 = L.tall_tiles == 2;
  if (price_lists) {
    auto rounds = [&](int n) { return (float)((n + (1 << units_log2) - 1) >> units_log2); };
    const float t0 = est[0] > 0 ? rounds(est[0]) * (float)est[1] / (float)est[0] : 0.f;
    const float t1 = est[2] > 0 ? rounds(est[2]) * (float)est[3] / (float)est[2] : 0.f;
    use_tall1 = est[2] < est[0] && t1 <= t0;
  }
  __shared__ int total1_l;
  Item1* items1 = (Item1*)(ws + L.o_items1);
  const int nt1_max = max(L.NT1, has_sh ? L.NT1_sh : 0), n_q = total_tiles * P;
  //    Up to kPlanRecords (row tile, partition) pairs leave what their items need in LDS, and a power of two of threads, as many as would
  //    otherwise idle, share the neuron tiles of each; the threads of more pairs write the items of one after the other themselves.
  const bool direct = n_q > kPlanRecords;
  int ls = 0;
  while (!direct && ls < 5 && (1 << ls) < nt1_max && n_q << (ls + 1) <= kPlanThreads) ++ls;
  int total1 = 0, first_half = 0;
  for (int q0 = 0; q0 == 0 || q0 < n_q; q0 += kPlanRecords) {
    //  What this thread's pair needs ...
    int4 mine = make_int4(0, 0, 0, 0);
    if (wv > 0 && q0 + tid - 64 < n_q) {
      const int q = q0 + tid - 64, g = q / P, p = q - g * P;
      const int e = tile_expert(g), n = ne[e], i = g - ts[e], nt = tiles_of(n);
      const bool routed = e < E_res;
      const int last = short_rows(n);  // rows of the expert's short last tile
      const int fill = min(n - i * BM, BM);
      TileUse u = {p == 0 ? fill : 0, last, i, true};
      if (routed) u = tile_use<NSB>(bin_count, e, i, bm, p);
      int rows = u.rows, nfill = fill;
      if (rows > 0 && last && i + 1 == nt && use_tall1 && u.full_before) rows = 0;  // computed by the tall item of the tile before
      if (rows > 0 && last && i + 2 == nt) {
        if (use_tall1 && rows == BM && u.next_rows > 0) {  // a tall item: the rows of the expert's short last tile follow directly
          rows += u.next_rows;
          nfill += last;
        } else if ((ab[e] & 1) && u.next_rows == 0) {
          // the tall GEMM-2 items of this tile multiply partition p over the short last tile's rows too, none
          // of which keeps it: their part of H is zeros, written by this item
          nfill += last;
        }
      }
      mine = make_int4(rows | nfill << 16, u.before, ((sh_first ? (routed ? e + 1 : 0) : e) * P + p) << 16 | p << 12 | e, g * BM);
      if (!direct) rec[tid - 64] = mine;
    }
    if (q0 == 0) {
      //  ... and, by the first wavefront, the item bases of the groups
      if (wv == 0) {
        const int sh_lo = sh_first ? 0 : E_res * P, sh_hi = has_sh ? sh_lo + P : sh_lo;  // the shared pseudo-expert's groups
        int sum = 0;
#pragma unroll 4
        for (int g0 = 0; g0 < NG; g0 += 64) {
          const int gi = g0 + lane, v = gi < NG ? ga[gi] : 0, n = (v >> 1) - (use_tall1 ? v & 1 : 0);
          const int items = n * (gi >= sh_lo && gi < sh_hi ? L.NT1_sh : L.NT1), incl = wave_incl_sum(items);
          if (gi < NG) ga[gi] = n, gb[gi] = sum + incl - items;
          sum += __builtin_amdgcn_readlane(incl, 63);
        }
        if (lane == 0) total1_l = sum;
      }
      lds_barrier();
      //  In the weight-streaming regime (few rows per expert) every item lasts as long as its weight
      //  tile takes to arrive, so the kernel lasts a whole number of rounds of one item per compute
      //  unit: when the last round is at most half full, its items are cut into halves of 64
      //  neurons, which fill it (an item of more than 128 rows, or of a last neuron tile of at most
      //  64 neurons, stays whole).
      total1 = first_half = total1_l;  // list positions >= first_half belong to that last round
      if (may_halve_items1(L, T)) {
        const int rest = total1 & (L.split_items - 1);
        if (rest > 0 && rest * 2 <= L.split_items) first_half = total1 - rest;
      }
    }
    for (int qs = direct ? 0 : tid; qs < (direct ? 1 : n_q << ls); qs += kPlanThreads) {
      const int4 r = direct ? mine : rec[qs >> ls];
      Item1 v;
      v.nrows = r.x & 0xffff;
      if (v.nrows == 0) continue;  // no row of the tile keeps p, or no item of its own
      v.nfill = r.x >> 16;
      v.e = r.z & 0xfff;
      v.p = (r.z >> 12) & 15;
      v.row0 = r.w;
      const int n_act = ga[r.z >> 16], base = gb[r.z >> 16] + r.y, nt1 = v.e < E_res ? L.NT1 : L.NT1_sh, width = v.e < E_res ? L.Fp : L.F_shT;
      v.once = n_act == 1 ? 1 : 0;
      for (int jt = qs & ((1 << ls) - 1); jt < nt1; jt += 1 << ls) {
        v.jt = jt;
        // MFMA path, at most 128 rows, a last neuron tile of at most 64 neurons: the half-tile variant of
        // the kernel takes it as a first half without a second one (half the weight bytes)
        v.half = L.mfma && v.nrows <= kMfmaBM / 2 && width - jt * kMfmaNeur <= kMfmaNeur / 2 ? 1 : 0;
        const int at = base + jt * n_act;
        if (at < first_half) items1[at] = v;
        else ((Item1*)tail)[at - first_half] = v;
      }
    }
  }
  int total_slots = total1;
  if (first_half < total1) {  // the same for every thread
    // the items of the last round are cut in two where that is possible (at most 128 rows, both halves
    // of the neuron tile exist); the list stays dense: item i moves up by the cuts before it
    __shared__ int slots_wave0, slots_all;
    lds_barrier();  // the tail is complete
    const int rest = total1 - first_half;  // <= kHalvedMost: wavefronts 0 and 1
    Item1 mine;
    int slots = 0;
    if (tid < rest) {
      mine = ((const Item1*)tail)[tid];
      const int live = (mine.e < E_res ? L.Fp : L.F_shT) - mine.jt * kMfmaNeur;
      slots = mine.nrows <= kMfmaBM / 2 && live > kMfmaNeur / 2 ? 2 : 1;
    }
    const int incl = wave_incl_sum(slots);
    if (tid == 63) slots_wave0 = incl;
    lds_barrier();
    if (tid < rest) {
      const int at = first_half + incl - slots + (tid >= 64 ? slots_wave0 : 0);
      if (slots == 2) {
        mine.half = 1;
        items1[at] = mine;
        mine.half = 2;
        items1[at + 1] = mine;
      } else {
        items1[at] = mine;
      }
      if (tid == rest - 1) slots_all = at + slots;
    }
    lds_barrier();
    total_slots = slots_all;
  }
  if (tid == 0) {
    counters[0] = total_slots;
    counters[8] = 0;  // see take_piece
    counters[kNonfiniteH] = 0;
  }
}

template <int LANES, int NSB, bool MANY>
static hipError_t launch_plan_many(const Layout& L, int T, char* ws, const RouteArgs& ra, int blocks, int chunk, hipStream_t s) {
  size_t sh = sizeof(int32_t) * (size_t)plan_lds_words(L);
  sh += sizeof(int32_t) * (size_t)(LANES != 0 ? T * L.K + L.E * L.P : kSumWords);
  if (sh > 48 * 1024) {  // hundreds of experts x 8 parts: above what a launch gets without asking
    static PerDeviceOnce once;
    hipError_t e = once.run([] { return hipFuncSetAttribute((const void*)plan_kernel<LANES, NSB, MANY>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024); });
    if (e != hipSuccess) return e;
  }
  plan_kernel<LANES, NSB, MANY><<<dim3(2 + blocks), dim3(kPlanThreads), sh, s>>>(L, T, ws, ra, chunk);
  return hipGetLastError();
}
template <int LANES, int NSB>
static hipError_t launch_plan_nsb(const Layout& L, int T, char* ws, const RouteArgs& ra, int blocks, int chunk, hipStream_t s) {
  if constexpr (LANES == 0)
    if (L.E_res > 64 || (L.nbins & 3)) return launch_plan_many<LANES, NSB, true>(L, T, ws, ra, blocks, chunk, s);
  return launch_plan_many<LANES, NSB, false>(L, T, ws, ra, blocks, chunk, s);
}
template <int LANES>
static hipError_t launch_plan_kernel(const Layout& L, int T, char* ws, const RouteArgs& ra, int blocks, int chunk, hipStream_t s) {
  switch (L.P) {
    case 1: return launch_plan_nsb<LANES, 1>(L, T, ws, ra, blocks, chunk, s);
    case 2: return launch_plan_nsb<LANES, 2>(L, T, ws, ra, blocks, chunk, s);
    case 3: return launch_plan_nsb<LANES, 3>(L, T, ws, ra, blocks, chunk, s);
    default: return launch_plan_nsb<LANES, kSubBits>(L, T, ws, ra, blocks, chunk, s);
  }
}

// The plan and, in further workgroups of the same launch, the row lists.  Each of these reads all the histograms, so it does that only
// as long as they are small (256 KiB: 16384 tokens on 64 experts in two parts); beyond, the scatter kernel follows, whose workgroups claim
// their rows with atomics.  Plan kernel + scatter kernel, before (an LDS table and a barrier for every step, fourteen in all) -> now, us: 8192
// tokens top-8 on 64 experts in 2 parts 17.5 + 6.2 -> 11.5, 4096 top-2 on 8 in 4 parts 23.2 + 5.2 -> 13, 16384 on 2 of 8 in 4 parts
// 18.8 + 5.0 -> 12.5, 333 on 64 + 2 in 2 parts 11.7 + 4.8 -> 9, 777 on 64 + 2 in 8 parts 20.7 + 5.5 -> 15.5; routed here as well: 1 token top-8
// on 64 experts 12.3 -> 9, 64 top-2 on 8 in 2 parts 9.7 -> 6.5.
static int route_blocks(const Layout& L, int T) {
  const int bt = route_block_tokens(L.E, T);
  return (T + bt - 1) / bt;
}
static int list_chunk(const Layout& L, int T) {  // route blocks to a workgroup of the row lists; 0: no such workgroups
  const int nblk = route_blocks(L, T), per_blk = route_block_tokens(L.E, T) * L.K;  // pairs of a route block
  int chunk = (nblk + 63) / 64;                                         // up to 64 workgroups ...
  if (chunk * per_blk < kPlanThreads) chunk = kPlanThreads / per_blk;   // ... of a pair per thread and more
  return T > 0 && (int64_t)nblk * L.nbins <= 65536 && (int64_t)chunk * per_blk <= kListPairs * kPlanThreads ? chunk : 0;
}
bool plan_writes_rows(const Layout& L, int T) { return list_chunk(L, T) > 0; }
hipError_t launch_plan(const Layout& L, int T, char* ws, hipStream_t s) {
  const int chunk = list_chunk(L, T);
  return launch_plan_kernel<0>(L, T, ws, RouteArgs{}, chunk ? (route_blocks(L, T) + chunk - 1) / chunk : 0, chunk, s);
}

// Routing, plan and row lists of a small batch in one launch: one workgroup routes 64 tokens at once with sixteen lanes each (more than 32
// experts), up to 1024 with a lane each, so each of three does it for itself and they write the two work lists and the row lists side by side.
// Layer times, route + plan + scatter -> this: 100 / 1000 tokens top-2 on 8 experts of 128 x 256 in fp32 29.0 -> 21.9 us, 46.6 -> 40.9; 128 / 512
// top-4 on 16 of 1024 x 512 45.0 -> 38.5, 62.4 -> 57.8, on 32 56.8 -> 46.1, 66.7 -> 59.4; 1024 on either (4096 pairs for one workgroup to
// place) no gain, 80.2 -> 80.5 and 75.9 -> 76.0: those take the three steps.
bool small_plan(const Layout& L, int T) {
  return L.E <= 32 ? T <= kPlanThreads && T * L.K <= kLanePlanPairs : T <= kRowPlanTokens && L.E <= 64;
}
hipError_t launch_small_plan(const Layout& L, int T, const float* logits, const float* tau, char* ws, hipStream_t s) {
  RouteArgs a = {};
  a.logits = logits;
  a.tau = tau;
  a.idx = (int32_t*)(ws + L.o_idx);
  a.w = (float*)(ws + L.o_w);
  a.keep = (uint8_t*)(ws + L.o_keep);
  a.bins = 1;
  a.T = T;
  set_route_layer(L, a);
  if (L.E <= 8) return launch_plan_kernel<8>(L, T, ws, a, 1, 0, s);
  if (L.E <= 32) return launch_plan_kernel<32>(L, T, ws, a, 1, 0, s);
  return launch_plan_kernel<16>(L, T, ws, a, 1, 0, s);
}

// ------------------------------------------------------------------------------------- scatter
// The row lists of batches whose histograms are too large for the plan kernel's workgroups to read them all (see launch_plan):
// places every pair with at least one kept unit into its bin's row range.
constexpr int kScatterThreads = 256;
// PPT pairs per thread (pair u of a thread is block base + u * 256 + thread: coalesced).  A block
// claims its rows with one global atomic per bin it fills, so larger blocks mean fewer of those
// (with 256 bins and 256 pairs per block they were the whole cost on the fine-grained layers).
template <int PPT>
__global__ __launch_bounds__(kScatterThreads) void scatter_kernel(Layout L, int T, char* ws) {
  extern __shared__ int32_t lh[];  // [nbins]
  const int32_t* idx = (const int32_t*)(ws + L.o_idx);
  const uint8_t* keep = (const uint8_t*)(ws + L.o_keep);
  int32_t* cursor = (int32_t*)(ws + L.o_cursor);
  int32_t* pair_row = (int32_t*)(ws + L.o_pair_row);
  int32_t* row_token = (int32_t*)(ws + L.o_row_token);
  uint8_t* row_bits = (uint8_t*)(ws + L.o_row_bits);
  const int nsub_bits = L.P < kSubBits ? L.P : kSubBits;
  const int64_t npairs = (int64_t)T * L.K;
  const int64_t pr0 = (int64_t)blockIdx.x * (kScatterThreads * PPT) + threadIdx.x;
  for (int i = threadIdx.x; i < L.nbins; i += kScatterThreads) lh[i] = 0;
  int bits[PPT], ex[PPT], bin[PPT], rank[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int64_t pr = pr0 + u * kScatterThreads;
    bits[u] = pr < npairs ? keep[pr] : 0;
    ex[u] = pr < npairs ? idx[pr] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    bin[u] = -1;
    rank[u] = 0;
    if (bits[u]) {
      bin[u] = (ex[u] - L.lo) * L.nsub + sub_of_bits(bits[u], nsub_bits);
      rank[u] = atomicAdd(&lh[bin[u]], 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < L.nbins; i += kScatterThreads) {
    int c = lh[i];
    if (c) lh[i] = atomicAdd(&cursor[i], c);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int64_t pr = pr0 + u * kScatterThreads;
    if (pr < npairs) {
      int row = -1;
      if (bin[u] >= 0) {
        row = lh[bin[u]] + rank[u];
        row_token[row] = (int32_t)(pr / L.K);
        row_bits[row] = (uint8_t)bits[u];
      }
      pair_row[pr] = row;
    }
    // the shared pseudo-expert's rows are the tokens themselves, at the start of the row space
    if (L.n_shared > 0 && pr < T) {
      row_token[pr] = (int32_t)pr;
      row_bits[pr] = 1;
    }
  }
}

hipError_t launch_scatter(const Layout& L, int T, char* ws, hipStream_t s) {
  int64_t n = (int64_t)T * L.K;
  if (n <= 0) return hipSuccess;
  size_t sh = sizeof(int32_t) * (size_t)(L.nbins > 0 ? L.nbins : 1);
  // as many pairs per thread as leave about 64 blocks or more
  const int64_t per = n / (64 * kScatterThreads);
  auto blocks = [&](int ppt) { return dim3((unsigned)((n + (int64_t)kScatterThreads * ppt - 1) / ((int64_t)kScatterThreads * ppt))); };
  if (per >= 8) scatter_kernel<8><<<blocks(8), dim3(kScatterThreads), sh, s>>>(L, T, ws);
  else if (per >= 4) scatter_kernel<4><<<blocks(4), dim3(kScatterThreads), sh, s>>>(L, T, ws);
  else if (per >= 2) scatter_kernel<2><<<blocks(2), dim3(kScatterThreads), sh, s>>>(L, T, ws);
  else scatter_kernel<1><<<blocks(1), dim3(kScatterThreads), sh, s>>>(L, T, ws);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------- combine
// y[t] = sum_k g[t][k] * Yp[row(t,k)] (+ Yp[shared row t]); Eq. 3 restricted to the kept units.
// One writer per output element, slots added in slot order: no atomics.
// Partial outputs still carry the powers of two of the packed weights; w2_inv = 2^-(s+k) takes them
// out here (exact, so the result is the one unscaled weights would give; 1 on the full-precision path).
// They are fp32, or (HALF) half precision times kYpHalfScale, which is taken out here as well.
// 16 bytes of partial outputs: VEC = 4 floats, or 8 half-precision values.  The rows of a token are
// loaded as raw 16-byte vectors (all in flight together) and widened one row at a time, so that the
// kernel stays within the registers of full occupancy.
template <bool HALF>
struct Partials {
  static constexpr int VEC = HALF ? 8 : 4;
  static __device__ __forceinline__ uint4 load(const char* base, size_t idx) { return *(const uint4*)(base + idx * (HALF ? 2 : 4)); }
  static __device__ __forceinline__ void widen(const uint4& r, float (&v)[VEC]) {
    if constexpr (HALF) {
      typedef _Float16 h8 __attribute__((ext_vector_type(8)));
      const h8 h = __builtin_bit_cast(h8, r);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = (float)h[i];
    } else {
      v[0] = __uint_as_float(r.x), v[1] = __uint_as_float(r.y), v[2] = __uint_as_float(r.z), v[3] = __uint_as_float(r.w);
    }
  }
};

template <typename OutT, int KB, bool HALF>
__global__ __launch_bounds__(256) void combine_kernel(Layout L, int T, const char* ws, OutT* y, const float* w2_inv_p) {
  using PT = Partials<HALF>;
  constexpr int VEC = PT::VEC;  // columns per thread (D % 8 == 0 where HALF is used: the matrix-core path)
  const float w2_inv = (w2_inv_p ? *w2_inv_p : 1.f) * (HALF ? 1.0f / kYpHalfScale : 1.f);
  const char* Yp = ws + L.o_Yp;
  const float* w = (const float*)(ws + L.o_w);
  const int32_t* pair_row = (const int32_t*)(ws + L.o_pair_row);
  const int DV = L.D / VEC;
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= (int64_t)T * DV) return;
  const int t = (int)(q / DV);
  const int d = (int)(q % DV) * VEC;
  // all row indices first, then all row loads in flight together, then the sum in slot order
  int row[KB];
  float g[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    row[k] = k < L.K ? pair_row[(size_t)t * L.K + k] : -1;
    g[k] = k < L.K ? w[(size_t)t * L.K + k] * w2_inv : 0.f;
  }
  uint4 raw[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) raw[k] = row[k] >= 0 ? PT::load(Yp, (size_t)row[k] * L.D + d) : make_uint4(0, 0, 0, 0);
  float acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
  const int32_t* counters = (const int32_t*)(ws + L.o_counters);
  const int nsplit = counters[3];
  const int split_row0 = counters[4] * L.BM;  // rows before it belong to tiles without split items
  const int32_t* split_of = (const int32_t*)(ws + L.o_split_of);
  const char* pool = ws + L.o_pool;
  const int jd = d / L.BN2, dc = d - jd * L.BN2;
  // GEMM-2 split K: the partial-output tiles of the extra K ranges of row r are added in range order
  auto add_extra = [&](int r, float (&into)[VEC]) {
    const int tile = r / L.BM;
    int first = split_of[(size_t)tile * L.ND2 + jd];
    if (first < 0) return;
    const int rofs = first & kSplitRowsOffset ? L.BM : 0;  // a short last tile: its rows follow those of the tile before
    first &= ~kSplitRowsOffset;
    size_t src = ((size_t)first * L.pool_rows + (r - tile * L.BM) + rofs) * L.BN2 + dc;
    for (int sp = 1; sp < nsplit; ++sp) {
      float u[VEC];
      PT::widen(PT::load(pool, src), u);
#pragma unroll
      for (int i = 0; i < VEC; ++i) into[i] += u[i];
      src += (size_t)L.pool_rows * L.BN2;
    }
  };
  if (L.n_shared > 0) {  // the shared experts' rows sit first in the row space (weight 1)
    PT::widen(PT::load(Yp, (size_t)t * L.D + d), acc);
    if (nsplit > 1 && t >= split_row0) add_extra(t, acc);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] *= w2_inv;
  }
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    if (row[k] >= 0) {
      float v[VEC];
      PT::widen(raw[k], v);
      if (nsplit > 1 && row[k] >= split_row0) add_extra(row[k], v);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] += g[k] * v[i];
    }
  }
  if constexpr (sizeof(OutT) == 4) {
    float* dst = (float*)y + (size_t)t * L.D + d;
#pragma unroll
    for (int i = 0; i < VEC; i += 4) *(float4*)(dst + i) = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
  } else {
    uint16_t* dst = (uint16_t*)y + (size_t)t * L.D + d;
    uint16_t o[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) o[i] = f32_to_bf16(acc[i]);
    if constexpr (VEC == 8) {
      *(uint4*)dst = make_uint4(o[0] | ((uint32_t)o[1] << 16), o[2] | ((uint32_t)o[3] << 16), o[4] | ((uint32_t)o[5] << 16),
                                o[6] | ((uint32_t)o[7] << 16));
    } else {
      *(uint2*)dst = make_uint2(o[0] | ((uint32_t)o[1] << 16), o[2] | ((uint32_t)o[3] << 16));
    }
  }
}

// The same sum for small batches, where the layer waits for this kernel's latency: a thread per (slot, 16 bytes of partial
// outputs) instead of one that goes through the slots and their extra K ranges one after the other, the slots added in the
// same order through LDS.  A workgroup takes 32 such column groups of one token.
// 1 token top-8 on 2048 columns, 8 K ranges: 11.4 -> 3.9 us; 64 tokens top-2 on 4096 columns 6.2 -> 5.3.
constexpr int kSlotCols = 32;
constexpr int kSlotThreads = 32768;  // (tokens x column groups) up to here; beyond, combine_kernel fills the chip by itself (within 1 us of each other up to 200000)
template <typename OutT, bool HALF>
__global__ __launch_bounds__(1024) void combine_slots_kernel(Layout L, const char* ws, OutT* y, const float* w2_inv_p) {
  using PT = Partials<HALF>;
  constexpr int VEC = PT::VEC;
  extern __shared__ __attribute__((aligned(16))) float part[];  // [slots][kSlotCols * VEC]
  __shared__ float weight[kMaxTopK + 1];  // of every slot; 0 where nothing was kept: a dropped pair's own weight may be NaN
  const int32_t* counters = (const int32_t*)(ws + L.o_counters);
  const int nsplit = counters[3], split_row0 = counters[4] * L.BM;
  const int has_sh = L.n_shared > 0 ? 1 : 0, slots = L.K + has_sh;
  const int DV = L.D / VEC, per = (DV + kSlotCols - 1) / kSlotCols;
  const int t = blockIdx.x / per, c0 = (blockIdx.x % per) * kSlotCols, tid = threadIdx.x;
  const int slot = tid / kSlotCols, c = c0 + tid % kSlotCols;  // slot 0: the shared experts, where there are any
  if (slot < slots) {
    float v[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = 0.f;
    const int row = slot < has_sh ? t : ((const int32_t*)(ws + L.o_pair_row))[(size_t)t * L.K + slot - has_sh];
    if (tid % kSlotCols == 0) weight[slot] = slot < has_sh ? 1.f : row >= 0 ? ((const float*)(ws + L.o_w))[(size_t)t * L.K + slot - has_sh] : 0.f;
    if (row >= 0 && c < DV) {
      const int d = c * VEC, tile = row / L.BM;
      const uint4 raw = PT::load(ws + L.o_Yp, (size_t)row * L.D + d);
      int first = nsplit > 1 && row >= split_row0 ? ((const int32_t*)(ws + L.o_split_of))[(size_t)tile * L.ND2 + d / L.BN2] : -1;
      uint4 u[kMaxSplit - 1];
      if (first >= 0) {  // see add_extra in combine_kernel
        const int rofs = first & kSplitRowsOffset ? L.BM : 0;
        first &= ~kSplitRowsOffset;
        const size_t src = ((size_t)first * L.pool_rows + (row - tile * L.BM) + rofs) * L.BN2 + d % L.BN2;
#pragma unroll
        for (int sp = 0; sp < kMaxSplit - 1; ++sp)
          u[sp] = sp + 1 < nsplit ? PT::load(ws + L.o_pool, src + (size_t)sp * L.pool_rows * L.BN2) : make_uint4(0, 0, 0, 0);
      }
      PT::widen(raw, v);
      if (first >= 0) {
#pragma unroll
        for (int sp = 0; sp < kMaxSplit - 1; ++sp) {
          float e[VEC];
          PT::widen(u[sp], e);
          if (sp + 1 < nsplit) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) v[i] += e[i];
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < VEC; i += 4) *(float4*)&part[(slot * kSlotCols + tid % kSlotCols) * VEC + i] = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
  }
  const float w2_inv = (w2_inv_p ? *w2_inv_p : 1.f) * (HALF ? 1.0f / kYpHalfScale : 1.f);
  __syncthreads();
  for (int o = tid; o < kSlotCols * VEC && c0 * VEC + o < L.D; o += blockDim.x) {
    float acc = has_sh ? part[o] * w2_inv : 0.f;
    for (int k = 0; k < L.K; ++k) {
      const float g = weight[k + has_sh] * w2_inv;
      acc += g * part[(k + has_sh) * kSlotCols * VEC + o];
    }
    if constexpr (sizeof(OutT) == 4) ((float*)y)[(size_t)t * L.D + c0 * VEC + o] = acc;
    else ((uint16_t*)y)[(size_t)t * L.D + c0 * VEC + o] = f32_to_bf16(acc);
  }
}

// any D (no vector access): one thread per output element, from q0 on
template <typename OutT>
__global__ __launch_bounds__(256) void combine_scalar_kernel(Layout L, int T, const char* ws, OutT* y, int64_t q0) {
  const float* Yp = (const float*)(ws + L.o_Yp);
  const float* w = (const float*)(ws + L.o_w);
  const int32_t* pair_row = (const int32_t*)(ws + L.o_pair_row);
  const int64_t q = q0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= (int64_t)T * L.D) return;
  const int t = (int)(q / L.D);
  const int d = (int)(q % L.D);
  const int32_t* counters = (const int32_t*)(ws + L.o_counters);
  const int nsplit = counters[3], split_row0 = counters[4] * L.BM;
  const int jd = d / L.BN2;
  auto partial = [&](int r) {  // row r of Yp and the partial-output tiles of its extra K ranges (see combine_kernel)
    float v = Yp[(size_t)r * L.D + d];
    if (nsplit > 1 && r >= split_row0) {
      const int tile = r / L.BM;
      int first = ((const int32_t*)(ws + L.o_split_of))[(size_t)tile * L.ND2 + jd];
      if (first >= 0) {
        const int rofs = first & kSplitRowsOffset ? L.BM : 0;
        first &= ~kSplitRowsOffset;
        const float* pool = (const float*)(ws + L.o_pool) + ((size_t)first * L.pool_rows + (r - tile * L.BM) + rofs) * L.BN2 + (d - jd * L.BN2);
        for (int sp = 1; sp < nsplit; ++sp) v += pool[(size_t)(sp - 1) * L.pool_rows * L.BN2];
      }
    }
    return v;
  };
  float acc = 0.f;
  for (int k = 0; k < L.K; ++k) {
    int row = pair_row[(size_t)t * L.K + k];
    if (row >= 0) acc += w[(size_t)t * L.K + k] * partial(row);
  }
  if (L.n_shared > 0) acc += partial(t);
  if constexpr (sizeof(OutT) == 4) ((float*)y)[q] = acc;
  else ((uint16_t*)y)[q] = f32_to_bf16(acc);
}

hipError_t launch_combine(const Layout& L, int T, const char* packed, char* ws, void* y, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const float* w2_inv = L.mfma ? &((const PackRecord*)(packed + L.p_scale))->unscale : nullptr;
  const int DV = L.D / (L.yp_half ? 8 : 4);
  if (L.D % 4 == 0 && (int64_t)T * DV <= kSlotThreads) {
    const int slots = L.K + (L.n_shared > 0 ? 1 : 0);
    const dim3 grid((unsigned)((DV + kSlotCols - 1) / kSlotCols * T)), block((slots * kSlotCols + 63) & ~63);
    const size_t sh = (size_t)slots * kSlotCols * 16 * (L.yp_half ? 2 : 1);
    if (L.yp_half) {
      if (L.y_f32) combine_slots_kernel<float, true><<<grid, block, sh, s>>>(L, ws, (float*)y, w2_inv);
      else combine_slots_kernel<uint16_t, true><<<grid, block, sh, s>>>(L, ws, (uint16_t*)y, w2_inv);
    } else {
      if (L.y_f32) combine_slots_kernel<float, false><<<grid, block, sh, s>>>(L, ws, (float*)y, w2_inv);
      else combine_slots_kernel<uint16_t, false><<<grid, block, sh, s>>>(L, ws, (uint16_t*)y, w2_inv);
    }
    return hipGetLastError();
  }
  if (L.D % 4 == 0) {
    int64_t n = (int64_t)T * (L.D / (L.yp_half ? 8 : 4));
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
#define DSMOE_COMBINE(KB)                                                                      \
  do {                                                                                          \
    if (L.yp_half) {                                                                              \
      if (L.y_f32) combine_kernel<float, KB, true><<<grid, block, 0, s>>>(L, T, ws, (float*)y, w2_inv); \
      else combine_kernel<uint16_t, KB, true><<<grid, block, 0, s>>>(L, T, ws, (uint16_t*)y, w2_inv);  \
    } else {                                                                                      \
      if (L.y_f32) combine_kernel<float, KB, false><<<grid, block, 0, s>>>(L, T, ws, (float*)y, w2_inv); \
      else combine_kernel<uint16_t, KB, false><<<grid, block, 0, s>>>(L, T, ws, (uint16_t*)y, w2_inv);  \
    }                                                                                             \
  } while (0)
    if (L.K <= 2) DSMOE_COMBINE(2);
    else if (L.K <= 4) DSMOE_COMBINE(4);
    else if (L.K <= 8) DSMOE_COMBINE(8);
    else DSMOE_COMBINE(16);
#undef DSMOE_COMBINE
  } else {
    const int64_t n = (int64_t)T * L.D, most = (int64_t)1 << 31;  // (a launch of 2^32 threads and more is silently cut short)
    for (int64_t q0 = 0; q0 < n; q0 += most) {
      const dim3 grid((unsigned)(((n - q0 < most ? n - q0 : most) + 255) / 256)), block(256);
      if (L.y_f32) combine_scalar_kernel<float><<<grid, block, 0, s>>>(L, T, ws, (float*)y, q0);
      else combine_scalar_kernel<uint16_t><<<grid, block, 0, s>>>(L, T, ws, (uint16_t*)y, q0);
    }
  }
  return hipGetLastError();
}

}  // namespace dsmoe
