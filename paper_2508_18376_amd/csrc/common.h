// Internal declarations shared by the translation units of libdsmoe (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/dsmoe.h"

namespace dsmoe {

constexpr int kMaxTopK = 16;
constexpr int kMaxExperts = 512;
constexpr int kMaxPart = 8;
constexpr int kSubBits = 4;  // partitions that take part in the row sort key
constexpr int kSplitItems = 256;  // one GEMM-2 item per compute unit: the granularity K splits aim at (measured best)
constexpr int kMaxSplit = 8;      // most K ranges an item is split into when there are few row tiles (decode-sized batches)
constexpr int kTallExtra = 64;    // rows beyond a full tile that a tall GEMM item takes along
constexpr int kPoolRows = 256 + kTallExtra;  // rows of a partial-output tile of the pool (kMfmaBM + kTallExtra)
constexpr int kSplitRowsOffset = 1 << 30;    // flag in the (row tile, column tile) -> pool tile table: the tile's rows sit kMfmaBM rows down
constexpr int kMaxTailSplit = 8;  // most K ranges an item of the last, partly filled round of items is split into
constexpr int kPoolTiles = 768;   // partial-output tiles (256 x 256) the extra K ranges can need at most
// Half-precision partial outputs hold the sums of GEMM-2 times 2^-10.  These are sums
// over the kept neurons of (activation x 2^k) x (W2 x 2^S) with the largest |W2 x 2^S| in [2^14, 2^15) (the images of W2 may
// carry another power of two, see PackRecord):
// for activations of order one they are of order sqrt(neurons) x 5000, i.e. 1e2 .. 1e3 after the
// scaling, with a factor 60 and more up to half precision's largest value and seven decades down to its
// smallest normal one, whatever the scale of the weights (and, through cfg.h_scale_log2, of the activations).
constexpr float kYpHalfScale = 1.0f / 1024.0f;
constexpr int kSelBins = 4096;  // grid of the row-budget thresholds: multiples of 2^-12 (a power of two keeps n * kSelBins exact)
constexpr int kSelRow = kSelBins + 4;  // a score histogram: kSelBins + 1 bins and a pair count, in whole 16-byte groups
constexpr int kSelBlocks = 16;          // workgroups of the drop-rate histogram, one row each
constexpr int kRouteBlockTokens = 64;  // tokens per block of the route kernels, one histogram row each ...
constexpr int kWaveBlockTokens = 16;   // ... except the sixteen-lanes-per-token kernel (E > 32) on small batches: 4 wavefronts x 4 tokens
constexpr int kWaveSmallBatch = 2048;  // largest batch that uses the small blocks (more blocks would swamp the plan kernel's sum)
inline __host__ __device__ int route_block_tokens(int E, int T) {
  return (E <= 32 || T > kWaveSmallBatch) ? kRouteBlockTokens : kWaveBlockTokens;
}

// MFMA path tile shape: 256 rows (token-expert pairs) x 128 neurons (gate+up = 256 weight rows)
// for GEMM-1, 256 rows x 256 output columns for GEMM-2, K stage 32.
constexpr int kMfmaBM = 256;
constexpr int kMfmaNeur = 128;
constexpr int kMfmaBN2 = 256;
constexpr int kStreamRows = 64;             // rows that a workgroup of the streaming kernels takes: batches of at most that many tokens
constexpr int kBK = 32;                     // K values per pipeline stage
constexpr int kChunksPerRow = kBK / 8;      // 16-byte chunks in one tile row
constexpr int kStageBytes = 256 * kBK * 2;  // one operand tile of one stage (bf16): 16 KiB

// full-precision path (gemm_full.hip): 64 rows (up to 128 with the expert's short last tile) x 64 neurons (gate+up = 128
// weight rows) for GEMM-1, x 128 output columns for GEMM-2, K stage 32
constexpr int kFullBM = 64;
constexpr int kFullNeur = 64;
constexpr int kFullBN2 = 128;
constexpr int kFullRows = kFullBM + kTallExtra;
constexpr int kFullSplitItems = 512;  // two GEMM-2 workgroups per compute unit
constexpr int kNonfiniteH = 10;       // counter that tiles of two weight images set: some activation is infinite or NaN (cleared by the plan)

struct Item1 {  // one tile of GEMM-1: rows [row0, row0+nrows) x neurons tile jt of partition p
  int32_t row0, nrows, e, p, jt;
  int32_t nfill;  // rows of the whole row tile (>= nrows): rows [nrows, nfill) keep nothing of p and get zeros
  int32_t half;   // 0: the whole neuron tile; 1 / 2: its first / second 64 neurons (MFMA path, at most 128 rows)
  int32_t once;   // the only item of its expert and partition that reads this weight tile
};
struct Item2 {  // one tile of GEMM-2: rows x output column tile jd, summed over partitions in kmask
  int32_t row0, nrows, e, jd, kmask;
  int32_t ks_lo, ks_n;  // K stages [ks_lo, ks_lo + ks_n) of every kept partition (the whole partition unless K is split)
  int32_t split;        // 0: the item writes its rows of Yp; n > 0: it writes partial-output tile n-1 of the pool
};

// What packing leaves beside the weights (at Layout::p_scale, cleared before it).  MFMA layout: the images of W2 carry a power of two, which is
// the sample's (pack.hip) except in the column tiles (256 columns of an expert, the unit of a GEMM-2 item) with a weight that does not fit half
// precision so.  A byte for each of them follows the record, the shared pseudo-expert's last: the (biased) exponent of its largest |W2|
// if that is of a higher binade than the sample's, else 0.
struct PackRecord {
  uint32_t largest;  // MFMA layout: bits of the sample's largest |W2|; full-precision layout of bf16: 1 if W2 has an infinity or NaN
  int32_t room;      // MFMA layout: the largest exponent that fits at the sample's scale (0: a sample that is zero or subnormal sets no scale)
  int32_t shift0;    // ... 2^shift0 is the scale of the column tiles without a larger one
  int32_t shift;     // ... 2^shift is the scale that the largest |W2| of all gives: GEMM-2's partial outputs carry it, so that their range
                     // does not hang on the sample and they all add up
  float unscale;     // ... 2^-(shift + h_shift), which the combine kernel applies
  int32_t beyond;    // ... some column tile's byte is set
  int32_t bad_perm;
  int32_t pad;
};
// the power of two that takes |W2| of (biased) exponent e to [2^14, 2^15)
__device__ __forceinline__ int w2_shift(int e) {
  const int s = e == 0 ? 0 : 14 - (e - 127);  // (0: zero or subnormal)
  return s < -80 ? -80 : s > 80 ? 80 : s;
}
// ... and that of a column tile
__device__ __forceinline__ int w2_tile_shift(int room, int shift0, int beyond) { return beyond > room ? w2_shift(beyond) : shift0; }

// Everything the device code needs to know about the layer and the workspace.
struct Layout {
  // layer
  int32_t D, F, E, K, P, Fp;
  int32_t lo, hi, E_res;      // resident window
  int32_t n_shared, F_shT;    // shared experts fused into one pseudo-expert of F_shT neurons (id E_res)
  int32_t renorm, dtype, mfma, router_mfma;
  int32_t y_f32;  // 1: y is float even though the layer's tensors are bf16
  int32_t yp_half;  // MFMA path: GEMM-2 stores its per-pair partial outputs (Yp, pool tiles) in half precision (times kYpHalfScale)
  int32_t h_shift;  // MFMA path: the intermediate activation is stored times 2^h_shift (folded into the packed W3)
  int32_t g2_rows_inner;  // GEMM-2 item order: 1 = (expert, column tile, row tile), 0 = (expert, row tile, column tile)
  int32_t tall_tiles;     // MFMA path: a GEMM item of a full row tile may also take the expert's last row tile if that has at most
                          // kTallExtra rows: 0 never, 1 where the plan's estimate says it pays (GEMM-1; always in GEMM-2), 2 wherever possible
  int32_t stream;       // MFMA path, set per call: the batch takes the streaming kernels
  int32_t split_items;  // GEMM-2 items that fill the chip: the granularity K splits aim at
  // full-precision path: K dimensions padded to whole stages (equal to the unpadded ones on the matrix-core path)
  int32_t Dk, Fpk, Fh, Fsk;  // D; F/P; row length of H (P * Fpk); F_shT
  int32_t pool_rows, BN2;    // rows of a partial-output tile of the pool; output columns of a GEMM-2 tile
  int32_t max_tokens;
  // plan geometry
  int32_t BM;                 // row tile height
  int32_t NT1, NT1_sh;        // neuron tiles per partition (routed / shared)
  int32_t ND2;                // output column tiles of GEMM-2
  int32_t wide;               // full-precision path, set per call (bf16 layers): tiles of two weight images (NT1, NT1_sh, ND2, BN2 are then those of such tiles)
  int32_t NI1, NI1_sh, NI2;   // full-precision path: weight images of a partition (routed / shared), and of W2
  int32_t nsub, nbins;        // sort bins: E_res * nsub
  int32_t sh_rows;            // rows of the shared region (multiple of BM), first in the row space: the context holds the
                              // capacity for max_tokens, the copy a call hands to its kernels the boundary for its T
  int32_t row_cap;            // total row capacity
  int32_t max_tiles, max_items1, max_items2;
  int32_t pool_tiles;         // partial-output tiles of the workspace (GEMM-2 K splits)
  // workspace byte offsets
  int64_t o_idx, o_w, o_keep, o_pair_row, o_bin_count, o_cursor, o_exp_nrows, o_exp_row0, o_counters;
  int64_t o_items1, o_items2;
  int64_t o_row_token, o_row_bits, o_H, o_Hs, o_Yp, o_sel, o_logits, o_perm_check, o_pool, o_split_of, ws_bytes;
  // packed weights byte offsets
  int64_t p_w13, p_w2, p_sw13, p_sw2, p_scale, packed_bytes, router_bytes;  // p_scale: the PackRecord and what follows it
  int64_t w13_expert_bytes, w2_expert_bytes;  // strides between experts (mfma layout)
};

// A set-up step that HIP keeps per device (hipFuncSetAttribute, hipGetSymbolAddress): run once for
// every device, with that device current, from whichever host thread gets there first.
constexpr int kMaxDevices = 64;
struct PerDeviceOnce {
  std::mutex mu;
  bool done[kMaxDevices] = {};
  template <class F>
  hipError_t run(F&& f) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return f();  // beyond the table: every time
    std::lock_guard<std::mutex> g(mu);
    if (done[dev]) return hipSuccess;
    e = f();
    if (e == hipSuccess) done[dev] = true;
    return e;
  }
};

constexpr int kNumKernels = 7;  // router, route, plan, scatter, gemm1, gemm2, combine (the first and the fourth where there are any)

struct Profile {
  int level = 0;       // 0 off, 1 GEMM-1 only, 2 every kernel
  int max_calls = 0;
  int calls = 0;
  hipEvent_t* ev = nullptr;  // level 1: 2 per call; level 2: kNumKernels + 1 per call
  uint8_t* ran = nullptr;    // per call, bit k: kernel k was launched (steps that another one's launch includes are not)
};

struct Ctx {
  dsmoe_config cfg;
  Layout L;
  int last_hip;
  int last_sh_rows;  // rows the last call reserved for the shared experts (for dsmoe_plan_layout)
  Profile prof;
};

// upper bounds of the plan sizes for a call with T tokens (the exact sizes only exist on the device)
inline int routed_tiles_bound(const Layout& L, int T) { return (int)(((int64_t)T * L.K) / L.BM) + L.E_res; }
inline int shared_tiles(const Layout& L, int T) { return L.n_shared > 0 ? (T + L.BM - 1) / L.BM : 0; }
inline int items1_whole_bound(const Layout& L, int T) {
  return routed_tiles_bound(L, T) * L.P * L.NT1 + shared_tiles(L, T) * L.NT1_sh;
}
// A last round of items may be cut into halves only in the weight-streaming regime: at most half a
// tile of rows per expert on average.
__host__ __device__ inline bool may_halve_items1(const Layout& L, int T) {
  return L.mfma && (int64_t)T * L.K <= (int64_t)L.E_res * (L.BM / 2);
}
inline int items1_bound(const Layout& L, int T) {
  return items1_whole_bound(L, T) + (may_halve_items1(L, T) ? L.split_items / 2 : 0);
}
// column tiles of W2, the shared pseudo-expert's among them
inline int w2_tiles(const Layout& L) { return (L.E_res + (L.n_shared > 0 ? 1 : 0)) * L.ND2; }
inline int items2_bound(const Layout& L, int T) {
  const int whole = (routed_tiles_bound(L, T) + shared_tiles(L, T)) * L.ND2;
  return whole + L.pool_tiles;  // every extra K range of a split item is one more item
}

// Workgroups of 256 threads for n values, one each up to 2^30 and in turns beyond: a launch of 2^32 threads and more is
// silently cut short.
inline int64_t blocks_of_256(int64_t n) { return n < (int64_t)1 << 30 ? (n + 255) / 256 : 1 << 22; }

// launchers (each returns hipError_t of the launch)
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s);
// tau == nullptr: thresholds of zero
hipError_t launch_route(const Layout& L, const float* logits, int T, const float* tau, int32_t* idx, float* w,
                        uint8_t* keep, int32_t* bin_count, int32_t* group_count, hipStream_t s);
// The normalised scores instead of routing results: their histograms per expert of the whole router (sel: rows of kSelRow,
// cleared by the caller), or the scores themselves (n [T][K], -1 where the expert is not resident; sel == nullptr).
hipError_t launch_route_scores(const Layout& L, const float* logits, int T, int32_t* sel, float* n, hipStream_t s);
// plan and, where plan_writes_rows says so, row lists; else launch_scatter has to follow
bool plan_writes_rows(const Layout& L, int T);
hipError_t launch_plan(const Layout& L, int T, char* ws, hipStream_t s);
// small batches: routing, plan and row lists in one launch
bool small_plan(const Layout& L, int T);
hipError_t launch_small_plan(const Layout& L, int T, const float* logits, const float* tau, char* ws, hipStream_t s);
hipError_t launch_scatter(const Layout& L, int T, char* ws, hipStream_t s);
hipError_t launch_combine(const Layout& L, int T, const char* packed, char* ws, void* y, hipStream_t s);
// epi: what GEMM-1 stores per (row, neuron): 0 = Swish(gate)*up (the layer), 1..4 = the profiling
// metrics Swish(gate), |Swish(gate)|, Swish(gate)*up, |Swish(gate)*up|
bool full_wide(const Layout& L, int T);
hipError_t launch_gemm1_full(const Layout& L, int T, const char* packed, const void* x, char* ws, int epi, hipStream_t s);
hipError_t launch_gemm2_full(const Layout& L, int T, const char* packed, char* ws, hipStream_t s);
hipError_t launch_gemm1_mfma(const Layout& L, int T, const char* packed, const void* x, char* ws, int epi, hipStream_t s);
hipError_t launch_select_thresholds(const Layout& L, int T, const float* logits, const float* tau_max, int group_size, int row_cap, char* ws,
                                    float* tau, int32_t* pair_count, hipStream_t s);
hipError_t launch_router_pack(const Layout& L, const void* wg, char* out, hipStream_t s);
// the router product and the routing of its batch in one launch, where router_routes() says so
bool router_routes(const Layout& L, int T);
hipError_t launch_router_route(const Layout& L, int T, const char* router_packed, const void* x, float* logits, const float* tau, char* ws,
                               hipStream_t s);
hipError_t launch_router(const Layout& L, int T, const char* router_packed, const void* x, float* logits, hipStream_t s);
hipError_t launch_transform_complete(const Layout& L, const void* wg, const void* w1, const void* w3, const void* w2,
                                     const int32_t* perm, void* wg_out, void* w1_out, void* w3_out, void* w2_out,
                                     hipStream_t s);
hipError_t launch_drop_rate_thresholds(const Layout& L, int T, const float* logits, double rate, const int32_t* offset_bins, char* ws, float* tau,
                                       int32_t* stats, hipStream_t s);
hipError_t launch_colsum(const Layout& L, const char* ws, int metric, float* importance, hipStream_t s);
hipError_t launch_perm_from_importance(const Layout& L, const float* importance, int32_t* perm, hipStream_t s);
hipError_t launch_gemm2_mfma(const Layout& L, int T, const char* packed, char* ws, hipStream_t s);
hipError_t launch_pack(const Layout& L, const void* w1, const void* w3, const void* w2, const void* sw1, const void* sw3,
                       const void* sw2, const int32_t* perm, char* packed, int n_shared, int F_sh, hipStream_t s);
// the inverse of perm; *bad: perm is not a permutation
hipError_t launch_invert_perm(const Layout& L, const int32_t* perm, int32_t* inv, int32_t* bad, hipStream_t s);

// ---- device helpers ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {  // round to nearest, ties to even
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float silu_f32(float a) { return a / (1.0f + expf(-a)); }       // Swish, beta = 1
__device__ __forceinline__ float silu_fast(float a) { return a * __builtin_amdgcn_rcpf(1.0f + __expf(-a)); }
// value GEMM-1 stores for gate g and up u (see launch_gemm1_*): Eq. 4's inner term, or one of the
// four importance metrics of Sec. 4.2 b
template <bool FAST>
__device__ __forceinline__ float epi_value(int epi, float g, float u) {
  const float sg = FAST ? silu_fast(g) : silu_f32(g);
  switch (epi) {
    case 1: return sg;
    case 2: return fabsf(sg);
    case 4: return fabsf(sg * u);
    default: return sg * u;  // 0 (layer) and 3
  }
}

// All-reductions inside a row of sixteen lanes: four data-parallel steps (mirror, half mirror, two
// quad permutations) leave the result in every lane of the row, with no LDS or scalar round trip.
constexpr int kRowMirror = 0x140, kRowHalfMirror = 0x141, kQuadSwap2 = 0x4E, kQuadSwap1 = 0xB1;
template <int CTRL>
__device__ __forceinline__ int dpp_all(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, __int_as_float(dpp_all<kRowMirror>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_all<kRowHalfMirror>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_all<kQuadSwap2>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_all<kQuadSwap1>(__float_as_int(v))));
  return v;
}
__device__ __forceinline__ float row_sum(float v) {  // every step adds two partners' values: the same bits in every lane
  v += __int_as_float(dpp_all<kRowMirror>(__float_as_int(v)));
  v += __int_as_float(dpp_all<kRowHalfMirror>(__float_as_int(v)));
  v += __int_as_float(dpp_all<kQuadSwap2>(__float_as_int(v)));
  v += __int_as_float(dpp_all<kQuadSwap1>(__float_as_int(v)));
  return v;
}

// The piece of a list of n pieces of work that this workgroup takes (n: none).  Consecutive workgroups land on different XCDs
// (round robin over 8), so each XCD gets a run of 32 consecutive pieces out of every 256 (the last ones: eight equal runs): pieces
// that share a weight tile then share an L2.
// Runs of 32 to the end left whole rounds to the first XCDs: 834 items of GEMM-1 (333 tokens on 64 + 2 experts of 2048 x 1408) were 128 each
// for two XCDs and 96 for the others, the former done after 166 us, the latter after 122; with equal runs 1 token on 64 experts of
// 2048 x 1024 takes 47.8 us instead of 49.7.
// FREE: the XCDs' shares are never equally long, so of a list of kFreeFrom pieces and more the last 128 to 383 are handed out one by one
// (*taken counts them; twice as many workgroups ask, so that an XCD that is ahead takes over from the others).  Dealt to the end -> free, us:
// 7001 tokens on 64 + 2 of 2048 x 1408 853 -> 838, 16384 on two of 8 of 4096 x 14336 1974 -> 1963, calibration with 8192 tokens on 64 of
// 2048 x 1024 592 -> 587; 4096 tokens on 8 of 4096 x 14336 and 8192 on 64 of 2048 x 1024 no difference.  Full-precision path: 777 tokens on
// 64 + 2 in parts of 176 416 -> 399, 250 / 1024 fp32 tokens on 64 of 2048 x 1024 439 -> 420 and 1169 -> 1090, 512 by the box 552 -> 544 or
// 521 -> 528, 64 on 64 of 2048 x 1000 in parts of 250 177 -> 179.  In shorter lists the free pieces are too large a part of the list for what their
// neighbours could share: free from 257 on, 128 / 512 tokens on 64 of 2048 x 1024 lost 162 -> 167 and 186 -> 193 us.  The dealt part is whole
// runs: with the last 128 or 256 free exactly, its last runs are cut at other places than the items that share a tile, and half of the gain is
// lost.  The streaming kernels, two workgroups to a unit, gain nothing from free pieces.
// lds: scratch of the workgroup, free again on return.
constexpr int kFreeFrom = 1024;
template <bool FREE>
__device__ __forceinline__ int take_piece(int n, int32_t* taken, char* lds) {
  const int b = blockIdx.x, base = b & ~255, x = b & 7, i = (b & 255) >> 3;
  const int dealt = !FREE || n < kFreeFrom ? n : (n - 128) & ~255;
  if (b < dealt) {
    const int left = min(dealt - base, 256), q = left >> 3, r = left & 7;
    return base + x * q + min(x, r) + i;
  }
  if (dealt == n || b >= 2 * n - dealt) return n;
  if (threadIdx.x == 0) *(volatile int32_t*)lds = dealt + atomicAdd(taken, 1);
  __syncthreads();
  const int id = __builtin_amdgcn_readfirstlane(*(volatile int32_t*)lds);
  __syncthreads();
  return id < n ? id : n;
}
// workgroups that take_piece<FREE> needs for at most n pieces
inline int piece_blocks(bool free, int n) { return n + (free && n >= kFreeFrom ? 384 : 0); }

// Position of the 16-byte chunk `chunk` (0..3) of row `row` inside a [rows][32] bf16 LDS tile
// (64-byte rows).  The chunks of a row are XOR-rotated by bits 2..3 of the row so that an MFMA
// operand read (consecutive rows, same logical chunk) touches every LDS bank once per 16 lanes.
// XOR is its own inverse: the same function maps physical to logical positions.
__device__ __host__ __forceinline__ int swz_chunk(int row, int chunk) { return chunk ^ ((row >> 2) & 3); }
// the same for the full-precision path's tiles, whose rows have CH = 4 (bf16) or 8 (fp32) chunks
template <int CH>
__device__ __host__ __forceinline__ int swz_full(int row, int chunk) {
  return CH == 4 ? swz_chunk(row, chunk) : chunk ^ (row & 7);
}

}  // namespace dsmoe
