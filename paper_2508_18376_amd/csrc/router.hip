// Gating logits l = x W_g (Sec. 3.1 of the paper, first equation; W_g is [d_model][E]): the small
// product in front of the softmax of Eq. 1.  HBM-bound: x is read once, W_g stays in L2.
//
// bf16 layers with d_model % 64 == 0 use the matrix cores.  W_g is repacked once into MFMA operand
// order, so a lane fetches its 8 values of an operand with one 16-byte load and a wavefront reads
// 1 KiB contiguous per operand.  x comes straight from memory in operand order too: with 16 x 16 blocks four lanes
// cover 64 contiguous bytes of a token (32 x 32 blocks would touch 64 separate 16-byte pieces per load, which the
// address units take one by one).
#include "route.h"

namespace dsmoe {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kRouterStep = 64;    // contraction values per step
// Workgroups of 16 tokens up to here, of 32 beyond (which read W_g half as often): there the smaller ones would be more than
// the compute units.
constexpr int kRouterFewTokens = 16 * 256;

// packed W_g, MFMA path: chunk ((ks*2 + m)*NT + nt)*64 + lane holds W_g[ks*64 + m*32 + (lane/16)*8 + i][nt*16 + lane%16],
// i = 0..7 (zero for experts >= E).  One thread per chunk.
__global__ void router_pack_mfma_kernel(const uint16_t* __restrict__ wg, uint16_t* __restrict__ out, int D, int E, int NT) {
  const int64_t total = (int64_t)(D / kRouterStep) * 2 * NT * 64;
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= total) return;
  const int lane = (int)(q & 63);
  int64_t r = q >> 6;
  const int nt = (int)(r % NT);
  r /= NT;
  const int m = (int)(r & 1);
  const int ks = (int)(r >> 1);
  const int e = nt * 16 + (lane & 15);
  const int d0 = ks * kRouterStep + m * 32 + (lane >> 4) * 8;
  for (int i = 0; i < 8; ++i) out[q * 8 + i] = e < E ? wg[(size_t)(d0 + i) * E + e] : (uint16_t)0;
}

// generic path: W_g widened to float, same [D][E] layout
template <typename T>
__global__ void router_pack_generic_kernel(const T* __restrict__ wg, float* __restrict__ out, int64_t n) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  if constexpr (sizeof(T) == 2) out[q] = bf16_to_f32(wg[q]);
  else out[q] = wg[q];
}

// Workgroup = MT * 16 tokens x (NT tiles of 16 experts); its W wavefronts take every W-th 64-step of the
// contraction (enough loads in flight to stream x at HBM rate even for a few thousand tokens) and
// add their partial tiles through LDS in a fixed order, so results are reproducible bit for bit.
// ROUTE: the workgroup's logits (all E experts are in it) stay in LDS and are routed there, one histogram row per workgroup, as
// route_row_kernel would: a launch and a round trip through memory less.
// Measured: 1 token x 2048 x 64 experts 7.1 -> 4.2 us, 64 x 4096 x 8 16.5 -> 9, 333 x 2048 x 64 12.2 -> 7.2, 8192 x 2048 x 64 20.6 -> 18.
template <int NT, int W, int MT, bool ROUTE>
__global__ __launch_bounds__(W * 64) void router_mfma_kernel(const uint16_t* __restrict__ x, const uint4* __restrict__ wgp,
                                                             float* __restrict__ logits, int T, int D, int E, int NT_all, RouteArgs ra) {
  extern __shared__ float part[];  // [W][MT][NT][4][64]: wavefront, 16 tokens, tile, accumulator register, lane
  float* rows = part + W * MT * NT * 256;                    // ROUTE: [16][E] logits,
  int32_t* hist = (int32_t*)(rows + 16 * NT * 16);           // the histogram
  float* tau_l = (float*)(hist + ra.nhist);                  // and the threshold table
  static_assert(!ROUTE || (MT == 1 && MT * 16 == kWaveBlockTokens), "one histogram row for 16 tokens");
  if (ROUTE) route_row_setup(ra, hist, tau_l, W * 64);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int t0 = blockIdx.x * (MT * 16);
  const int nt0 = blockIdx.y * NT;
  const uint4* xa[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)  // rows past the end re-read the last token; not stored
    xa[i] = (const uint4*)(x + (size_t)min(t0 + i * 16 + (lane & 15), T - 1) * D + (lane >> 4) * 8);
  const int KS = D / kRouterStep;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int tile[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) tile[j] = min(nt0 + j, NT_all - 1);  // a group's tiles past the end repeat the last one; not stored
  // S steps at a time, all their loads of x (the ones that come from HBM) in flight together: a wavefront has only a few
  // steps in all, and one load latency per step was most of the kernel
  constexpr int S = NT * MT <= 4 ? 4 : 2;
  for (int k0 = w; k0 < KS; k0 += S * W) {
    uint4 a[S][2][MT];
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int ks = min(k0 + u * W, KS - 1);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < MT; ++i) a[u][m][i] = xa[i][ks * 8 + m * 4];
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int ks = k0 + u * W;
      if (ks >= KS) break;
      uint4 b[2][NT];
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j) b[m][j] = wgp[((size_t)(ks * 2 + m) * NT_all + tile[j]) * 64 + lane];
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int i = 0; i < MT; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u][m][i]), __builtin_bit_cast(bf16x8, b[m][j]), acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[(((w * MT + i) * NT + j) * 4 + v) * 64 + lane] = acc[i][j][v];
  __syncthreads();
  // value (i, j, v, l): token t0 + 16*i + 4*(l/16) + v, expert (nt0+j)*16 + l%16
  for (int o = tid; o < MT * NT * 256; o += W * 64) {
    const int l = o & 63, v = (o >> 6) & 3, j = (o >> 8) % NT, i = (o >> 8) / NT;
    float sum = 0.f;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) sum += part[(((ww * MT + i) * NT + j) * 4 + v) * 64 + l];
    const int e = (nt0 + j) * 16 + (l & 15);
    const int t = t0 + 16 * i + 4 * (l >> 4) + v;
    if (nt0 + j < NT_all && e < E && t < T) {
      logits[(size_t)t * E + e] = sum;
      if (ROUTE) rows[(t - t0) * E + e] = sum;
    }
  }
  if constexpr (ROUTE) {
    __syncthreads();
    route_row_tokens<(NT + 3) / 4, 1, W, kRoute>(ra, rows, t0, min(T, t0 + 16), hist, tau_l, nullptr);
    __syncthreads();
    flush_hist(ra, hist, W * 64);
  }
}

// generic path: a wavefront per token, lanes stride over d_model, experts in chunks of 8
template <typename T>
__global__ __launch_bounds__(256) void router_generic_kernel(const T* __restrict__ x, const float* __restrict__ wgf,
                                                             float* __restrict__ logits, int Tn, int D, int E) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= Tn) return;
  for (int e0 = 0; e0 < E; e0 += 8) {
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    for (int d = lane; d < D; d += 64) {
      float xv;
      if constexpr (sizeof(T) == 2) xv = bf16_to_f32(x[(size_t)t * D + d]);
      else xv = x[(size_t)t * D + d];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (e0 + j < E) acc[j] = fmaf(xv, wgf[(size_t)d * E + e0 + j], acc[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float v = acc[j];
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == 0 && e0 + j < E) logits[(size_t)t * E + e0 + j] = v;
    }
  }
}

hipError_t launch_router_pack(const Layout& L, const void* wg, char* out, hipStream_t s) {
  if (L.router_mfma) {
    const int NT = (L.E + 31) / 32 * 2;
    const int64_t total = (int64_t)(L.D / kRouterStep) * 2 * NT * 64;
    router_pack_mfma_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>((const uint16_t*)wg, (uint16_t*)out, L.D,
                                                                                        L.E, NT);
  } else {
    const int64_t n = (int64_t)L.D * L.E;
    const dim3 grid((unsigned)((n + 255) / 256));
    if (L.dtype == DSMOE_F32) router_pack_generic_kernel<float><<<grid, dim3(256), 0, s>>>((const float*)wg, (float*)out, n);
    else router_pack_generic_kernel<uint16_t><<<grid, dim3(256), 0, s>>>((const uint16_t*)wg, (float*)out, n);
  }
  return hipGetLastError();
}

template <int NT, int W, int MT, bool ROUTE>
static hipError_t launch_router_tokens(const Layout& L, int T, const uint4* wgp, const void* x, float* logits, int NT_all, const RouteArgs& ra, hipStream_t s) {
  constexpr int lds = W * MT * NT * 4 * 64 * 4, most = lds + (ROUTE ? 16 * NT * 16 * 4 + NT * 16 * ((1 << kSubBits) + kMaxPart) * 4 : 0);
  static PerDeviceOnce once;  // one per instantiation
  hipError_t e = once.run([] { return hipFuncSetAttribute((const void*)router_mfma_kernel<NT, W, MT, ROUTE>, hipFuncAttributeMaxDynamicSharedMemorySize, most); });
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((T + MT * 16 - 1) / (MT * 16)), (unsigned)((NT_all + NT - 1) / NT));
  router_mfma_kernel<NT, W, MT, ROUTE><<<grid, dim3(W * 64), most, s>>>((const uint16_t*)x, wgp, logits, T, L.D, L.E, NT_all, ra);
  return hipGetLastError();
}
template <int NT, int W>
static hipError_t launch_router_mfma(const Layout& L, int T, const uint4* wgp, const void* x, float* logits, int NT_all, hipStream_t s) {
  if (T <= kRouterFewTokens) return launch_router_tokens<NT, W, 1, false>(L, T, wgp, x, logits, NT_all, RouteArgs{}, s);
  return launch_router_tokens<NT, W, 2, false>(L, T, wgp, x, logits, NT_all, RouteArgs{}, s);
}

// Batches whose routing goes with the router product: those that route_row_kernel routes in blocks of the 16 tokens that a
// router workgroup has, if that workgroup sees all experts.  (Up to 32 experts routing takes a lane per token instead; beyond 128 an
// expert group each has its own workgroup; larger batches count 64 tokens to a histogram row, so that the plan has fewer rows to add.)
// 333 tokens on 64 + 2 experts of 2048 x 1408: 242.7 us in two launches, 238.9 in one.
bool router_routes(const Layout& L, int T) { return L.router_mfma && L.E > 32 && L.E <= 128 && T <= kWaveSmallBatch; }

hipError_t launch_router_route(const Layout& L, int T, const char* router_packed, const void* x, float* logits, const float* tau, char* ws,
                               hipStream_t s) {
  if (T <= 0) return hipSuccess;
  RouteArgs a = {};
  a.tau = tau;
  a.idx = (int32_t*)(ws + L.o_idx);
  a.w = (float*)(ws + L.o_w);
  a.keep = (uint8_t*)(ws + L.o_keep);
  a.bin_count = (int32_t*)(ws + L.o_bin_count);
  a.T = T;
  set_route_layer(L, a);
  const uint4* wgp = (const uint4*)router_packed;
  const int NT = (L.E + 31) / 32 * 2;
  if (NT == 4) return launch_router_tokens<4, 16, 1, true>(L, T, wgp, x, logits, NT, a, s);
  return launch_router_tokens<8, 8, 1, true>(L, T, wgp, x, logits, NT, a, s);
}

hipError_t launch_router(const Layout& L, int T, const char* router_packed, const void* x, float* logits, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  if (L.router_mfma) {
    const int NT = (L.E + 31) / 32 * 2;
    const uint4* wgp = (const uint4*)router_packed;
    if (NT == 2) return launch_router_mfma<2, 16>(L, T, wgp, x, logits, NT, s);
    if (NT == 4) return launch_router_mfma<4, 16>(L, T, wgp, x, logits, NT, s);
    return launch_router_mfma<8, 8>(L, T, wgp, x, logits, NT, s);
  } else {
    const dim3 grid((unsigned)((T + 3) / 4));
    if (L.dtype == DSMOE_F32) router_generic_kernel<float><<<grid, dim3(256), 0, s>>>((const float*)x, (const float*)router_packed, logits, T, L.D, L.E);
    else router_generic_kernel<uint16_t><<<grid, dim3(256), 0, s>>>((const uint16_t*)x, (const float*)router_packed, logits, T, L.D, L.E);
  }
  return hipGetLastError();
}

}  // namespace dsmoe
