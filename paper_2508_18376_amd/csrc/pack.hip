// moe_partition_weights kernels: neuron reorder through perm (Sec. 4.2 b), even split into P
// sub-experts with no W2 scaling (Sec. 3.2), written in the layout the GEMM kernels read.
//
// Full-precision layout (element type = layer dtype): the same idea with tiles of 128 weight rows x 32 K values:
//   W13  stage ((e*P + p)*NT1 + jt)*(Dk/32) + ks : weight row q*32 + gu*16 + j is neuron p*Fp + jt*64 + q*16 + j of W1
//        (gu=0) or W3 (gu=1)
//   W2   stage (e*ND2 + jd)*(P*Fpk/32) + kt : 128 output columns x 32 neurons; every partition is padded with zeros to
//        whole stages (Fpk), as is D (Dk)
//   bf16 layers: int32 at p_scale, 1 if some W2 value is infinite or NaN (GEMM-2 then treats such weights apart)
// MFMA layout (bf16): 16 KiB "stage images", each the exact LDS contents of one operand tile of
//   one pipeline stage, rows of kBK = 32 K-values with the 16-byte chunks XOR-rotated (swz_chunk):
//   W13  stage ((e*P + p)*NT1 + jt)*(D/32) + ks : 256 weight rows x 32 values of d; weight row
//        q*64 + gu*32 + j  is neuron  p*Fp + jt*128 + q*32 + j  of W1 (gu=0) or W3 (gu=1): every 64
//        weight rows hold the gate and the up projection of the same 32 neurons
//   W2   stage (e*ND2 + jd)*(F/32) + kt : 256 output columns x 32 neurons (positions kt*32..),
//        as IEEE half precision times 2^s (GEMM-2 multiplies half-precision operands: its left
//        operand, the intermediate activation, needs more significant bits than bf16 has).  s is
//        chosen per layer so that the largest |W2| of a sample lands in [2^14, 2^15) (all of a W2 of up to 16 M values;
//        otherwise every 3rd to 63rd run of 2048): every bf16 value within a factor 2^-29 of that is then exactly
//        representable (smaller ones round to the subnormal grid, 2^-39 of it).  A layer with a larger |W2| that no longer
//        fits half precision is packed again from the largest of all.  The combine kernel multiplies by 2^-s, exactly.
//        The record (PackRecord) sits at p_scale.
//   W3 carries the factor 2^k of cfg.h_scale_log2 (exact in bf16), so that the intermediate activation
//        comes out of GEMM-1 times 2^k, in the range half precision resolves best, at no run-time cost.
//   neurons / columns past the end are zero.
#include "common.h"

namespace dsmoe {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_once(const void* p) {  // non-temporal
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// largest finite |w| of a bf16 tensor, as its bit pattern (monotone in the value), into *out: of every stride-th run of 2048
// values.  Bound by HBM: four runs in flight per workgroup, non-temporal, and one atomic per workgroup (all on one address).
// 0.94 GB, all of it: 160 us (with plain loads and an atomic per wavefront 205); of it a sample of 16 M values 27 us (the atomics of
// 2048 workgroups), of 8 M values by 512 workgroups 10 us.
constexpr int kAbsmaxRun = 2048;
__global__ __launch_bounds__(256) void absmax_bf16_kernel(const uint16_t* w, int64_t n, int stride, uint32_t* out) {
  uint32_t m = 0;
  auto one = [&](uint32_t a) { m = a < 0x7f80u && a > m ? a : m; };
  auto eight = [&](uint4 v) {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      one(d[k] & 0x7fffu);
      one((d[k] >> 16) & 0x7fffu);
    }
  };
  const bool vec = (((uintptr_t)w) & 15) == 0;
  const int64_t step = (int64_t)gridDim.x * stride * kAbsmaxRun;
  int64_t i = (int64_t)blockIdx.x * stride * kAbsmaxRun + threadIdx.x * 8;
  if (vec) {
    for (; i + 3 * step + 8 <= n; i += 4 * step) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = load_once(w + i + u * step);
#pragma unroll
      for (int u = 0; u < 4; ++u) eight(v[u]);
    }
    for (; i + 8 <= n; i += step) eight(load_once(w + i));
  }
  for (; i < n; i += step)
    for (int64_t k = i; k < n && k < i + 8; ++k) one(w[k] & 0x7fffu);
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  __shared__ uint32_t wave_max[4];
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
    if (m) atomicMax(out, m);
  }
}
static void launch_absmax(const void* w, int64_t n, int stride, PackRecord* rec, hipStream_t s) {
  const int most = stride == 1 && n > (int64_t)1 << 26 ? 2048 : 512;
  const int64_t runs = (n + (int64_t)stride * kAbsmaxRun - 1) / ((int64_t)stride * kAbsmaxRun);
  const int blocks = (int)(runs < most ? runs : most);
  absmax_bf16_kernel<<<dim3(blocks), dim3(256), 0, s>>>((const uint16_t*)w, n, stride, &rec->largest);
}
// The scale is needed before the first value is packed, and finding the largest of all |W2| reads W2 once more (a tenth
// of the packing of 8 experts of 4096 x 14336, which took 1.52 ms with it and takes 1.36 without).  A sample of 8 to 16 M values tells its
// binade as well as that binade and the next have room for: only a W2 whose largest value is more than twice (for some, four
// times) the sample's largest is packed twice.  Odd strides: a row of a power of two of values is met in all of its columns.
static int absmax_stride(int64_t n) {
  const int64_t k = n >> 23;
  return k < 2 ? 1 : k > 63 ? 63 : (int)(k | 1);
}

// largest |W2| bits -> s with largest * 2^s in [2^14, 2^15)
__device__ __forceinline__ int w2_shift(uint32_t largest) {
  const int e = (int)(largest >> 7);  // biased exponent (0: zero or subnormal)
  const int s = e == 0 ? 0 : 14 - (e - 127);
  return s < -80 ? -80 : s > 80 ? 80 : s;
}

// a bf16 value times 2^k (k = L.h_shift), exact unless it leaves bf16's exponent range
__device__ __forceinline__ uint16_t bf16_shift(uint16_t b, int k) {
  return k == 0 ? b : f32_to_bf16(ldexpf(bf16_to_f32(b), k));
}

__device__ __forceinline__ uint16_t bf16_to_scaled_half(uint16_t b, float scale) {
  const _Float16 h = (_Float16)(bf16_to_f32(b) * scale);  // the product is exact; one rounding (none for values in range)
  return __builtin_bit_cast(uint16_t, h);
}

// The MFMA stage images are made by transposing tiles of 32 source rows x 512 bytes through LDS: rows come in
// as whole 512-byte segments (16 bytes per lane), image rows leave as 64-byte runs (four 16-byte chunks of
// neighbouring lanes), so both directions move a tensor once and in wide pieces; bound by HBM.  Weights of 8
// experts of 4096 x 14336: W1 / W3 (3.76 GB read + written, random order) 835 us = 4.5 TB/s, W2 (1.88 GB) 430 us
// = 4.4 TB/s.  (One thread per column with 32 2-byte loads, resp. per 16-byte chunk with eight of them, took 1295 and
// 1181 us: 2.9 and 1.6 TB/s.)  W1 / W3 are read with the non-temporal hint (850 -> 835 us).  Nothing else is: the scattered
// 64-byte runs need the caches to become whole lines (835 -> 900 us), and the hint on W2's rows or images gained nothing for
// the pass and the first batch together.  (W2 took 390 us while absmax_bf16_kernel, in front of it, still left a part of W2 in
// the last-level cache; that kernel gained more.)
constexpr int kTileStride = 128 + 2;  // dwords between tile rows in LDS: a wavefront reads 4 chunks x 16 column pairs (bf16) or
                                      // 8 chunks x 8 columns (fp32) at once, whose rows then lie on 64 different banks
template <typename T>
struct PackTile {
  static constexpr int V = 16 / sizeof(T);         // values of a 16-byte chunk
  static constexpr int COLS = 512 / sizeof(T);     // columns of a tile
  static constexpr int CH = kBK / V;               // chunks of an image row
  static constexpr int COLS_GET = sizeof(T) == 2 ? 2 : 1;  // columns that get() returns
  static constexpr int PASSES = COLS * CH / COLS_GET / 256;
  uint32_t at[kBK * kTileStride];
  // sixteen bytes of a source row from column col on (zeros past the end; nullptr: a row of zeros)
  template <bool ONCE>
  static __device__ __forceinline__ uint4 load(const T* row, int col, int ncols, bool vec) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row == nullptr || col >= ncols) return v;
    if (vec) return ONCE ? load_once(row + col) : *(const uint4*)(row + col);
    uint32_t u[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (col + i < ncols) {
        if constexpr (sizeof(T) == 2) u[i >> 1] |= (uint32_t)row[col + i] << (16 * (i & 1));
        else u[i] = __float_as_uint(row[col + i]);
      }
    return make_uint4(u[0], u[1], u[2], u[3]);
  }
  __device__ __forceinline__ void put(int r, int lane32, uint4 v) {
    uint2* d = (uint2*)&at[r * kTileStride + lane32 * 4];
    d[0] = make_uint2(v.x, v.y);
    d[1] = make_uint2(v.z, v.w);
  }
  // chunk lc (V K values: tile rows lc * V ..) of columns c * COLS_GET ..
  __device__ __forceinline__ void get(int lc, int c, uint4 (&o)[COLS_GET]) const {
    uint32_t u[V];
#pragma unroll
    for (int i = 0; i < V; ++i) u[i] = at[(lc * V + i) * kTileStride + c];
    if constexpr (sizeof(T) == 2) {
      o[0] = make_uint4(__builtin_amdgcn_perm(u[1], u[0], 0x05040100), __builtin_amdgcn_perm(u[3], u[2], 0x05040100),
                        __builtin_amdgcn_perm(u[5], u[4], 0x05040100), __builtin_amdgcn_perm(u[7], u[6], 0x05040100));
      o[1] = make_uint4(__builtin_amdgcn_perm(u[1], u[0], 0x07060302), __builtin_amdgcn_perm(u[3], u[2], 0x07060302),
                        __builtin_amdgcn_perm(u[5], u[4], 0x07060302), __builtin_amdgcn_perm(u[7], u[6], 0x07060302));
    } else {
      o[0] = make_uint4(u[0], u[1], u[2], u[3]);
    }
  }
};

template <class Op>
__device__ __forceinline__ uint4 map_halves(uint4 v, Op op) {
  uint32_t* u = (uint32_t*)&v;
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = op((uint16_t)u[i]) | ((uint32_t)op((uint16_t)(u[i] >> 16)) << 16);
  return v;
}

// The largest finite one of eight bf16 values, as its bits, if it is of a higher binade than `sampled`, the largest of the sample (or normal
// where all of the sample is zero or subnormal); else 0.
__device__ __forceinline__ uint32_t beyond_sample(uint4 raw, uint32_t sampled) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  const uint32_t r[4] = {raw.x, raw.y, raw.z, raw.w}, binade = sampled | 0x7fu;
  u16x2 m = {0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, r[i] & 0x7fff7fffu));
  uint32_t most = 0;
  if (m.x > binade || m.y > binade) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a = r[i >> 1] >> (16 * (i & 1)) & 0x7fffu;
      if (a > binade && a < 0x7f80u) most = max(most, a);
    }
  }
  return most;
}
// the largest exponent that fits half precision at the scale of the sample; 0: a sample that is zero or subnormal sets no scale
__device__ __forceinline__ int w2_room(uint32_t sampled) { return sampled < 0x80u ? 0 : 142 - w2_shift(sampled); }

// some of the eight bf16 values is infinite or NaN
__device__ __forceinline__ bool not_finite(uint4 v) {
  auto one = [](uint32_t u) { return (u & 0x7f80u) == 0x7f80u || (u & 0x7f800000u) == 0x7f800000u; };
  return one(v.x) || one(v.y) || one(v.z) || one(v.w);
}

// Where neuron nin of a partition sits in its W13 images: neuron tile, image row of its gate projection; the up row is UP
// rows further down.  FULL: the full-precision layout.
template <typename T, bool FULL>
struct W13Image {
  static constexpr int NEUR = FULL ? kFullNeur : kMfmaNeur, UP = FULL ? 16 : 32, RB = kBK * sizeof(T);
  static constexpr int64_t STAGE = 2 * NEUR * RB;
  static __device__ __forceinline__ int row(int nin) { return nin % NEUR / UP * (2 * UP) + nin % UP; }
  static __device__ __forceinline__ int at(int row, int lc) { return row * RB + swz_full<RB / 16>(row, lc) * 16; }
};

// W1 / W3 -> W13 images.  A workgroup takes the COLS original neurons (columns) of one expert and one K stage (32
// rows d) of both matrices and writes each neuron's gate and up image rows at the place the inverse permutation
// names (inv == nullptr: identity order).  w1, w3: [experts][D][Fs]; column c of expert e is neuron pos0 * e + c of
// image expert e * per_expert (the shared experts are consecutive neurons of one image expert: per_expert 0).
// What is left to the 5.3 TB/s of a large copy are the 64-byte runs that a random order scatters.
template <typename T, bool FULL>
__global__ __launch_bounds__(256) void pack_w13_kernel(const T* w1, const T* w3, const int32_t* inv, char* out, int D, int KS1,
                                                       int Fs, int Fp, int P, int NT1, int pos0, int per_expert, int h_shift, int vec) {
  using PT = PackTile<T>;
  using Im = W13Image<T, FULL>;
  __shared__ PT t1, t3;
  const int nc = (Fs + PT::COLS - 1) / PT::COLS;
  const int c0 = (int)(blockIdx.x % nc) * PT::COLS, ks = blockIdx.x / nc, e = blockIdx.y, tid = threadIdx.x;
  uint4 a[4], b[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int d = ks * kBK + u * 8 + (tid >> 5);
    const size_t row = ((size_t)e * D + d) * Fs;
    a[u] = PT::template load<true>(d < D ? w1 + row : nullptr, c0 + (tid & 31) * PT::V, Fs, vec);
    b[u] = PT::template load<true>(d < D ? w3 + row : nullptr, c0 + (tid & 31) * PT::V, Fs, vec);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    t1.put(u * 8 + (tid >> 5), tid & 31, a[u]);
    if (!FULL && h_shift) b[u] = map_halves(b[u], [&](uint16_t v) { return (uint32_t)bf16_shift(v, h_shift); });
    t3.put(u * 8 + (tid >> 5), tid & 31, b[u]);
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < PT::PASSES; ++pass) {
    const int lc = tid % PT::CH, cg = (pass * 256 + tid) / PT::CH;
    uint4 g[PT::COLS_GET], u[PT::COLS_GET];
    t1.get(lc, cg, g);
    t3.get(lc, cg, u);
#pragma unroll
    for (int i = 0; i < PT::COLS_GET; ++i) {
      const int c = c0 + cg * PT::COLS_GET + i;
      if (c >= Fs) continue;
      const int pos = inv ? inv[(size_t)e * Fs + c] : pos0 * e + c;
      if (inv && (uint32_t)pos >= (uint32_t)Fs) continue;  // not a permutation (reported when all is done)
      const int p = pos / Fp, nin = pos - p * Fp;
      const int row = Im::row(nin);
      char* stage = out + ((((int64_t)e * per_expert * P + p) * NT1 + nin / Im::NEUR) * KS1 + ks) * Im::STAGE;
      *(uint4*)(stage + Im::at(row, lc)) = g[i];
      *(uint4*)(stage + Im::at(row + Im::UP, lc)) = u[i];
    }
  }
}

// W2 -> W2 images (matrix-core path: half precision times the layer's power of two).  A workgroup takes 32 neuron positions
// (source rows, in permuted order; zeros past the end of a partition) x COLS output columns: one stage image, or two
// of 128 columns.  w2: [experts][P * Fp][D]; KSp: stages of a partition, KT: of the expert, nd: column tiles of the images.
template <typename T, bool FULL>
__global__ __launch_bounds__(256) void pack_w2_kernel(const T* w2, const int32_t* perm, char* out, PackRecord* rec, int D, int F, int Fp,
                                                      int KSp, int KT, int nd, int vec) {
  using PT = PackTile<T>;
  constexpr int BN = FULL ? kFullBN2 : kMfmaBN2, RB = kBK * sizeof(T);
  __shared__ PT t;
  const int nb = (D + PT::COLS - 1) / PT::COLS;
  const int c0 = (int)(blockIdx.x % nb) * PT::COLS, kt = blockIdx.x / nb, e = blockIdx.y, tid = threadIdx.x;
  float scale = 1.f;
  uint32_t sampled = 0;  // largest |W2| of the sample
  if (!FULL) {
    sampled = rec->largest;
    scale = __uint_as_float((uint32_t)(127 + w2_shift(sampled)) << 23);
  }
  uint4 a[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int in = kt % KSp * kBK + u * 8 + (tid >> 5), pos = kt / KSp * Fp + in;
    const T* row = nullptr;
    if (in < Fp) {
      const int src = perm ? perm[(size_t)e * F + pos] : pos;
      if ((uint32_t)src < (uint32_t)F) row = w2 + ((size_t)e * F + src) * D;  // (not a permutation: reported when all is done)
    }
    a[u] = PT::template load<false>(row, c0 + (tid & 31) * PT::V, D, vec);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if constexpr (!FULL) {
      if (const uint32_t most = beyond_sample(a[u], sampled)) {
        atomicMax(&rec->beyond, (int)(most >> 7));
        if ((int)(most >> 7) > w2_room(sampled)) rec->repack = 1;
      }
      a[u] = map_halves(a[u], [&](uint16_t v) { return (uint32_t)bf16_to_scaled_half(v, scale); });
    }
    if (FULL && sizeof(T) == 2 && not_finite(a[u])) rec->largest = 1;
    t.put(u * 8 + (tid >> 5), tid & 31, a[u]);
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < PT::PASSES; ++pass) {
    const int lc = tid % PT::CH, cg = (pass * 256 + tid) / PT::CH;
    uint4 o[PT::COLS_GET];
    t.get(lc, cg, o);
#pragma unroll
    for (int i = 0; i < PT::COLS_GET; ++i) {
      const int c = c0 + cg * PT::COLS_GET + i, jd = c / BN, row = c % BN;
      if (jd >= nd) continue;
      char* stage = out + (((int64_t)e * nd + jd) * KT + kt) * (BN * RB);
      *(uint4*)(stage + row * RB + swz_full<RB / 16>(row, lc) * 16) = o[i];
    }
  }
}

// image rows of the neurons past the end of a partition (its last neuron tile is not full): zeros.
// groups: (expert, partition) pairs of the images at `out`
template <typename T, bool FULL>
__global__ __launch_bounds__(256) void pack_w13_padding_kernel(char* out, int groups, int Fp, int NT1, int KS1) {
  using Im = W13Image<T, FULL>;
  constexpr int CH = Im::RB / 16;
  const int pad = NT1 * Im::NEUR - Fp;  // neurons per group that do not exist
  const int64_t total = (int64_t)groups * KS1 * pad * 2 * CH;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
    const int pc = (int)(t % CH);
    int64_t r = t / CH;
    const int gu = (int)(r % 2);
    r /= 2;
    const int nin = Fp + (int)(r % pad);
    r /= pad;
    const int ks = (int)(r % KS1);
    const int64_t ep = r / KS1;  // e * P + p
    char* stage = out + ((ep * NT1 + nin / Im::NEUR) * KS1 + ks) * Im::STAGE;
    *(uint4*)(stage + (Im::row(nin) + gu * Im::UP) * Im::RB + pc * 16) = make_uint4(0, 0, 0, 0);
  }
}

// inv[e][perm[e][pos]] = pos
__global__ void invert_perm_kernel(const int32_t* perm, int32_t* inv, int F, int64_t n) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int64_t e = t / F;
  const int src = perm[t];
  if (src >= 0 && src < F) inv[e * F + src] = (int32_t)(t % F);
}
// *bad: some neuron is not the one that perm names at the position inv has for it, i.e. none names it (inv is whatever was
// there before), so perm is no permutation
__global__ void perm_check_kernel(const int32_t* perm, const int32_t* inv, int F, int64_t n, int32_t* bad) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int64_t e = t / F;
  const int pos = inv[t];
  if (pos < 0 || pos >= F || perm[e * F + pos] != (int)(t % F)) *bad = 1;
}
hipError_t launch_invert_perm(const Layout& L, const int32_t* perm, int32_t* inv, int32_t* bad, hipStream_t s) {
  const int64_t n = (int64_t)L.E_res * L.F;
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  invert_perm_kernel<<<grid, block, 0, s>>>(perm, inv, L.F, n);
  perm_check_kernel<<<grid, block, 0, s>>>(perm, inv, L.F, n, bad);
  return hipGetLastError();
}

// the powers of two that GEMM-2 and the combine kernel apply, once all of W2 has been looked at
__global__ void w2_record_kernel(PackRecord* rec, int h_shift) {
  const int packed = w2_shift(rec->largest), all = rec->beyond ? w2_shift((uint32_t)rec->beyond << 7) : packed;
  rec->yscale = ldexpf(1.f, all - packed);
  rec->unscale = ldexpf(1.f, -all - h_shift);
}

template <typename T, bool FULL>
static void w2_images(const Layout& L, const void* w2, const void* sw2, const int32_t* perm, char* packed, hipStream_t s) {
  auto images = [&](const void* w, const int32_t* order, char* out, int experts, int F, int Fp, int Fpk) {
    const int KSp = Fpk / kBK, KT = F / Fp * KSp, C = PackTile<T>::COLS;
    const int vec = L.D % PackTile<T>::V == 0 && ((uintptr_t)w & 15) == 0;
    pack_w2_kernel<T, FULL><<<dim3((unsigned)((L.D + C - 1) / C * KT), experts), dim3(256), 0, s>>>(
        (const T*)w, order, out, (PackRecord*)(packed + L.p_scale), L.D, F, Fp, KSp, KT, L.ND2, vec);
  };
  images(w2, perm, packed + L.p_w2, L.E_res, L.F, L.Fp, L.Fpk);
  if (L.n_shared > 0) images(sw2, nullptr, packed + L.p_sw2, 1, L.F_shT, L.F_shT, L.Fsk);
  if (!FULL) w2_record_kernel<<<dim3(1), dim3(1), 0, s>>>((PackRecord*)(packed + L.p_scale), L.h_shift);
}

template <typename T, bool FULL>
static hipError_t pack_images(const Layout& L, const void* w1, const void* w3, const void* w2, const void* sw1, const void* sw3, const void* sw2,
                              const int32_t* perm, char* packed, int n_shared, int F_sh, hipStream_t s) {
  const dim3 block(256);
  const int KS1 = L.Dk / kBK, C = PackTile<T>::COLS;
  // The W1 / W3 stages are written from source columns (see pack_w13_kernel), which needs the inverse
  // permutation: it is parked in the W2 region of the packed buffer, which the W2 kernel overwrites.
  // (That region has at least E_res * F * 32 * sizeof(T) bytes, the table E_res * F * 4.)
  int32_t* inv = nullptr;
  if (perm) {
    inv = (int32_t*)(packed + L.p_w2);
    const hipError_t e = launch_invert_perm(L, perm, inv, &((PackRecord*)(packed + L.p_scale))->bad_perm, s);
    if (e != hipSuccess) return e;
  }
  auto aligned = [](const void* a, const void* b) { return (((uintptr_t)a | (uintptr_t)b) & 15) == 0; };
  auto w13 = [&](const void* a, const void* b, const int32_t* order, char* out, int experts, int Fs, int Fp, int P, int NT1, int per_expert) {
    const int vec = Fs % PackTile<T>::V == 0 && aligned(a, b);
    pack_w13_kernel<T, FULL><<<dim3((unsigned)((Fs + C - 1) / C * KS1), experts), block, 0, s>>>(
        (const T*)a, (const T*)b, order, out, L.D, KS1, Fs, Fp, P, NT1, per_expert ? 0 : Fs, per_expert, L.h_shift, vec);
    const int pad = NT1 * W13Image<T, FULL>::NEUR - Fp, groups = (per_expert ? experts : 1) * P;
    if (pad > 0) {
      const int64_t total = (int64_t)groups * KS1 * pad * 2 * PackTile<T>::CH;
      pack_w13_padding_kernel<T, FULL><<<dim3((unsigned)blocks_of_256(total)), block, 0, s>>>(out, groups, Fp, NT1, KS1);
    }
  };
  w13(w1, w3, inv, packed + L.p_w13, L.E_res, L.F, L.Fp, L.P, L.NT1, 1);
  if (n_shared > 0) w13(sw1, sw3, nullptr, packed + L.p_sw13, n_shared, F_sh, L.F_shT, 1, L.NT1_sh, 0);
  w2_images<T, FULL>(L, w2, sw2, perm, packed, s);
  return hipGetLastError();
}

hipError_t launch_pack(const Layout& L, const void* w1, const void* w3, const void* w2, const void* sw1, const void* sw3,
                       const void* sw2, const int32_t* perm, char* packed, int n_shared, int F_sh, hipStream_t s) {
  PackRecord* rec = (PackRecord*)(packed + L.p_scale);
  const hipError_t e = launch_fill_i32((int32_t*)rec, sizeof(PackRecord) / 4, 0, s);
  if (e != hipSuccess) return e;
  if (L.mfma) {
    const int64_t n = (int64_t)L.E_res * L.F * L.D, n_sh = (int64_t)L.F_shT * L.D;
    launch_absmax(w2, n, absmax_stride(n), rec, s);
    if (n_shared > 0) launch_absmax(sw2, n_sh, absmax_stride(n_sh), rec, s);
    return pack_images<uint16_t, false>(L, w1, w3, w2, sw1, sw3, sw2, perm, packed, n_shared, F_sh, s);
  }
  if (L.dtype == DSMOE_F32) return pack_images<float, true>(L, w1, w3, w2, sw1, sw3, sw2, perm, packed, n_shared, F_sh, s);
  return pack_images<uint16_t, true>(L, w1, w3, w2, sw1, sw3, sw2, perm, packed, n_shared, F_sh, s);
}

hipError_t launch_repack_w2(const Layout& L, const void* w2, const void* sw2, const int32_t* perm, char* packed, hipStream_t s) {
  PackRecord* rec = (PackRecord*)(packed + L.p_scale);
  launch_absmax(w2, (int64_t)L.E_res * L.F * L.D, 1, rec, s);
  if (L.n_shared > 0) launch_absmax(sw2, (int64_t)L.F_shT * L.D, 1, rec, s);
  w2_images<uint16_t, false>(L, w2, sw2, perm, packed, s);
  return hipGetLastError();
}

}  // namespace dsmoe
