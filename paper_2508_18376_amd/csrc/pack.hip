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
//        representable (smaller ones round to the subnormal grid, 2^-39 of it).  Column tiles of an expert with a larger
//        |W2| that no longer fits half precision are packed again with an s of their own.  GEMM-2 and the combine
//        kernel take the powers of two out again, exactly.  The record (PackRecord) sits at p_scale.
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
  const int64_t runs = (n + (int64_t)stride * kAbsmaxRun - 1) / ((int64_t)stride * kAbsmaxRun);
  absmax_bf16_kernel<<<dim3((unsigned)(runs < 512 ? runs : 512)), dim3(256), 0, s>>>((const uint16_t*)w, n, stride, &rec->largest);
}
// The scale is needed before the first value is packed, and finding the largest of all |W2| reads W2 once more (a tenth
// of the packing of 8 experts of 4096 x 14336, which takes 1.53 ms with it and 1.36 without).  A sample of 8 to 16 M values tells its
// binade as well as that binade and the next have room for (see repack_w2_kernel): only column tiles whose largest value is more than twice (for some, four
// times) the sample's largest are packed twice.  Odd strides: a row of a power of two of values is met in all of its columns.
static int absmax_stride(int64_t n) {
  const int64_t k = n >> 23;
  return k < 2 ? 1 : k > 63 ? 63 : (int)(k | 1);
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
// byte i becomes at least v (rarely called: for weights beyond the sample)
__device__ __forceinline__ void raise_byte(uint32_t* words, int i, uint32_t v) {
  uint32_t* at = words + (i >> 2);
  const int sh = 8 * (i & 3);
  uint32_t old = *(volatile uint32_t*)at;
  while ((old >> sh & 255) < v) {
    const uint32_t seen = atomicCAS(at, old, (old & ~(255u << sh)) | v << sh);
    if (seen == old) break;
    old = seen;
  }
}

// some of the eight bf16 values is infinite or NaN
__device__ __forceinline__ bool not_finite(uint4 v) {
  auto one = [](uint32_t u) { return (u & 0x7f80u) == 0x7f80u || (u & 0x7f800000u) == 0x7f800000u; };
  return one(v.x) || one(v.y) || one(v.z) || one(v.w);
}

// Neuron c of an expert is not the one that perm names at the position inv has for it, i.e. none names it (inv is whatever was
// there before): perm is no permutation.
__device__ __forceinline__ bool not_inverse(const int32_t* perm, int pos, int c, int F) { return (uint32_t)pos >= (uint32_t)F || perm[pos] != c; }

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
// The workgroups of the first K stage also check perm against inv, see not_inverse (a launch of its own for that is the seventh in front of
// the host's read of the outcome, and with seven that takes 27 us longer than with six).
// What is left to the 5.3 TB/s of a large copy are the 64-byte runs that a random order scatters.
template <typename T, bool FULL>
__global__ __launch_bounds__(256) void pack_w13_kernel(const T* w1, const T* w3, const int32_t* perm, const int32_t* inv, int32_t* bad, char* out, int D, int KS1,
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
      if (inv && (ks | lc) == 0 && not_inverse(perm + (size_t)e * Fs, pos, c, Fs)) *bad = 1;
      if (inv && (uint32_t)pos >= (uint32_t)Fs) continue;  // not a permutation (reported when all is done)
      const int p = pos / Fp, nin = pos - p * Fp;
      const int row = Im::row(nin);
      char* stage = out + ((((int64_t)e * per_expert * P + p) * NT1 + nin / Im::NEUR) * KS1 + ks) * Im::STAGE;
      *(uint4*)(stage + Im::at(row, lc)) = g[i];
      *(uint4*)(stage + Im::at(row + Im::UP, lc)) = u[i];
    }
  }
}

// W2 of the routed experts, or of the shared ones, and its images.  w2: [experts][F][D]; neurons of a partition; stages of a
// partition and of the expert; 16-byte loads are aligned.
template <typename T>
struct W2Tensor {
  const T* w2;
  const int32_t* perm;
  char* out;
  int F, Fp, KSp, KT, vec;
};
// One K stage of PackTile::COLS output columns from c0 on: 32 neuron positions (source rows, in permuted order; zeros past the end of a
// partition), one stage image, or two of 128 columns; nd: column tiles of the images.  op(v): eight (four) values as the images hold them.
template <typename T, bool FULL, class Op>
__device__ __forceinline__ void pack_w2_stage(PackTile<T>& t, const W2Tensor<T>& w, int D, int nd, int e, int kt, int c0, Op&& op) {
  using PT = PackTile<T>;
  constexpr int BN = FULL ? kFullBN2 : kMfmaBN2, RB = kBK * sizeof(T);
  const int tid = threadIdx.x;
  uint4 a[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int in = kt % w.KSp * kBK + u * 8 + (tid >> 5), pos = kt / w.KSp * w.Fp + in;
    const T* row = nullptr;
    if (in < w.Fp) {
      const int src = w.perm ? w.perm[(size_t)e * w.F + pos] : pos;
      if ((uint32_t)src < (uint32_t)w.F) row = w.w2 + ((size_t)e * w.F + src) * D;  // (not a permutation: reported when all is done)
    }
    a[u] = PT::template load<false>(row, c0 + (tid & 31) * PT::V, D, w.vec);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) t.put(u * 8 + (tid >> 5), tid & 31, op(a[u]));
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
      char* stage = w.out + (((int64_t)e * nd + jd) * w.KT + kt) * (BN * RB);
      *(uint4*)(stage + row * RB + swz_full<RB / 16>(row, lc) * 16) = o[i];
    }
  }
}
__device__ __forceinline__ uint4 scaled_halves(uint4 v, int shift) {
  const float scale = __uint_as_float((uint32_t)(127 + shift) << 23);
  return map_halves(v, [&](uint16_t b) { return (uint32_t)bf16_to_scaled_half(b, scale); });
}

// W2 -> W2 images (matrix-core path: half precision times the sample's power of two).  A workgroup takes one stage, see above.
// beyond: matrix-core path, the bytes of these experts' column tiles, see PackRecord
template <typename T, bool FULL>
__global__ __launch_bounds__(256) void pack_w2_kernel(W2Tensor<T> w, PackRecord* rec, int beyond0, int D, int nd) {
  using PT = PackTile<T>;
  static_assert(FULL || PT::COLS == kMfmaBN2, "one column tile");
  __shared__ PT t;
  const int nb = (D + PT::COLS - 1) / PT::COLS, jd = blockIdx.x % nb, e = blockIdx.y;
  const uint32_t sampled = FULL ? 0 : rec->largest;
  pack_w2_stage<T, FULL>(t, w, D, nd, e, blockIdx.x / nb, jd * PT::COLS, [&](uint4 v) {
    if constexpr (FULL) {
      if (sizeof(T) == 2 && not_finite(v)) rec->largest = 1;
      return v;
    } else {
      if (const uint32_t most = beyond_sample(v, sampled)) raise_byte((uint32_t*)(rec + 1), beyond0 + e * nd + jd, most >> 7);
      return scaled_halves(v, w2_shift(sampled >> 7));
    }
  });
}

// Once all of W2 has been looked at: the powers of two of the record, and the column tiles whose largest weight does not fit at the
// sample's scale once more with their own.  Outliers are few, and so are those tiles: loading 8 experts of 4096 x 14336 (128 column
// tiles) takes 1.36 ms, with a weight far beyond the others in 1 / 4 / 16 / 64 places that the sample misses 1.37 / 1.38 / 1.41 / 1.51
// (all of W2 again from its largest, which the host asked for when it had seen the record: 1.92 for any of them; the largest of all
// found first: 1.53 always); 64 experts of 2048 x 1024 0.39, with 1 or 4 of them 0.40 (0.57; 0.47).
// n: words of four column tiles.  (Every workgroup has an order of its own in todo: its stages of a tile do not follow from it.)
constexpr int kRepackBlocks = 1024;
__global__ __launch_bounds__(256) void repack_w2_kernel(W2Tensor<uint16_t> routed, W2Tensor<uint16_t> shared, PackRecord* rec, int n, int E_res, int D, int nd,
                                                        int h_shift) {
  __shared__ PackTile<uint16_t> t;
  __shared__ uint32_t todo[1024];  // column tile << 8 | exponent
  __shared__ int count, top;
  const int blocks = gridDim.x, tid = threadIdx.x;
  const bool usable = rec->largest >= 0x80u;
  const int sampled = w2_shift(rec->largest >> 7), room = usable ? 142 - sampled : 0;
  if (tid == 0) top = 0;
  for (int base = 0; base < n; base += 256) {
    if (tid == 0) count = 0;
    __syncthreads();
    const uint32_t word = base + tid < n ? ((const uint32_t*)(rec + 1))[base + tid] : 0;
    for (int i = 0; i < 4; ++i) {
      const int b = word >> (8 * i) & 255;
      if (b) atomicMax(&top, b);
      if (b > room) todo[atomicAdd(&count, 1)] = (uint32_t)((base + tid) * 4 + i) << 8 | b;
    }
    __syncthreads();
    for (int i = 0; i < count; ++i) {
      const int tile = todo[i] >> 8, shift = w2_shift(todo[i] & 255), e = tile / nd;
      const W2Tensor<uint16_t>& w = e < E_res ? routed : shared;
      for (int kt = (blockIdx.x + tile * 97) % blocks; kt < w.KT; kt += blocks) {
        __syncthreads();
        pack_w2_stage<uint16_t, false>(t, w, D, nd, e < E_res ? e : 0, kt, tile % nd * kMfmaBN2, [&](uint4 v) { return scaled_halves(v, shift); });
      }
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && tid == 0) {
    const int shift = top ? w2_shift(top) : sampled;
    rec->room = room;
    rec->shift0 = usable ? sampled : shift;  // (column tiles of zeros and subnormals alone: zeros at any scale)
    rec->shift = shift;
    rec->beyond = top;
    rec->unscale = ldexpf(1.f, -shift - h_shift);  // undoes 2^shift of the partial outputs and 2^h_shift of W3
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

// inv[e][perm[e][pos]] = pos; *bad, which what follows may set, is cleared
__global__ void invert_perm_kernel(const int32_t* perm, int32_t* inv, int F, int64_t n, int32_t* bad) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  if (t == 0) *bad = 0;
  const int64_t e = t / F;
  const int src = perm[t];
  if (src >= 0 && src < F) inv[e * F + src] = (int32_t)(t % F);
}
__global__ void perm_check_kernel(const int32_t* perm, const int32_t* inv, int F, int64_t n, int32_t* bad) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int64_t e = t / F;
  const int pos = inv[t];
  if (not_inverse(perm + e * F, pos, (int)(t % F), F)) *bad = 1;
}
static dim3 perm_grid(const Layout& L) { return dim3((unsigned)(((int64_t)L.E_res * L.F + 255) / 256)); }
hipError_t launch_invert_perm(const Layout& L, const int32_t* perm, int32_t* inv, int32_t* bad, hipStream_t s) {
  const int64_t n = (int64_t)L.E_res * L.F;
  invert_perm_kernel<<<perm_grid(L), dim3(256), 0, s>>>(perm, inv, L.F, n, bad);
  perm_check_kernel<<<perm_grid(L), dim3(256), 0, s>>>(perm, inv, L.F, n, bad);
  return hipGetLastError();
}

template <typename T, bool FULL>
static void w2_images(const Layout& L, const void* w2, const void* sw2, const int32_t* perm, char* packed, hipStream_t s) {
  PackRecord* rec = (PackRecord*)(packed + L.p_scale);
  auto tensor = [&](const void* w, const int32_t* order, int64_t out, int F, int Fp, int Fpk) {
    const int KSp = Fpk / kBK;
    return W2Tensor<T>{(const T*)w, order, packed + out, F, Fp, KSp, Fp ? F / Fp * KSp : 0, L.D % PackTile<T>::V == 0 && ((uintptr_t)w & 15) == 0};
  };
  const W2Tensor<T> routed = tensor(w2, perm, L.p_w2, L.F, L.Fp, L.Fpk), shared = tensor(sw2, nullptr, L.p_sw2, L.F_shT, L.F_shT, L.Fsk);
  auto images = [&](const W2Tensor<T>& w, int experts, int beyond0) {
    const int C = PackTile<T>::COLS;
    pack_w2_kernel<T, FULL><<<dim3((unsigned)((L.D + C - 1) / C * w.KT), experts), dim3(256), 0, s>>>(w, rec, beyond0, L.D, L.ND2);
  };
  images(routed, L.E_res, 0);
  if (L.n_shared > 0) images(shared, 1, L.E_res * L.ND2);
  if constexpr (!FULL) {
    const int words = (w2_tiles(L) + 3) / 4;
    repack_w2_kernel<<<dim3(kRepackBlocks), dim3(256), 0, s>>>(routed, shared, rec, words, L.E_res, L.D, L.ND2, L.h_shift);
  }
}

template <typename T, bool FULL>
static hipError_t pack_images(const Layout& L, const void* w1, const void* w3, const void* w2, const void* sw1, const void* sw3, const void* sw2,
                              const int32_t* perm, char* packed, int n_shared, int F_sh, hipStream_t s) {
  const dim3 block(256);
  const int KS1 = L.Dk / kBK, C = PackTile<T>::COLS;
  // The W1 / W3 stages are written from source columns (see pack_w13_kernel), which needs the inverse
  // permutation: it is parked in the W2 region of the packed buffer, which the W2 kernel overwrites.
  // (That region has at least E_res * F * 32 * sizeof(T) bytes, the table E_res * F * 4.)
  int32_t *inv = nullptr, *bad = &((PackRecord*)(packed + L.p_scale))->bad_perm;
  if (perm) {
    inv = (int32_t*)(packed + L.p_w2);
    invert_perm_kernel<<<perm_grid(L), block, 0, s>>>(perm, inv, L.F, (int64_t)L.E_res * L.F, bad);
  }
  auto aligned = [](const void* a, const void* b) { return (((uintptr_t)a | (uintptr_t)b) & 15) == 0; };
  auto w13 = [&](const void* a, const void* b, const int32_t* order, char* out, int experts, int Fs, int Fp, int P, int NT1, int per_expert) {
    const int vec = Fs % PackTile<T>::V == 0 && aligned(a, b);
    pack_w13_kernel<T, FULL><<<dim3((unsigned)((Fs + C - 1) / C * KS1), experts), block, 0, s>>>(
        (const T*)a, (const T*)b, perm, order, bad, out, L.D, KS1, Fs, Fp, P, NT1, per_expert ? 0 : Fs, per_expert, L.h_shift, vec);
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
  const hipError_t e = launch_fill_i32((int32_t*)rec, sizeof(PackRecord) / 4 + (L.mfma ? (w2_tiles(L) + 3) / 4 : 0), 0, s);
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

}  // namespace dsmoe
