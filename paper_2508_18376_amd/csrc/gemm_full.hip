// Full-precision grouped GEMMs on the matrix cores: fp32 layers, and bf16 layers that the half-precision path of
// gemm_mfma.hip does not take (widths that are no multiple of 32, batches of 2 GiB and more).  The intermediate
// activation H and the per-pair partial outputs are fp32 here whatever the layer's type:
//   GEMM-1  H[row][p*Fpk + j] = Swish(x_row . W1[:, j]) * (x_row . W3[:, j])      (Eq. 4, gate/up)
//   GEMM-2  Yp[row][d] = sum over kept partitions p, neurons j of H[row][p*Fpk + j] * W2[p*Fpk + j][d]
// Same work lists and row lists as the other path, with tiles of 64 rows (up to 128 where an item takes the expert's
// short last tile along) x 64 neurons, resp. x 128 output columns: a weight image of 128 rows (see pack.hip); in large batches of
// bf16 layers of many experts two images (full_wide).
//
// Matrix instructions: fp32 layers multiply with v_mfma_f32_16x16x4_f32 (the precision of an fmaf chain, 256 flop
// per clock and compute unit, the chip's fp32 peak of ~155 TFLOP/s; without packed fp32 the vector units reach
// half of that).  bf16 layers multiply x with W1 / W3 by v_mfma_f32_32x32x16_bf16 (exact products); for GEMM-2 the fp32
// activation is cut into three bf16 values h = hi + mid + lo (8 + 8 + 8 significant bits: exact from |h| = 2^-110 on, below that
// to within bf16's smallest value, 2^-133) and multiplied with the bf16 weights in three such instructions, which keeps all 24
// bits of H at 5 x the rate of the fp32 instruction.  mid and lo can be zero: layers with an infinity or NaN in W2 (the packed
// weights say so) leave those weights out of the two smaller products.
//
// Tiles of two images (bf16 layers) read the pair rows and cut fp32 activations half as often; the sums are the same bit for bit (K splits apart).  There
// GEMM-1 notes whether an activation came out infinite or NaN (kNonfiniteH), and GEMM-2 of other batches does without the clamp: 777 tokens on 64 + 2
// experts of 2048 x 1408 in parts of 176 408 -> 397 us; with an infinite token or infinities in W2 427 (single images 431 and 453).
// fp32 layers keep single images and the fp32 instruction: six products of bf16 parts of both operands are 2.7 x as fast (512 tokens on 64 experts of
// 2048 x 1024 559 -> 503 us), but they leave products of up to 2^-21 out and the bf16 instruction cuts its sums off towards zero, so that sums
// carried by one term are less exact than fp32 (2.6e-8 -> 6.5e-8), as are products of values below 2^-110.
//
// A workgroup is 4 wavefronts; wavefront w owns the weight rows 32 w .. 32 w + 31 of the tile's 128 and multiplies them
// with all pair rows, so a tile of r rows costs ceil(r/32) blocks (fp32: ceil(r/16) of half the size).  The 32 weight rows of a GEMM-1 wavefront are the gate
// and the up projection of the same 16 neurons, which meet in one lane.  64 rows against 128 weight rows are 2048 matrix
// cycles for 24 KiB of operands in fp32 (12 bytes per clock: well below what L2 and HBM deliver), so for fp32 the
// tile does not have to be larger; with few rows the kernels stream weights.  Operands travel HBM/L2 -> LDS by 16-byte
// direct-to-LDS loads through a ring of 80 KiB (2 to 6 stages of 32 K values, by the height of the tile): two workgroups
// per compute unit, so that one streams while the other starts or ends an item.
//
// Measured, before (vector FMAs on 64 x 64 tiles with guarded loads) -> now:
//   fp32, 64 experts of 2048 x 1024, 512 tokens top-8, 25 % dropped: GEMM-1 1250 -> 375 us (2.9 TB/s of weights), GEMM-2 545 -> 189 us
//   bf16, 64 + 2 shared experts of 2048 x 1408 in parts of 176, 777 tokens top-6: GEMM-1 2309 -> 208 us (4 TB/s), GEMM-2 1041 -> 224 us
//   fp32, 8 experts of 128 x 256, 64 tokens: GEMM-1 27 -> 6 us, GEMM-2 33 -> 4 us (K split over several workgroups)
// and with tiles of two images, the whole layer: 777 tokens of the second 431 -> 399 (GEMM-2 224 -> 160).
#include <type_traits>

#include "common.h"

namespace dsmoe {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kFullLds = 80 * 1024;  // two workgroups per compute unit

// 16 bytes per lane from a 64-bit address into LDS at (lds_addr + lane * 16), lds_addr wave-uniform
// ONCE: the non-temporal hint (see gemm_mfma.hip)
template <bool ONCE = false>
__device__ __forceinline__ void dma16g(const char* src, uint32_t lds_addr) {
#define DSMOE_DMA16G(POLICY)                 \
  asm volatile(                              \
      "s_mov_b32 m0, %0\n\t"                 \
      "s_nop 0\n\t"                          \
      "global_load_lds_dwordx4 %1, off" POLICY \
      :                                      \
      : "s"(lds_addr), "v"(src)              \
      : "memory")
  if (ONCE) DSMOE_DMA16G(" nt");
  else DSMOE_DMA16G("");
#undef DSMOE_DMA16G
}
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Barrier behind which a stage may be overwritten: this wavefront's LDS reads have arrived.
__device__ __forceinline__ void read_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ uint32_t lds_byte(const char* p) {
  return (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const char*)p);
}

// eight fp32 values as sums of three bf16 values each: the top 16 bits, the top 16 bits of the (exact) rest, the rest
// CLAMP: an infinite value leaves NaN as the rest: it is clamped (no finite value has a rest beyond 2^120), so that the first part decides
template <bool CLAMP>
__device__ __forceinline__ void split3(const f32x4& v0, const f32x4& v1, u32x4 (&part)[3]) {
  float r[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      part[k][i] = __builtin_amdgcn_perm(__float_as_uint(r[2 * i + 1]), __float_as_uint(r[2 * i]), 0x07060302);
    if (k < 2) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        r[i] -= __uint_as_float(__float_as_uint(r[i]) & 0xffff0000u);
        if (CLAMP && k == 0) r[i] = __builtin_amdgcn_fmed3f(r[i], -1.4e36f, 1.4e36f);
      }
    }
  }
}

// eight weights with zeros in place of infinities and NaN
__device__ __forceinline__ bf16x8 finite_only(const bf16x8& a) {
  u32x4 v = __builtin_bit_cast(u32x4, a);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if ((v[i] & 0x7f80u) == 0x7f80u) v[i] &= 0xffff0000u;
    if ((v[i] & 0x7f800000u) == 0x7f800000u) v[i] &= 0xffffu;
  }
  return __builtin_bit_cast(bf16x8, v);
}

// One tile product: 128 / SUBS weight rows (WE bytes per value) x NJ blocks of BR pair rows (XE bytes per value), K stages of 32.
// fp32 weights: blocks of 16 rows (v_mfma_f32_16x16x4_f32, the rate of the 32-row instruction): an expert's few rows are
// padded half as far (with blocks of 32: 512 tokens top-8 on 64 experts of 2048 x 1024, 48 rows an expert, 522 -> 472 us for the layer, 300 tokens 415 -> 360;
// 144 tokens, 14 rows, where weights only stream, 310 -> 315).
// The sums of fp32 products are kept apart for the two halves of every stage's K values and added at the end: half as long chains of roundings
// (2048 x 1024, 2 experts of 8 per token: 1.27e-6 -> 0.88e-6 off the 64-bit result).
// SUBS = 2: two wavefronts share 32 weight rows.  fp32: each multiplies 16 of them, so that the sums are those of a whole tile bit for bit; bf16: each
// multiplies one half of every stage's K values, and the sums meet in the first one (w < 2) at the end.
// NONFINITE (bf16 weights x fp32 activations): some weights are infinite or NaN, see above
template <int WE, int XE, int NJ, int SUBS, bool NONFINITE = false>
struct FullTile {
  static constexpr int WR = kBK * WE, XR = kBK * XE;           // bytes of a tile row
  static constexpr int WCH = WR / 16, XCH = XR / 16;           // 16-byte chunks of a row
  static constexpr int WROWS = 128 / SUBS;
  static constexpr int NW = WROWS * WR / 4096;                 // 4 KiB loads of the weight tile per stage
  static constexpr int BR = WE == 4 ? 16 : 32;                 // pair rows of a block
  static constexpr int XROWS_LOAD = 256 / XCH;                 // rows per load
  static constexpr int NX = (NJ * BR + XROWS_LOAD - 1) / XROWS_LOAD;
  static constexpr int NL = NW + NX;
  static constexpr int SB = NL * 4096;                         // bytes of a stage
  static constexpr int NS = kFullLds / SB < 6 ? kFullLds / SB : 6;
  static_assert(NS >= 2 && (NS - 2) * NL < 64, "ring");

  static constexpr bool SPLIT = WE == 4 && SUBS == 2;  // two wavefronts, 16 weight rows each
  static constexpr int NI = SPLIT ? 1 : 2;             // fp32: blocks of 16 weight rows of a wavefront
  static constexpr int NQ = WE == 4 ? NI : 4;          // groups of four accumulators per block and lane
  f32x4 acc4[WE == 4 ? NJ : 1][2];                     // fp32: of the first half of every stage, in the end of both (SPLIT: [1] is only used by other_rows)
  f32x4 acc4b[WE == 4 ? NJ : 1][NI];                   // of the second half
  f32x16 acc[WE == 4 ? 1 : NJ];

  // the 32 weight rows that a wavefront works on
  static __device__ __forceinline__ int rows32(int w) { return SPLIT ? w >> 1 : w % (4 / SUBS); }
  // Group q of block j: four consecutive weight rows of these 32, the first of them w_row(q) (SPLIT: + 16 in odd wavefronts), times pair row x_row(j).
  __device__ __forceinline__ f32x4 group(int j, int q) const {
    if constexpr (WE == 4) return acc4[j][q];
    else return f32x4{acc[j][q * 4], acc[j][q * 4 + 1], acc[j][q * 4 + 2], acc[j][q * 4 + 3]};
  }
  static __device__ __forceinline__ int w_row(int q, int lane) { return WE == 4 ? q * 16 + (lane >> 4) * 4 : q * 8 + (lane >> 5) * 4; }
  static __device__ __forceinline__ int x_row(int j, int lane) { return j * BR + (lane & (BR - 1)); }

  // rowp[i]: where this thread's chunk of its i-th row starts (K position 0); wsrc: this thread's chunk of the first weight
  // stage; next(st): byte offset of stage st in a pair row and in the weight stages, called once per stage in order
  template <class Next>
  __device__ __forceinline__ void run(int n, const char* const (&rowp)[NX], const char* wsrc, Next&& next, const char* lds, int w, int lane) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if constexpr (WE == 4)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc4[j][i] = acc4b[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      else
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    }
    const uint32_t base = lds_byte(lds) + (uint32_t)w * 1024;
    auto issue = [&](int st) {
      int64_t xo, wo;
      next(xo, wo);
      const uint32_t slot = base + (uint32_t)(st % NS) * SB;
#pragma unroll
      for (int q = 0; q < NW; ++q) dma16g(wsrc + wo + q * 4096, slot + q * 4096);
#pragma unroll
      for (int q = 0; q < NX; ++q) dma16g(rowp[q] + xo, slot + (NW + q) * 4096);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < n) issue(s);
    int st = 0;
    for (; st + NS - 1 < n; ++st) {
      wait_loads<(NS - 2) * NL>();  // stage st has landed (for this wavefront; the barrier makes it so for all)
      read_barrier();
      issue(st + NS - 1);           // into the slot of stage st - 1, which every wavefront has finished reading
      multiply(lds + (st % NS) * SB, w, lane);
    }
    for (; st < n; ++st) {
      const int left = n - 1 - st;  // later stages still in flight
      if (NS > 2 && left >= NS - 2) wait_loads<(NS - 2) * NL>();
      else if (NS > 3 && left == NS - 3) wait_loads<(NS > 3 ? NS - 3 : 0) * NL>();
      else if (NS > 4 && left == NS - 4) wait_loads<(NS > 4 ? NS - 4 : 0) * NL>();
      else if (NS > 5 && left == NS - 5) wait_loads<(NS > 5 ? NS - 5 : 0) * NL>();
      else wait_loads<0>();
      read_barrier();
      multiply(lds + (st % NS) * SB, w, lane);
    }
    if constexpr (WE == 4) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc4[j][i] += acc4b[j][i];
    }
    if constexpr (SUBS == 2 && !SPLIT) {
      read_barrier();  // every wavefront is done reading the last stage
      f32x4* part = (f32x4*)const_cast<char*>(lds) + (w & 1) * (NJ * NQ * 64) + lane;  // [NQ NJ][64 lanes]
      if (w >= 2) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int q = 0; q < NQ; ++q) part[(j * NQ + q) * 64] = group(j, q);
      }
      __syncthreads();
      if (w < 2) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            const f32x4 o = part[(j * NQ + q) * 64];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[j][q * 4 + c] += o[c];
          }
      }
    }
  }

  // SPLIT: the odd wavefronts' sums go to the even ones, as group 1
  __device__ __forceinline__ void other_rows(const char* lds, int w, int lane) {
    read_barrier();  // every wavefront is done reading the last stage
    f32x4* part = (f32x4*)const_cast<char*>(lds) + (w >> 1) * (NJ * 64) + lane;  // [NJ][64 lanes]
    if (w & 1)
#pragma unroll
      for (int j = 0; j < NJ; ++j) part[j * 64] = acc4[j][0];
    __syncthreads();
    if (!(w & 1))
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc4[j][1] = part[j * 64];
  }

  __device__ __forceinline__ void multiply(const char* stage, int w, int lane) {
    const int r32 = lane & 31, h = lane >> 5;
    const int k0 = SUBS == 2 ? w >> 1 : 0;  // bf16: this wavefront's half of the stage
    const char* wrow = stage + (rows32(w) * 32 + r32) * WR;
    const char* xrow = stage + NW * 4096 + r32 * XR;
    if constexpr (WE == 4) {  // fp32 x fp32: chunk 4s + h of a row holds K values 16s + 4h .. 16s + 4h + 3; instruction i takes every lane's i-th
      const int r16 = lane & 15, h16 = lane >> 4;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int at = swz_full<WCH>(r16, 4 * s + h16) * 16;  // (rows 16 apart have the same rotation)
        f32x4 a[NI], b[NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) a[i] = *(const f32x4*)(stage + (rows32(w) * 32 + (SPLIT ? (w & 1) * 16 : i * 16) + r16) * WR + at);
#pragma unroll
        for (int j = 0; j < NJ; ++j) b[j] = *(const f32x4*)(stage + NW * 4096 + (j * 16 + r16) * XR + at);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
              f32x4& c = s == 0 ? acc4[j][i] : acc4b[j][i];
              c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][k], b[j][k], c, 0, 0, 0);
            }
      }
    } else if constexpr (XE == 2) {  // bf16 x bf16: K values 16s + 8h .. 16s + 8h + 7
#pragma unroll
      for (int s0 = 0; s0 < 2 / SUBS; ++s0) {
        const int s = s0 + k0;
        const bf16x8 a = *(const bf16x8*)(wrow + swz_full<WCH>(r32, 2 * s + h) * 16);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bf16x8 b = *(const bf16x8*)(xrow + j * 32 * XR + swz_full<XCH>(r32, 2 * s + h) * 16);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[j], 0, 0, 0);
        }
      }
    } else {  // bf16 weights x fp32 activations
#pragma unroll
      for (int s0 = 0; s0 < 2 / SUBS; ++s0) {
        const int s = s0 + k0;
        const bf16x8 a = *(const bf16x8*)(wrow + swz_full<WCH>(r32, 2 * s + h) * 16);
        const bf16x8 small = NONFINITE ? finite_only(a) : a;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const char* x = xrow + j * 32 * XR;
          const f32x4 v0 = *(const f32x4*)(x + swz_full<XCH>(r32, 4 * s + 2 * h) * 16);
          const f32x4 v1 = *(const f32x4*)(x + swz_full<XCH>(r32, 4 * s + 2 * h + 1) * 16);
          u32x4 part[3];
          split3<true>(v0, v1, part);
#pragma unroll
          for (int k = 2; k >= 0; --k)  // the small parts first
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k == 0 ? a : small, __builtin_bit_cast(bf16x8, part[k]), acc[j], 0, 0, 0);
        }
      }
    }
  }
};

// The pieces of a list: whole items, the last kFullHalved as two halves of their weight tile (tiles of two images: an image each).
constexpr int kFullHalved = 256;
struct FullPiece {
  int item, half;  // half -1: the whole item
};
__device__ __forceinline__ int full_pieces(int items) { return items + min(items, kFullHalved); }
__device__ __forceinline__ FullPiece full_piece(int items, int id) {
  const int whole = max(items - kFullHalved, 0), cut = id - whole;
  return cut < 0 ? FullPiece{id, -1} : FullPiece{whole + (cut >> 1), cut & 1};
}

// ------------------------------------------------------------------------------------- GEMM-1
template <typename T, int NJ, int SUBS>
__device__ __forceinline__ void gemm1_full_tile(const Layout& L, const Item1& it, int sub, const char* packed, const char* x, int64_t x_row, char* ws,
                                                int epi, char* lds, int w, int lane) {
  constexpr int E = sizeof(T);
  using Tile = FullTile<E, E, NJ, SUBS>;
  const int tid = w * 64 + lane;
  const bool sh = it.e == L.E_res;
  const int Fpk = sh ? L.Fsk : L.Fpk, ld = sh ? L.Fsk : L.Fh, NI1 = sh ? L.NI1_sh : L.NI1;
  const int KS = L.Dk / kBK;
  const int32_t* row_token = (const int32_t*)(ws + L.o_row_token) + it.row0;
  const uint8_t* row_bits = (const uint8_t*)(ws + L.o_row_bits) + it.row0;
  const char* wsrc = packed + (sh ? L.p_sw13 : L.p_w13) + (((int64_t)(sh ? 0 : it.e * L.P + it.p) * NI1 + it.jt) * KS) * (128 * Tile::WR) + sub * (Tile::WROWS * Tile::WR) + tid * 16;
  const char* rowp[Tile::NX];
#pragma unroll
  for (int i = 0; i < Tile::NX; ++i) {
    const int r = i * Tile::XROWS_LOAD + tid / Tile::XCH;
    const int rr = r < it.nrows ? r : it.nrows - 1;  // rows past the end re-read the last one
    rowp[i] = x + (int64_t)row_token[rr] * x_row + swz_full<Tile::XCH>(r, tid % Tile::XCH) * 16;
  }
  Tile t;
  int64_t k = 0;
  t.run(KS, rowp, wsrc, [&](int64_t& xo, int64_t& wo) {
    xo = k * Tile::XR;
    wo = k * (128 * Tile::WR);
    ++k;
  }, lds, w, lane);
  // the wavefront's 32 weight rows are 16 gate rows, then the 16 up rows of the same neurons
  float* H = (float*)(ws + (sh ? L.o_Hs : L.o_H)) + (size_t)(sh ? it.row0 : it.row0 - L.sh_rows) * ld + (size_t)it.p * Fpk;
  if constexpr (Tile::SPLIT) t.other_rows(lds, w, lane);
  if (Tile::SPLIT ? w & 1 : SUBS == 2 && w >= 2) return;
  const int n_tile = it.jt * kFullNeur + sub * (kFullNeur / SUBS) + Tile::rows32(w) * 16;
  constexpr int NG = sizeof(T) == 4 ? 1 : 2;  // groups of gate rows, and of up rows

  // the neurons that pad a partition to whole stages are zeros whatever came out: zero weights times an infinite x are NaN
  const int Fp = sh ? L.F_shT : L.Fp;
  float z = 0.f;  // stays zero as long as every activation is finite
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int r = Tile::x_row(j, lane);
    if (r >= it.nfill) continue;
    const bool kept = r < it.nrows && ((row_bits[r] >> it.p) & 1);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const f32x4 gate = t.group(j, q), up = t.group(j, NG + q);
      const int n = n_tile + Tile::w_row(q, lane);
      f32x4 o;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        o[c] = kept && n + c < Fp ? epi_value<false>(epi, gate[c], up[c]) : 0.f;
        z = __builtin_fmaf(o[c], 0.f, z);
      }
      if (n < Fpk) *(f32x4*)(H + (size_t)r * ld + n) = o;
    }
  }
  if (sizeof(T) == 2 && SUBS == 1 && L.wide && z != 0.f) ((int32_t*)(ws + L.o_counters))[kNonfiniteH] = 1;  // (true for NaN)
  for (int r = Tile::x_row(NJ, lane); r < it.nfill; r += Tile::BR) {  // rows that keep nothing of this partition, beyond the blocks multiplied: zeros
    for (int q = 0; q < NG; ++q) {
      const int n = n_tile + Tile::w_row(q, lane);
      if (n < Fpk) *(f32x4*)(H + (size_t)r * ld + n) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
}

// f(blocks) with the number of blocks of pair rows (see FullTile) as a compile-time constant
template <typename T, class F>
__device__ __forceinline__ void with_blocks(int nrows, F&& f) {
  if constexpr (sizeof(T) == 4) {
    switch ((nrows + 15) >> 4) {
      case 1: f(std::integral_constant<int, 1>()); break;
      case 2: f(std::integral_constant<int, 2>()); break;
      case 3: f(std::integral_constant<int, 3>()); break;
      case 4: f(std::integral_constant<int, 4>()); break;
      case 5: f(std::integral_constant<int, 5>()); break;
      case 6: f(std::integral_constant<int, 6>()); break;
      case 7: f(std::integral_constant<int, 7>()); break;
      default: f(std::integral_constant<int, 8>()); break;
    }
  } else {
    switch ((nrows + 31) >> 5) {
      case 1: f(std::integral_constant<int, 1>()); break;
      case 2: f(std::integral_constant<int, 2>()); break;
      case 3: f(std::integral_constant<int, 3>()); break;
      default: f(std::integral_constant<int, 4>()); break;
    }
  }
}

// SUBS: 2: all items in two halves; 1: none; 0: the last ones of the list (see full_parts)
template <int SUBS>
__device__ __forceinline__ int pieces_of(int items) { return SUBS == 2 ? items * 2 : SUBS == 0 ? full_pieces(items) : items; }
template <int SUBS>
__device__ __forceinline__ FullPiece piece_of(int items, int id) {
  return SUBS == 2 ? FullPiece{id >> 1, id & 1} : SUBS == 0 ? full_piece(items, id) : FullPiece{id, -1};
}
template <typename T, int SUBS>
__global__ __launch_bounds__(256, 2) void gemm1_full_kernel(Layout L, const char* packed, const char* x, int64_t x_row, char* ws, int epi) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int32_t* counters = (int32_t*)(ws + L.o_counters);
  const int items = counters[0], n = pieces_of<SUBS>(items), id = take_piece<true>(n, counters + 8, lds);
  if (id >= n) return;
  const FullPiece piece = piece_of<SUBS>(items, id);
  const Item1 it = ((const Item1*)(ws + L.o_items1))[piece.item];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  with_blocks<T>(it.nrows, [&](auto blocks) {
    constexpr int N = decltype(blocks)::value;
    if (SUBS != 1 && piece.half >= 0) gemm1_full_tile<T, N, 2>(L, it, piece.half, packed, x, x_row, ws, epi, lds, w, lane);
    else if constexpr (SUBS != 2) gemm1_full_tile<T, N, 1>(L, it, 0, packed, x, x_row, ws, epi, lds, w, lane);
  });
}

// ------------------------------------------------------------------------------------- GEMM-2
template <typename T, int NJ, int SUBS, bool NONFINITE>
__device__ __forceinline__ void gemm2_full_tile(const Layout& L, const Item2& it, int sub, const char* packed, char* ws, char* lds, int w, int lane) {
  constexpr int E = sizeof(T);
  using Tile = FullTile<E, 4, NJ, SUBS, NONFINITE>;
  const int tid = w * 64 + lane;
  const bool sh = it.e == L.E_res;
  const int ld = sh ? L.Fsk : L.Fh;
  const int KSp = (sh ? L.Fsk : L.Fpk) / kBK, np = sh ? 1 : L.P;  // stages of one partition, partitions
  const float* H = (const float*)(ws + (sh ? L.o_Hs : L.o_H)) + (size_t)(sh ? it.row0 : it.row0 - L.sh_rows) * ld;
  const char* wsrc = packed + (sh ? L.p_sw2 : L.p_w2) + ((int64_t)(sh ? 0 : it.e) * L.NI2 + it.jd) * (np * KSp) * (128 * Tile::WR) + sub * (Tile::WROWS * Tile::WR) + tid * 16;
  const char* rowp[Tile::NX];
#pragma unroll
  for (int i = 0; i < Tile::NX; ++i) {
    const int r = i * Tile::XROWS_LOAD + tid / Tile::XCH;
    const int rr = r < it.nrows ? r : it.nrows - 1;
    rowp[i] = (const char*)(H + (size_t)rr * ld) + swz_full<Tile::XCH>(r, tid % Tile::XCH) * 16;
  }
  // stages run over the partitions that some row of the tile keeps (Sec. 4: dropped units cost nothing)
  int n = 0;
  for (int p = 0; p < np; ++p) n += ((it.kmask >> p) & 1) ? it.ks_n : 0;
  int p_cur = 0, k_in = 0;
  while (p_cur < np && !((it.kmask >> p_cur) & 1)) ++p_cur;
  Tile t;
  t.run(n, rowp, wsrc, [&](int64_t& xo, int64_t& wo) {
    const int64_t kt = p_cur * KSp + it.ks_lo + k_in;
    if (++k_in == it.ks_n) {
      k_in = 0;
      ++p_cur;
      while (p_cur < np && !((it.kmask >> p_cur) & 1)) ++p_cur;
    }
    xo = kt * Tile::XR;
    wo = kt * (128 * Tile::WR);
  }, lds, w, lane);
  float* Y;
  int ldy;
  if (it.split == 0) {  // the item's rows of Yp
    Y = (float*)(ws + L.o_Yp) + (size_t)it.row0 * L.D + it.jd * kFullBN2;
    ldy = L.D;
  } else {              // an extra K range of a split item: a partial-output tile of the pool
    Y = (float*)(ws + L.o_pool) + (size_t)(it.split - 1) * L.pool_rows * L.BN2 + (L.wide ? (it.jd & 1) * kFullBN2 : 0);
    ldy = L.BN2;
  }
  if (!Tile::SPLIT && SUBS == 2 && w >= 2) return;
  const int c0 = sub * (kFullBN2 / SUBS) + Tile::rows32(w) * 32 + (Tile::SPLIT ? (w & 1) * 16 : 0), d0 = it.jd * kFullBN2;
  const bool vec = (L.D & 3) == 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int r = Tile::x_row(j, lane);
    if (r >= it.nrows) continue;
#pragma unroll
    for (int q = 0; q < Tile::NQ; ++q) {
      const int c = c0 + Tile::w_row(q, lane);
      const f32x4 o = t.group(j, q);
      float* at = Y + (size_t)r * ldy + c;
      if (vec) {
        if (d0 + c < L.D) *(f32x4*)at = o;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (d0 + c + i < L.D) at[i] = o[i];
      }
    }
  }
}

template <typename T, int SUBS>
__global__ __launch_bounds__(256, 2) void gemm2_full_kernel(Layout L, const char* packed, char* ws) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int32_t* counters = (int32_t*)(ws + L.o_counters);
  const int items = counters[1], n = pieces_of<SUBS>(items), id = take_piece<true>(n, counters + 9, lds);
  if (id >= n) return;
  const FullPiece piece = piece_of<SUBS>(items, id);
  const Item2 it = ((const Item2*)(ws + L.o_items2))[piece.item];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto run = [&](auto nonfinite) {
    with_blocks<T>(it.nrows, [&](auto blocks) {
      constexpr int N = decltype(blocks)::value;
      constexpr bool NONFINITE = sizeof(T) == 2 && decltype(nonfinite)::value;
      if (SUBS != 1 && piece.half >= 0) gemm2_full_tile<T, N, 2, NONFINITE>(L, it, piece.half, packed, ws, lds, w, lane);
      else if constexpr (SUBS != 2) gemm2_full_tile<T, N, 1, NONFINITE>(L, it, 0, packed, ws, lds, w, lane);
    });
  };
  if (sizeof(T) == 2 && ((const PackRecord*)(packed + L.p_scale))->largest) run(std::integral_constant<bool, sizeof(T) == 2>());
  else run(std::false_type());
}

// ------------------------------------------------------------------------------------- two images to a tile
// The product of both images of a tile (2 x 128 weight rows, bf16) with NJ blocks of 32 pair rows (XE bytes per value), K stages of 32.
template <int XE, int NJ>
struct WideTile {
  static constexpr int XR = kBK * XE, XCH = XR / 16;           // bytes of a pair row in a stage, 16-byte chunks of it
  static constexpr int WR = kBK * 2;                           // bytes of a weight row in a stage
  static constexpr int IMG = 128 * WR;                         // bytes of a stage of an image
  static constexpr int NW = 2 * IMG / 4096;                    // 4 KiB loads of the weights per stage
  static constexpr int XROWS_LOAD = 4096 / XR;                 // pair rows per load
  static constexpr int NX = (NJ * 32 + XROWS_LOAD - 1) / XROWS_LOAD;
  static constexpr int NL = NW + NX;
  static constexpr int SB = NL * 4096;                         // bytes of a stage
  static constexpr int NS = kFullLds / SB;
  static_assert(NS >= 2 && NS <= 4, "ring");

  f32x16 acc[2][NJ];

  // rowp[i]: where this thread's chunk of its i-th row starts (K position 0); wsrc: this thread's chunk of the first weight
  // stage, img: bytes from one image to the next; once: no other item reads these weights (non-temporal loads, see gemm_mfma.hip);
  // next(xo, wo): byte offset of the next stage in a pair row and in the weight stages
  template <bool SAFE, class Next>
  __device__ __forceinline__ void run(int n, const char* const (&rowp)[NX], const char* wsrc, int64_t img, bool once, Next next, const char* lds, int w, int lane) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][j][v] = 0.f;
    const uint32_t base = lds_byte(lds) + (uint32_t)w * 1024;
    auto issue = [&](int st) {
      int64_t xo, wo;
      next(xo, wo);
      const uint32_t slot = base + (uint32_t)(st % NS) * SB;
      if (once) {
#pragma unroll
        for (int q = 0; q < NW; ++q) dma16g<true>(wsrc + (q >> 1) * img + wo + (q & 1) * 4096, slot + q * 4096);
      } else {
#pragma unroll
        for (int q = 0; q < NW; ++q) dma16g(wsrc + (q >> 1) * img + wo + (q & 1) * 4096, slot + q * 4096);
      }
#pragma unroll
      for (int q = 0; q < NX; ++q) dma16g(rowp[q] + xo, slot + (NW + q) * 4096);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < n) issue(s);
    int st = 0;
    for (; st + NS - 1 < n; ++st) {
      wait_loads<(NS - 2) * NL>();  // stage st has landed (for this wavefront; the barrier makes it so for all)
      read_barrier();
      issue(st + NS - 1);           // into the slot of stage st - 1, which every wavefront has finished reading
      multiply<SAFE>(lds + (st % NS) * SB, w, lane);
    }
    for (; st < n; ++st) {
      const int left = n - 1 - st;  // later stages still in flight
      if (left >= NS - 2) wait_loads<(NS - 2) * NL>();
      else if (NS > 3 && left == 1) wait_loads<NL>();
      else wait_loads<0>();
      read_barrier();
      multiply<SAFE>(lds + (st % NS) * SB, w, lane);
    }
  }

  // SAFE (fp32 activations): right for infinite and NaN operands as well: activations are clamped (see split3), and infinite and NaN weights left out
  // of the two smaller products, whose other operand may be zero.
  template <bool SAFE>
  __device__ __forceinline__ void multiply(const char* stage, int w, int lane) {
    const int r32 = lane & 31, h = lane >> 5;
    const char* wrow = stage + (w * 32 + r32) * WR;
    const char* xrow = stage + NW * 4096 + r32 * XR;
    auto wchunk = [&](int b, int c) { return wrow + b * IMG + swz_chunk(r32, c) * 16; };
    auto xchunk = [&](int j, int c) { return xrow + j * 32 * XR + swz_full<XCH>(r32, c) * 16; };
#pragma unroll
    for (int s = 0; s < 2; ++s) {  // K values 16s + 8h .. 16s + 8h + 7
      bf16x8 a[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) a[b] = *(const bf16x8*)wchunk(b, 2 * s + h);
      if constexpr (XE == 2) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bf16x8 x = *(const bf16x8*)xchunk(j, 2 * s + h);
#pragma unroll
          for (int b = 0; b < 2; ++b) acc[b][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[b], x, acc[b][j], 0, 0, 0);
        }
      } else {
        bf16x8 small[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) small[b] = SAFE ? finite_only(a[b]) : a[b];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          u32x4 part[3];
          split3<SAFE>(*(const f32x4*)xchunk(j, 4 * s + 2 * h), *(const f32x4*)xchunk(j, 4 * s + 2 * h + 1), part);
#pragma unroll
          for (int k = 2; k >= 0; --k)  // the small parts first
#pragma unroll
            for (int b = 0; b < 2; ++b)
              acc[b][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k == 0 ? a[b] : small[b], __builtin_bit_cast(bf16x8, part[k]), acc[b][j], 0, 0, 0);
          if (SAFE) __builtin_amdgcn_sched_barrier(0);  // (registers)
        }
      }
    }
  }
};

// it.jt: the tile
template <int NJ>
__device__ __forceinline__ void gemm1_wide_tile(const Layout& L, const Item1& it, const char* packed, const char* x, int64_t x_row, char* ws, int epi, char* lds,
                                                int w, int lane) {
  using Tile = WideTile<2, NJ>;
  const int tid = w * 64 + lane;
  const bool sh = it.e == L.E_res;
  const int Fpk = sh ? L.Fsk : L.Fpk, ld = sh ? L.Fsk : L.Fh, NI1 = sh ? L.NI1_sh : L.NI1;
  const int KS = L.Dk / kBK;
  const int32_t* row_token = (const int32_t*)(ws + L.o_row_token) + it.row0;
  const uint8_t* row_bits = (const uint8_t*)(ws + L.o_row_bits) + it.row0;
  const int64_t img = (int64_t)KS * Tile::IMG;  // bytes of an image
  const char* wsrc = packed + (sh ? L.p_sw13 : L.p_w13) + ((int64_t)(sh ? 0 : it.e * L.P + it.p) * NI1 + 2 * it.jt) * img + tid * 16;
  const char* rowp[Tile::NX];
#pragma unroll
  for (int i = 0; i < Tile::NX; ++i) {
    const int r = i * Tile::XROWS_LOAD + tid / Tile::XCH;
    const int rr = r < it.nrows ? r : it.nrows - 1;  // rows past the end re-read the last one
    rowp[i] = x + (int64_t)row_token[rr] * x_row + swz_full<Tile::XCH>(r, tid % Tile::XCH) * 16;
  }
  Tile t;
  t.template run<false>(KS, rowp, wsrc, img, it.once, [k = (int64_t)0](int64_t& xo, int64_t& wo) mutable {
    xo = k * Tile::XR;
    wo = k * Tile::IMG;
    ++k;
  }, lds, w, lane);
  // acc[b][j][v]: weight row 8*(v/4) + 4*h + v%4 of the wavefront's 32 of image b (see gemm1_full_tile), pair row j*32 + lane%32
  float* H = (float*)(ws + (sh ? L.o_Hs : L.o_H)) + (size_t)(sh ? it.row0 : it.row0 - L.sh_rows) * ld + (size_t)it.p * Fpk;
  const int n0 = it.jt * (2 * kFullNeur) + w * 16 + (lane >> 5) * 4;
  const int Fp = sh ? L.F_shT : L.Fp;  // the neurons that pad a partition are zeros, see gemm1_full_tile
  float z = 0.f;                       // stays zero as long as every activation is finite
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int r = j * 32 + (lane & 31);
    if (r >= it.nfill) continue;
    const bool kept = r < it.nrows && ((row_bits[r] >> it.p) & 1);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int n = n0 + b * kFullNeur + g * 8;
        f32x4 o;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          o[c] = kept && n + c < Fp ? epi_value<false>(epi, t.acc[b][j][g * 4 + c], t.acc[b][j][8 + g * 4 + c]) : 0.f;
          z = __builtin_fmaf(o[c], 0.f, z);
        }
        if (n < Fpk) *(f32x4*)(H + (size_t)r * ld + n) = o;
      }
  }
  if (z != 0.f) ((int32_t*)(ws + L.o_counters))[kNonfiniteH] = 1;  // (true for NaN)
  for (int r = NJ * 32 + (lane & 31); r < it.nfill; r += 32) {  // rows that keep nothing of this partition, beyond the blocks multiplied: zeros
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + (q >> 1) * kFullNeur + (q & 1) * 8;
      if (n < Fpk) *(f32x4*)(H + (size_t)r * ld + n) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
}

__global__ __launch_bounds__(256, 2) void gemm1_wide_kernel(Layout L, const char* packed, const char* x, int64_t x_row, char* ws, int epi) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int32_t* counters = (int32_t*)(ws + L.o_counters);
  const int items = counters[0], n = full_pieces(items), id = take_piece<true>(n, counters + 8, lds);
  if (id >= n) return;
  const FullPiece piece = full_piece(items, id);
  Item1 it = ((const Item1*)(ws + L.o_items1))[piece.item];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blocks = (it.nrows + 31) >> 5, images = min((it.e == L.E_res ? L.NI1_sh : L.NI1) - 2 * it.jt, 2);
  if (piece.half >= images) return;
  if (piece.half < 0 && images == 2) {
    switch (blocks) {
      case 1: gemm1_wide_tile<1>(L, it, packed, x, x_row, ws, epi, lds, w, lane); break;
      case 2: gemm1_wide_tile<2>(L, it, packed, x, x_row, ws, epi, lds, w, lane); break;
      case 3: gemm1_wide_tile<3>(L, it, packed, x, x_row, ws, epi, lds, w, lane); break;
      default: gemm1_wide_tile<4>(L, it, packed, x, x_row, ws, epi, lds, w, lane); break;
    }
    return;
  }
  it.jt = 2 * it.jt + max(piece.half, 0);
  switch (blocks) {
    case 1: gemm1_full_tile<uint16_t, 1, 1>(L, it, 0, packed, x, x_row, ws, epi, lds, w, lane); break;
    case 2: gemm1_full_tile<uint16_t, 2, 1>(L, it, 0, packed, x, x_row, ws, epi, lds, w, lane); break;
    case 3: gemm1_full_tile<uint16_t, 3, 1>(L, it, 0, packed, x, x_row, ws, epi, lds, w, lane); break;
    default: gemm1_full_tile<uint16_t, 4, 1>(L, it, 0, packed, x, x_row, ws, epi, lds, w, lane); break;
  }
}

// it.jd: the tile
template <int NJ, bool SAFE>
__device__ __forceinline__ void gemm2_wide_tile(const Layout& L, const Item2& it, const char* packed, char* ws, char* lds, int w, int lane) {
  using Tile = WideTile<4, NJ>;
  const int tid = w * 64 + lane;
  const bool sh = it.e == L.E_res;
  const int ld = sh ? L.Fsk : L.Fh;
  const int KSp = (sh ? L.Fsk : L.Fpk) / kBK, np = sh ? 1 : L.P;  // stages of one partition, partitions
  const float* H = (const float*)(ws + (sh ? L.o_Hs : L.o_H)) + (size_t)(sh ? it.row0 : it.row0 - L.sh_rows) * ld;
  const int64_t img = (int64_t)np * KSp * Tile::IMG;  // bytes of an image
  const char* wsrc = packed + (sh ? L.p_sw2 : L.p_w2) + ((int64_t)(sh ? 0 : it.e) * L.NI2 + 2 * it.jd) * img + tid * 16;
  const char* rowp[Tile::NX];
#pragma unroll
  for (int i = 0; i < Tile::NX; ++i) {
    const int r = i * Tile::XROWS_LOAD + tid / Tile::XCH;
    const int rr = r < it.nrows ? r : it.nrows - 1;
    rowp[i] = (const char*)(H + (size_t)rr * ld) + swz_full<Tile::XCH>(r, tid % Tile::XCH) * 16;
  }
  const int32_t* multi = (const int32_t*)(ws + L.o_counters) + 5;  // see gemm2_setup in gemm_mfma.hip
  const bool once = !sh && !((multi[(it.e >> 5) & 1] >> (it.e & 31)) & 1);
  // stages run over the partitions that some row of the tile keeps, see gemm2_full_tile
  const int ks_n = it.ks_n, ks_lo = it.ks_lo, kmask = it.kmask;
  int n = 0;
  for (int p = 0; p < np; ++p) n += ((kmask >> p) & 1) ? ks_n : 0;
  int p_cur = 0;
  while (p_cur < np && !((kmask >> p_cur) & 1)) ++p_cur;
  Tile t;
  t.template run<SAFE>(n, rowp, wsrc, img, once, [=, k_in = 0](int64_t& xo, int64_t& wo) mutable {
    const int64_t kt = p_cur * KSp + ks_lo + k_in;
    if (++k_in == ks_n) {
      k_in = 0;
      ++p_cur;
      while (p_cur < np && !((kmask >> p_cur) & 1)) ++p_cur;
    }
    xo = kt * Tile::XR;
    wo = kt * Tile::IMG;
  }, lds, w, lane);
  // acc[b][j][v]: output column b*128 + w*32 + 8*(v/4) + 4*h + v%4 of the tile, pair row j*32 + lane%32
  float* Y;
  int ldy;
  if (it.split == 0) {
    Y = (float*)(ws + L.o_Yp) + (size_t)it.row0 * L.D + it.jd * (2 * kFullBN2);
    ldy = L.D;
  } else {
    Y = (float*)(ws + L.o_pool) + (size_t)(it.split - 1) * L.pool_rows * (2 * kFullBN2);
    ldy = 2 * kFullBN2;
  }
  const int c0 = w * 32 + (lane >> 5) * 4;
  const bool vec = (L.D & 3) == 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int r = j * 32 + (lane & 31);
    if (r >= it.nrows) continue;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = c0 + b * kFullBN2 + g * 8, d = it.jd * (2 * kFullBN2) + c;
        float* at = Y + (size_t)r * ldy + c;
        if (vec) {
          if (d < L.D) *(f32x4*)at = f32x4{t.acc[b][j][g * 4], t.acc[b][j][g * 4 + 1], t.acc[b][j][g * 4 + 2], t.acc[b][j][g * 4 + 3]};
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (d + i < L.D) at[i] = t.acc[b][j][g * 4 + i];
        }
      }
  }
}

__global__ __launch_bounds__(256, 2) void gemm2_wide_kernel(Layout L, const char* packed, char* ws) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int32_t* counters = (int32_t*)(ws + L.o_counters);
  const int items = counters[1], n = full_pieces(items), id = take_piece<true>(n, counters + 9, lds);
  if (id >= n) return;
  const FullPiece piece = full_piece(items, id);
  Item2 it = ((const Item2*)(ws + L.o_items2))[piece.item];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blocks = (it.nrows + 31) >> 5, images = min(L.NI2 - 2 * it.jd, 2);
  const bool nonfinite = ((const PackRecord*)(packed + L.p_scale))->largest != 0;  // some weight of W2 is infinite or NaN
  if (piece.half >= images) return;
  if (piece.half < 0 && images == 2) {
#define DSMOE_ROWS(SAFE)                                                                 \
  switch (blocks) {                                                                      \
    case 1: gemm2_wide_tile<1, SAFE>(L, it, packed, ws, lds, w, lane); break;            \
    case 2: gemm2_wide_tile<2, SAFE>(L, it, packed, ws, lds, w, lane); break;            \
    case 3: gemm2_wide_tile<3, SAFE>(L, it, packed, ws, lds, w, lane); break;            \
    default: gemm2_wide_tile<4, SAFE>(L, it, packed, ws, lds, w, lane); break;           \
  }
    if (nonfinite || counters[kNonfiniteH]) {
      DSMOE_ROWS(true)
    } else {
      DSMOE_ROWS(false)
    }
#undef DSMOE_ROWS
    return;
  }
  it.jd = 2 * it.jd + max(piece.half, 0);
#define DSMOE_ROWS(NONFINITE)                                                                                 \
  switch (blocks) {                                                                                           \
    case 1: gemm2_full_tile<uint16_t, 1, 1, NONFINITE>(L, it, 0, packed, ws, lds, w, lane); break;            \
    case 2: gemm2_full_tile<uint16_t, 2, 1, NONFINITE>(L, it, 0, packed, ws, lds, w, lane); break;            \
    case 3: gemm2_full_tile<uint16_t, 3, 1, NONFINITE>(L, it, 0, packed, ws, lds, w, lane); break;            \
    default: gemm2_full_tile<uint16_t, 4, 1, NONFINITE>(L, it, 0, packed, ws, lds, w, lane); break;           \
  }
  if (nonfinite) {
    DSMOE_ROWS(true)
  } else {
    DSMOE_ROWS(false)
  }
#undef DSMOE_ROWS
}

// x with every row at the start of a 16-byte group and zeros up to a multiple of 32 values: made where the layer's width or
// the caller's pointer does not give that (one small pass; kept where GEMM-2 later writes Yp)
template <typename T>
__global__ __launch_bounds__(256) void pad_rows_kernel(const T* x, T* out, int D, int Dk, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (int64_t)gridDim.x * 256) {
    const int64_t t = q / Dk;
    const int d = (int)(q - t * Dk);
    out[q] = d < D ? x[t * D + d] : (T)0;
  }
}

static hipError_t set_lds_attr() {
  static PerDeviceOnce once;
  return once.run([] {
    for (const void* fn : {(const void*)gemm1_wide_kernel, (const void*)gemm2_wide_kernel,
                           (const void*)gemm1_full_kernel<float, 0>, (const void*)gemm2_full_kernel<float, 0>,
                           (const void*)gemm1_full_kernel<float, 1>, (const void*)gemm1_full_kernel<float, 2>, (const void*)gemm1_full_kernel<uint16_t, 1>,
                           (const void*)gemm1_full_kernel<uint16_t, 2>, (const void*)gemm2_full_kernel<float, 1>, (const void*)gemm2_full_kernel<float, 2>,
                           (const void*)gemm2_full_kernel<uint16_t, 1>, (const void*)gemm2_full_kernel<uint16_t, 2>}) {
      hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kFullLds);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
}

// Workgroups that share a weight tile.  With a few rows per expert the kernels stream weights in items that are too few or too
// long for the chip, and two halves are better: 64 tokens on 8 experts of 128 x 256 (16 pairs each) 27.0 -> 24.2 us, 64 tokens
// top-8 on 64 experts of 2048 x 1024 in fp32 311 -> 301, 100 top-6 on 64 + 2 of 2048 x 1408 in parts of 176 318 -> 303; under uneven
// routing more so (127 of the fp32 ones with popularity rank^-1.2 280 -> 204).  Beyond, the rows are read twice for nothing: 300
// tokens (37 pairs each) on the former 390 -> 414 us, 400 on the latter 335 -> 354.  An expert's share of the pairs does not
// depend on how many experts are resident: 64 tokens on 8 of those 64 experts 82 -> 68 us, on 2 of 8 of 1024 x 2048 49 -> 40.
// From 32 fp32 pairs per expert on (before any drop) the kernels are bound by the matrix cores, and the last items of the list are cut:
// 512 / 300 tokens top-8 on 64 experts of 2048 x 1024 472 -> 463 us, 360 -> 355, 400 / 1000 top-2 on 8 of 128 x 256 32.4 -> 28.4, 42.4 -> 35.9; 200 of the
// former (25 pairs each) 324 -> 328.
static int full_parts(const Layout& L, int T) {
  const int64_t pairs = (int64_t)T * L.K;
  return pairs <= (int64_t)L.E * 16 ? 2 : L.dtype == DSMOE_F32 && pairs >= (int64_t)L.E * 32 ? 0 : 1;
}

// Tiles of two images: bf16 layers, where experts have rows enough to reuse what was cut.  The line is in pairs per expert before any drop, as
// the host knows no more.  Single images -> two, us per layer, 700 / 777 / 1500 tokens on 64 + 2 experts of 2048 x 1408 in parts of 176, top-6
// (66 / 73 / 141 pairs per expert): nothing dropped 449 -> 440, 467 -> 422, 723 -> 632; 25 % dropped 419 -> 418, 431 -> 399, 641 -> 587;
// 50 % 383 -> 391, 399 -> 375, 550 -> 499; 25 % and popularity rank^-1.2 450 -> 408, 466 -> 437, 685 -> 612.  520 / 777 / 1500 on 64 of
// 2048 x 1000 in parts of 250, top-8 (65 / 97 / 188): 263 -> 266, 319 -> 320, 544 -> 448; 242 -> 237, 285 -> 286, 462 -> 427; 223 -> 219,
// 255 -> 250, 370 -> 329; 300 -> 249, 333 -> 292, 471 -> 395.  300 / 500 tokens (28 / 47 pairs) of the first 346 -> 352, 378 -> 379.
// Layers of few weight images (short lists) are not measured and keep single ones.
// fp32 layers: with both images to a tile and the fp32 instructions 250 / 300 / 400 / 512 tokens on 64 experts of 2048 x 1024, top-8, 25 % dropped,
// took 409 -> 432, 423 -> 440, 486 -> 454, 559 -> 571, and 488 -> 735 at 250 with popularity rank^-1.2.
bool full_wide(const Layout& L, int T) {
  return L.dtype == DSMOE_BF16 && (int64_t)T * L.K > 64 * (int64_t)L.E && (int64_t)L.E_res * L.P * L.NI1 >= 2 * kFullSplitItems &&
         (int64_t)L.E_res * L.NI2 >= 2 * kFullSplitItems;
}

hipError_t launch_gemm1_full(const Layout& L, int T, const char* packed, const void* x, char* ws, int epi, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  hipError_t e = set_lds_attr();
  if (e != hipSuccess) return e;
  const int64_t elem = L.dtype == DSMOE_F32 ? 4 : 2;
  const char* xs = (const char*)x;
  int64_t x_row = L.D * elem;
  if (L.D != L.Dk || ((uintptr_t)x & 15) != 0) {
    const int64_t n = (int64_t)T * L.Dk;
    const dim3 grid((unsigned)blocks_of_256(n)), block(256);
    if (elem == 4) pad_rows_kernel<float><<<grid, block, 0, s>>>((const float*)x, (float*)(ws + L.o_Yp), L.D, L.Dk, n);
    else pad_rows_kernel<uint16_t><<<grid, block, 0, s>>>((const uint16_t*)x, (uint16_t*)(ws + L.o_Yp), L.D, L.Dk, n);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    xs = ws + L.o_Yp;
    x_row = L.Dk * elem;
  }
  if (L.wide) {
    const dim3 grid(piece_blocks(true, items1_bound(L, T) + kFullHalved)), block(256);
    gemm1_wide_kernel<<<grid, block, kFullLds, s>>>(L, packed, xs, x_row, ws, epi);
    return hipGetLastError();
  }
  const int subs = full_parts(L, T);
  const int items = items1_bound(L, T);
  const dim3 block(256), grid(piece_blocks(true, subs == 2 ? 2 * items : items + (subs == 0 ? kFullHalved : 0)));
#define DSMOE_LAUNCH(TYPE, SUBS) gemm1_full_kernel<TYPE, SUBS><<<grid, block, kFullLds, s>>>(L, packed, xs, x_row, ws, epi)
  if (elem == 4 && subs == 2) DSMOE_LAUNCH(float, 2);
  else if (elem == 4 && subs == 0) DSMOE_LAUNCH(float, 0);
  else if (elem == 4) DSMOE_LAUNCH(float, 1);
  else if (subs == 2) DSMOE_LAUNCH(uint16_t, 2);
  else DSMOE_LAUNCH(uint16_t, 1);
#undef DSMOE_LAUNCH
  return hipGetLastError();
}

hipError_t launch_gemm2_full(const Layout& L, int T, const char* packed, char* ws, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  hipError_t e = set_lds_attr();
  if (e != hipSuccess) return e;
  if (L.wide) {
    const dim3 grid(piece_blocks(true, items2_bound(L, T) + kFullHalved)), block(256);
    gemm2_wide_kernel<<<grid, block, kFullLds, s>>>(L, packed, ws);
    return hipGetLastError();
  }
  const int subs = full_parts(L, T);
  const int items = items2_bound(L, T);
  const dim3 block(256), grid(piece_blocks(true, subs == 2 ? 2 * items : items + (subs == 0 ? kFullHalved : 0)));
#define DSMOE_LAUNCH(TYPE, SUBS) gemm2_full_kernel<TYPE, SUBS><<<grid, block, kFullLds, s>>>(L, packed, ws)
  if (L.dtype == DSMOE_F32 && subs == 2) DSMOE_LAUNCH(float, 2);
  else if (subs == 0) DSMOE_LAUNCH(float, 0);
  else if (L.dtype == DSMOE_F32) DSMOE_LAUNCH(float, 1);
  else if (subs == 2) DSMOE_LAUNCH(uint16_t, 2);
  else DSMOE_LAUNCH(uint16_t, 1);
#undef DSMOE_LAUNCH
  return hipGetLastError();
}

}  // namespace dsmoe
