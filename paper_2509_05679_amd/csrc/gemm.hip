// MFMA implicit-GEMM kernels for gfx950: convolution / linear forward and input gradient, and weight gradients with a
// split pixel reduction. Operands of the first two kernels of each list are copied global -> LDS without passing through registers.
//   forward and input gradient: conv3x3_dma_kernel (3x3 stride 1), conv_gather_kernel (any other layer of whole 64-byte
//     channel chunks), conv_gemm_kernel (the rest, e.g. the 3-channel stem)
//   weight gradient, bf16: wgrad_dma_body (sides that are powers of two, whole 128-pixel tiles), wgrad_flat_body (other
//     sizes), wgrad_rows_body (1x1, linear), wgrad_gemm_kernel (the rest); fp32: wgrad_f32_kernel
// (Plain products of few rows: linear.hip. 16-channel layers: narrow.hip.)
//
// Operand tiles are K-contiguous in LDS ([row][k]; wgrad_dma_body, wgrad_flat_body and wgrad_f32_kernel keep [pixel][channel])
// and feed v_mfma_f32_32x32x16_bf16 (bf16) or v_mfma_f32_32x32x2_f32 (fp32) with one 16-byte LDS read per operand fragment. The fp32 kernels
// of 3x3 stride-1 layers and of weight gradients multiply bf16 parts instead (split3): six of those products cost 3/8 of one on the fp32 unit.
// Lanes 0-31 read the first 16 bytes of a 32-byte k-step and lanes 32-63 the second, for A and B alike, so the
// pairing of k indices inside an instruction is consistent by construction.
//
// The fp32 sums of linear, 1x1 and strided layers keep one order per problem, whichever kernel or tile its size selects: a program's fp32
// results change by single ReLU decisions when the last bits of a sum do. That is why here and in linear.hip and misc.hip (update, pooling)
// some rules name the type; see wgrad_generic_split, linear_kernel, gap_fwd_kernel and update_elems. (The mixing update of misc.hip is not held
// to it: its sum runs over the row-lanes that the split count selects.) 3x3 stride-1 layers keep the order of their tile's kernel: a chunk of sixteen
// channels, its taps, resident weights apart from the rest.
#include <cstdlib>

#include "device_once.h"
#include "kernels.h"
#include "lds_copy.h"

namespace dds {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

struct bf16_t { uint16_t v; };

template <typename T> __device__ __forceinline__ void mfma16B(const uint4& a, const uint4& b, f32x16_t& c);
template <> __device__ __forceinline__ void mfma16B<bf16_t>(const uint4& a, const uint4& b, f32x16_t& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ void mfma16B<float>(const uint4& a, const uint4& b, f32x16_t& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

// Eight fp32 values as sums of three bf16 values each: every step rounds to nearest, the remainders are exact and the third part holds what is
// left (8 bits a step of 24). Of the nine products of parts the three smallest are below 2^-24 of the whole and left out. Relative 2-norm error
// against fp64, medians of 6 seeds, fp32 unit / parts: outputs of a layer of 64 channels 2.9e-7 / 1.6e-7, of 512 8.1e-7 / 2.0e-7; input gradients 3.1e-7
// / 1.9e-7 and 8.2e-7 / 2.6e-7; weights after 4 to 10 steps of the fp32 CNN at 1 x 8 6.7e-8 / 6.0e-8, 2 x 16 8.3e-7 / 1.6e-7, of ResNet-20 at 16 5.03e-8 / 5.03e-8,
// of the odd net at 12 x 12 5.29e-8 / 5.29e-8; worst layer of the normalised ResNet-18 in fp32 at 4 x 3 3.1e-5 / 1.7e-5. (The unit
// truncates where it adds, so the long sums are formed by the vector unit out of short ones: with six additions to the long sum for every
// sixteen terms a layer's errors were 1.15 times the fp32 unit's.)
// (value - part by v_dot2c_f32_bf16, one instruction for two: 99 -> 113 us a launch, it is slower than the two.)
struct Parts { uint4 part[3]; };
__device__ __forceinline__ uint32_t split_pair(float& lo, float& hi) {  // leaves the remainders
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const uint32_t pair = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), bf16x2_t));
  lo -= __uint_as_float(pair << 16);
  hi -= __uint_as_float(pair & 0xffff0000u);
  return pair;
}
__device__ __forceinline__ Parts split3(const float (&v)[8]) {
  Parts r;
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float lo = v[2 * e], hi = v[2 * e + 1];
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k][e] = split_pair(lo, hi);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) r.part[k] = make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]);
  return r;
}
__device__ __forceinline__ Parts split3(const uint4& x, const uint4& y) {
  return split3({__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w), __uint_as_float(y.x), __uint_as_float(y.y),
                 __uint_as_float(y.z), __uint_as_float(y.w)});
}
// c[] += b[] a over sixteen k: the six products of parts that reach 2^-24 of a term, smallest first, summed apart so that the
// long sum is rounded once in sixteen k.
constexpr int kPartA[6] = {0, 2, 1, 0, 1, 0}, kPartB[6] = {2, 0, 1, 1, 0, 0};
template <int N>
__device__ __forceinline__ void mfma_split(const Parts& a, const Parts (&b)[N], f32x16_t* const (&c)[N]) {
  f32x16_t t[N] = {};
#pragma unroll
  for (int k = 0; k < 6; ++k)
#pragma unroll
    for (int n = 0; n < N; ++n) mfma16B<bf16_t>(b[n].part[kPartA[k]], a.part[kPartB[k]], t[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) *c[n] += t[n];
}
template <int N>
__device__ __forceinline__ bool any_nan(const f32x16_t (&acc)[N]) {
  bool r = false;
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int e = 0; e < 16; ++e) r |= acc[n][e] != acc[n][e];
  return r;
}
// Is `mine` set in any lane of the workgroup? (words: of LDS, one per wave, that nobody reads or copies to any more when all waves are here)
__device__ __forceinline__ bool workgroup_any(bool mine, char* words, int wave, int nwaves) {
  __syncthreads();
  const bool w = __ballot(mine) != 0;
  volatile int* at = (volatile int*)words;
  at[wave] = w;
  __syncthreads();
  int r = 0;
  for (int i = 0; i < nwaves; ++i) r |= at[i];
  return r != 0;
}

__device__ __forceinline__ uint4 keep_if(bool ok, const uint4& v) {
  return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}

// One BKB-byte-deep step of a WM x WN wave tile. As / Bs point at the wave's first row.
template <typename T, int WM, int WN, int BKB>
__device__ __forceinline__ void mma_step(const char* As, const char* Bs, int lane, f32x16_t (&acc)[WM / 32][WN / 32]) {
  constexpr int LDK = BKB + 16;
  const int row = lane & 31, half = lane >> 5;
#pragma unroll
  for (int ks = 0; ks < BKB / 32; ++ks) {
    uint4 a[WM / 32], b[WN / 32];
#pragma unroll
    for (int i = 0; i < WM / 32; ++i) a[i] = *(const uint4*)(As + (i * 32 + row) * LDK + ks * 32 + half * 16);
#pragma unroll
    for (int j = 0; j < WN / 32; ++j) b[j] = *(const uint4*)(Bs + (j * 32 + row) * LDK + ks * 32 + half * 16);
#pragma unroll
    for (int i = 0; i < WM / 32; ++i)
#pragma unroll
      for (int j = 0; j < WN / 32; ++j) mfma16B<T>(a[i], b[j], acc[i][j]);
  }
}

// LDS loads through an explicit address-space pointer (HIP's vector classes cannot be
// referenced through one, so native vector types carry the bits)
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
template <typename R> __device__ __forceinline__ R lds_load(const char DDS_LDS_AS* p);
template <> __device__ __forceinline__ uint4 lds_load<uint4>(const char DDS_LDS_AS* p) {
  const u32x4_t v = *(const u32x4_t DDS_LDS_AS*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <> __device__ __forceinline__ uint2 lds_load<uint2>(const char DDS_LDS_AS* p) {
  const u32x2_t v = *(const u32x2_t DDS_LDS_AS*)p;
  return make_uint2(v.x, v.y);
}

// Four consecutive output channels of one pixel: v = alpha*(acc+bias) (+res) (relu) (mask),
// moved with one 8-byte (bf16) or 16-byte (fp32) access per operand. n is a multiple of 4.
template <typename T> __device__ __forceinline__ void load4(const void* p, size_t i, float* v);
template <> __device__ __forceinline__ void load4<float>(const void* p, size_t i, float* v) {
  const float4 t = *(const float4*)((const float*)p + i);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ __forceinline__ void load4<bf16_t>(const void* p, size_t i, float* v) {
  const uint2 t = *(const uint2*)((const uint16_t*)p + i);
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
}
template <typename T> __device__ __forceinline__ void store4(void* p, size_t i, const float* v);
template <> __device__ __forceinline__ void store4<float>(void* p, size_t i, const float* v) {
  *(float4*)((float*)p + i) = make_float4(v[0], v[1], v[2], v[3]);
}
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// two floats -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
template <> __device__ __forceinline__ void store4<bf16_t>(void* p, size_t i, const float* v) {
  uint2 t;
  t.x = pack_bf16(v[0], v[1]);
  t.y = pack_bf16(v[2], v[3]);
  *(uint2*)((uint16_t*)p + i) = t;
}

// Epilogue of one 32-pixel tile column of a wave: this lane owns pixel `pix` and, for each
// of the NJ channel tiles, four groups of 4 consecutive channels starting at
// nb + 32*j + 8*g. All residual / mask reads are issued up front from clamped addresses
// (no branch around a load, so none of them is waited for one by one), then
// v = alpha*(acc+bias) (+res) (relu) (mask) is formed and stored with predicated vector stores.
template <typename T> struct Raw4;
template <> struct Raw4<float> { typedef uint4 type; };
template <> struct Raw4<bf16_t> { typedef uint2 type; };
__device__ __forceinline__ void unpack4(const uint4& t, float* v) {
  v[0] = __uint_as_float(t.x); v[1] = __uint_as_float(t.y); v[2] = __uint_as_float(t.z); v[3] = __uint_as_float(t.w);
}
__device__ __forceinline__ void unpack4(const uint2& t, float* v) {
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
}

// x > 0 decided on the stored bits (no conversion): fp32 as is; a packed bf16 pair w holds
// lo in bits 0-15 and hi in bits 16-31: hi > 0 <=> (int)w >= 0x10000, lo > 0 <=> (int)(w << 16) >= 0x10000
__device__ __forceinline__ void positive4(const uint4& t, bool* pos) {
  pos[0] = __uint_as_float(t.x) > 0.f; pos[1] = __uint_as_float(t.y) > 0.f;
  pos[2] = __uint_as_float(t.z) > 0.f; pos[3] = __uint_as_float(t.w) > 0.f;
}
__device__ __forceinline__ void positive4(const uint2& t, bool* pos) {
  pos[0] = (int)(t.x << 16) >= 0x10000; pos[1] = (int)t.x >= 0x10000;
  pos[2] = (int)(t.y << 16) >= 0x10000; pos[3] = (int)t.y >= 0x10000;
}

// Four bytes of a sign plane row: channels cbase .. cbase+31 of pixel pix (zero where the row ends earlier).
__device__ __forceinline__ uint32_t load_bits32(const void* bits, size_t pix, int ldy, int cbase, bool valid) {
  if (!valid || cbase >= ldy) return 0u;
  const uint8_t* row = (const uint8_t*)bits + pix * (size_t)(ldy >> 3) + (cbase >> 3);
  if ((ldy & 31) == 0) return *(const uint32_t*)row;
  uint32_t w = 0;
  for (int b = 0; b < 4 && cbase + 8 * b < ldy; ++b) w |= (uint32_t)row[b] << (8 * b);
  return w;
}
__device__ __forceinline__ void store_bits32(void* bits, size_t pix, int ldy, int cbase, uint32_t w) {
  if (cbase >= ldy) return;
  uint8_t* row = (uint8_t*)bits + pix * (size_t)(ldy >> 3) + (cbase >> 3);
  if ((ldy & 31) == 0) { *(uint32_t*)row = w; return; }
  for (int b = 0; b < 4 && cbase + 8 * b < ldy; ++b) row[b] = (uint8_t)(w >> (8 * b));
}
// nibble i of x -> bits [8i, 8i+4)
__device__ __forceinline__ uint32_t spread_nibbles(uint32_t x) {
  return (x & 0xfu) | ((x & 0xf0u) << 4) | ((x & 0xf00u) << 8) | ((x & 0xf000u) << 12);
}

// bias values of this lane's channel groups (zero past Nout), read once per kernel
template <int NJ>
__device__ __forceinline__ void load_bias_groups(const ConvParams& p, int nb, float (&bias)[NJ][4][4]) {
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = nb + 32 * j + 8 * g + q;
        float b = 0.f;
        if (p.bias) b = p.bias[n < p.Nout ? n : 0];
        bias[j][g][q] = n < p.Nout ? b : 0.f;
      }
}

// res_off / mask_off >= 0: the tile's residual / mask values were staged in LDS as
// [tile row][row_bytes] with 16-byte column c of row m stored at column c ^ (m & (ncol-1));
// tile_row is this lane's row, ncol = row_bytes / 16, nloc0 the lane's first channel inside the tile.
// The function is laid out in phases (gather operands, arithmetic, store, sign plane) with one
// uniform branch per phase at most: every option inside the arithmetic is a select, not a
// branch, because each branch costs the compiler's conservative waits at its join.
template <typename T, int NJ, int NI>
__device__ __forceinline__ void epilogue_tile(const ConvParams& p, const f32x16_t (&acc)[NJ][NI], int i, bool valid,
                                              size_t pix, int nb, const float (&bias)[NJ][4][4],
                                              const char DDS_LDS_AS* lds = nullptr, int res_off = -1, int mask_off = -1,
                                              int tile_row = 0, int row_bytes = 0, int nloc0 = 0, int ab_off = -1,
                                              const uint32_t* mbits = nullptr, int out_off = -1) {
  typedef typename Raw4<T>::type raw_t;
  static_assert(NJ <= 2, "the sign words hold 8 nibbles");
  const int half = (threadIdx.x >> 5) & 1;   // which 4 channels of every 8 this lane holds
  const int nwave0 = nb - 4 * half;           // first channel of the wave's span
  const int ncolm = (row_bytes >> 4) - 1;
  // explicit LDS address space: a generic pointer would turn these into flat loads, which
  // also count as vector-memory operations and would wait for every earlier global store
  auto lds_at = [&](int base_off, int j, int g) {
    const int bytecol = (nloc0 + 32 * j + 8 * g) * (int)sizeof(T);
    return (char DDS_LDS_AS*)lds + base_off + tile_row * row_bytes + ((((bytecol >> 4) ^ tile_row) & ncolm) << 4) + (bytecol & 15);
  };
  size_t o[NJ][4];
  bool ok[NJ][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = nb + 32 * j + 8 * g;
      ok[j][g] = valid && n < p.ldy;
      o[j][g] = ok[j][g] ? pix * p.ldy + n : 0;
    }

  uint32_t signs = 0;  // nibble 4 j + g: this lane's four outputs of group (j, g) that are > 0
  const float lower = p.relu ? 0.f : -__builtin_inff();
#pragma unroll
  for (int j = 0; j < NJ; ++j) {  // one 32-channel tile at a time keeps the temporaries at 16 registers each
    // ---- gather: alpha * bias, residual, mask (defaults: 0, 0, keep everything)
    float ab[4][4], rs[4][4];
    uint32_t keep = 0xffffffffu;  // bit 8 g + 4 half + q: output (g, q) survives the mask
    if (ab_off >= 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint4 t = lds_load<uint4>(lds + ab_off + (nloc0 + 32 * j + 8 * g) * 4);
        ab[g][0] = __uint_as_float(t.x); ab[g][1] = __uint_as_float(t.y);
        ab[g][2] = __uint_as_float(t.z); ab[g][3] = __uint_as_float(t.w);
      }
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) ab[g][q] = p.alpha * bias[j][g][q];
    }
    if (res_off >= 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) unpack4(lds_load<raw_t>(lds_at(res_off, j, g)), rs[g]);
    } else if (p.res) {
      raw_t r[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) r[g] = *(const raw_t*)((const T*)p.res + o[j][g]);
#pragma unroll
      for (int g = 0; g < 4; ++g) unpack4(r[g], rs[g]);
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) rs[g][q] = 0.f;
    }
    if (p.maskbits) {
      keep = mbits ? mbits[j] : load_bits32(p.maskbits, pix, p.ldy, nwave0 + 32 * j, valid);
    } else if (p.mask) {
      raw_t mk[4];
#pragma unroll
      for (int g = 0; g < 4; ++g)
        mk[g] = mask_off >= 0 ? lds_load<raw_t>(lds_at(mask_off, j, g)) : *(const raw_t*)((const T*)p.mask + o[j][g]);
      keep = 0;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bool pos[4];
        positive4(mk[g], pos);
#pragma unroll
        for (int q = 0; q < 4; ++q) keep |= (pos[q] ? 1u : 0u) << (8 * g + 4 * half + q);
      }
    }

    // ---- arithmetic: v = alpha * acc + alpha * bias + res, clamp below at 0 (ReLU) or -inf, apply the mask.
    // The optional parts (residual, mask, sign bits) sit behind wave-uniform branches that hold arithmetic only:
    // the epilogue's vector instructions compete with the MFMAs of the workgroup that shares the CU, and a
    // launch that needs none of them runs 5 instead of 12 instructions per output.
    float v[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[g][q] = fmaf(p.alpha, acc[j][i][4 * g + q], ab[g][q]);
    if (res_off >= 0 || p.res) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) v[g][q] += rs[g][q];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[g][q] = __builtin_amdgcn_fmed3f(v[g][q], lower, __builtin_inff());  // one instruction; NaN -> lower
    if (p.maskbits || p.mask) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q)  // bit -> 0 / all ones, then and
          v[g][q] = __uint_as_float(__float_as_uint(v[g][q]) & (uint32_t)__builtin_amdgcn_sbfe((int)keep, 8 * g + 4 * half + q, 1));
    }
    if (p.bits_out) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) signs |= (v[g][q] > 0.f ? 1u : 0u) << (4 * (4 * j + g) + q);
    }

    // ---- store: into the LDS output tile (same layout as the staged residual tile, possibly the very
    // same bytes: this lane has read its residual values from them already; the workgroup writes the
    // tile out afterwards in whole rows), or straight to global memory
    if (out_off >= 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (sizeof(T) == 2) {
          u32x2_t t = {pack_bf16(v[g][0], v[g][1]), pack_bf16(v[g][2], v[g][3])};
          *(u32x2_t DDS_LDS_AS*)(lds_at(out_off, j, g)) = t;
        } else {
          u32x4_t t = {__float_as_uint(v[g][0]), __float_as_uint(v[g][1]), __float_as_uint(v[g][2]), __float_as_uint(v[g][3])};
          *(u32x4_t DDS_LDS_AS*)(lds_at(out_off, j, g)) = t;
        }
      }
    } else if (p.out_f32) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (ok[j][g]) store4<float>(p.y, o[j][g], v[g]);
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (ok[j][g]) store4<T>(p.y, o[j][g], v[g]);
    }
  }

  // ---- sign plane of the stored values
  if (p.bits_out) {
    // the other half of the wave holds the other four channels of every byte
    const uint32_t other = (uint32_t)__shfl_xor((int)signs, 32, 64);
    const uint32_t lo = half ? other : signs, hi = half ? signs : other;
    // half h writes word j = h (both halves hold all nibbles now); with NJ == 1 only half 0 writes
    const int jw = half;
    if (jw < NJ && valid) {
      const uint32_t w = spread_nibbles((lo >> (16 * jw)) & 0xffffu) | (spread_nibbles((hi >> (16 * jw)) & 0xffffu) << 4);
      store_bits32(p.bits_out, pix, p.ldy, nwave0 + 32 * jw, w);
    }
  }
}

// ------------------------------------------------------------------ forward / dgrad
// S2 (dgrad of a stride-2 convolution whose channel count is a multiple of the k-tile): the
// output pixels are dealt to workgroups by parity class (h % 2, w % 2), blockIdx.x =
// class * tiles_per_class + tile. A pixel of class (ch, cw) only receives taps r = ch + pad,
// s = cw + pad (mod 2), so a workgroup walks just those taps: on average 2.25 of the 9 taps
// of a 3x3 kernel, and 1 class in 4 has any tap at all for a 1x1 kernel.
template <typename T, int BM, int BN, int WM, int WN, int BKB, bool DGRAD, bool S2 = false>
__global__ __launch_bounds__(256, 2) void conv_gemm_kernel(ConvParams p_, int tiles_per_class) {
  ConvParams p = p_;
  constexpr int ES = sizeof(T);
  constexpr int CE = 16 / ES;     // elements per 16-byte chunk
  constexpr int BKE = BKB / ES;   // k elements per tile
  constexpr int CPR = BKB / 16;   // chunks per tile row
  constexpr int LDK = BKB + 16;
  constexpr int ROWS = 256 / CPR; // rows covered by one pass of all threads
  // loader passes over the A and B tiles; a B tile of fewer rows than one pass (BN < ROWS) leaves the
  // threads past its last row idle (their loads read row 0 and are not stored)
  constexpr int AP = BM / ROWS, BP = BN >= ROWS ? BN / ROWS : 1;
  static_assert((BM / WM) * (BN / WN) == 4, "four waves");
  static_assert(AP >= 1, "tile too small for the loader");
  __shared__ __align__(16) char smem[2 * (BM + BN) * LDK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave % (BM / WM), wave_n = wave / (BM / WM);
  const int cls = S2 ? blockIdx.x / tiles_per_class : 0;
  const int ch = cls >> 1, cw = cls & 1;
  const int Hc = (p.Ho - ch + 1) >> 1, Wc = (p.Wo - cw + 1) >> 1;  // pixels of this class per image column / row
  const int Mc = S2 ? p.Nimg * Hc * Wc : p.M;
  const int m0 = (S2 ? blockIdx.x - cls * tiles_per_class : blockIdx.x) * BM, n0 = blockIdx.y * BN;
  if (p.nrep > 1) {  // the launcher made sure that a tile never straddles two data-groups
    const int rows_per_rep = Mc / p.nrep;
    const int r = min(m0 / rows_per_rep, p.nrep - 1);
    p.w = (const char*)p.w + (size_t)r * p.w_rep;
    if (p.bias) p.bias += (size_t)r * p.bias_rep;
    if (p.w2) p.w2 = (const char*)p.w2 + (size_t)r * p.w2_rep;
  }
  const int chunk = tid % CPR, rbase = tid / CPR;
  const int sh = p.stride - 1;  // stride is 1 or 2
  // row of the tile -> output pixel (image, oh, ow) and its flat index
  auto row_pixel = [&](int m, int& img, int& oh, int& ow) {
    if (S2) {
      const int HW = Hc * Wc;
      img = m / HW;
      const int rem = m - img * HW;
      const int h2 = rem / Wc;
      oh = 2 * h2 + ch;
      ow = 2 * (rem - h2 * Wc) + cw;
    } else {
      const int HoWo = p.Ho * p.Wo;
      img = m / HoWo;
      const int rem = m - img * HoWo;
      oh = rem / p.Wo;
      ow = rem - oh * p.Wo;
    }
  };

  int a_h[AP], a_w[AP], a_img[AP];
  const char* a_base[AP];
  bool a_ok[AP];
#pragma unroll
  for (int i = 0; i < AP; ++i) {
    int m = m0 + rbase + i * ROWS;
    a_ok[i] = m < Mc;
    int mm = a_ok[i] ? m : 0;
    int img, oh, ow;
    row_pixel(mm, img, oh, ow);
    a_img[i] = img;
    if (DGRAD) { a_h[i] = oh + p.pad; a_w[i] = ow + p.pad; }
    else { a_h[i] = oh * p.stride - p.pad; a_w[i] = ow * p.stride - p.pad; }
    a_base[i] = (const char*)p.x + (size_t)img * p.H * p.W * p.Cx * ES;
  }
  const char* b_base[BP];
  bool b_ok[BP];
  int b_n[BP];
#pragma unroll
  for (int i = 0; i < BP; ++i) {
    int n = n0 + rbase + i * ROWS;
    b_n[i] = n;
    b_ok[i] = n < p.Nout && rbase + i * ROWS < BN;
    b_base[i] = (const char*)p.w + (size_t)(b_ok[i] ? n : 0) * p.Ktot * ES;
  }
  // position of this thread's chunk in (tap, channel) space
  int kc = chunk * CE, kr = 0, ks = 0, kflat = chunk * CE;
  while (kc >= p.Cx) { kc -= p.Cx; if (++ks == p.S) { ks = 0; ++kr; } }

  // Loads are unconditional (out-of-range taps read the tensor base and are zeroed when
  // parked in LDS): a branch around a load would make the compiler drain every
  // outstanding load at each use.
  uint4 ra[AP], rb[BP];
  bool oka[AP], okb[BP];
  auto load_global = [&]() {
#pragma unroll
    for (int i = 0; i < AP; ++i) {
      int hi, wi;
      bool ok;
      if (DGRAD) {
        int nh = a_h[i] - kr, nw = a_w[i] - ks;
        ok = nh >= 0 && nw >= 0 && ((nh | nw) & sh) == 0;
        hi = nh >> sh; wi = nw >> sh;
        ok = ok && hi < p.H && wi < p.W;
      } else {
        hi = a_h[i] + kr; wi = a_w[i] + ks;
        ok = (unsigned)hi < (unsigned)p.H && (unsigned)wi < (unsigned)p.W;
      }
      ok = ok && a_ok[i] && kr < p.R;
      oka[i] = ok;
      const size_t off = ok ? ((size_t)(hi * p.W + wi) * p.Cx + kc) * ES : 0;
      ra[i] = *(const uint4*)(a_base[i] + off);
    }
#pragma unroll
    for (int i = 0; i < BP; ++i) {
      okb[i] = b_ok[i] && kflat < p.Ktot;
      rb[i] = *(const uint4*)(b_base[i] + (size_t)(okb[i] ? kflat : 0) * ES);
    }
    kflat += BKE;
    kc += BKE;
    while (kc >= p.Cx) { kc -= p.Cx; if (++ks == p.S) { ks = 0; ++kr; } }
  };
  // extra reduction steps of a folded 1x1 stride-2 shortcut (class (0, 0) only): same pixel as the
  // centre tap, other tensor and weights
  int k2 = chunk * CE;
  auto load_global2 = [&]() {
#pragma unroll
    for (int i = 0; i < AP; ++i) {
      const int hi = (a_h[i] - p.pad) >> 1, wi = (a_w[i] - p.pad) >> 1;
      oka[i] = a_ok[i];
      const size_t off = oka[i] ? ((size_t)(hi * p.W + wi) * p.Cx2 + k2) * ES : 0;
      ra[i] = *(const uint4*)((const char*)p.x2 + (size_t)a_img[i] * p.H * p.W * p.Cx2 * ES + off);
    }
#pragma unroll
    for (int i = 0; i < BP; ++i) {
      okb[i] = b_ok[i];
      rb[i] = *(const uint4*)((const char*)p.w2 + ((size_t)(b_ok[i] ? b_n[i] : 0) * p.Cx2 + k2) * ES);
    }
    k2 += BKE;
  };
  auto store_lds = [&](int buf) {
    char* As = smem + buf * (BM + BN) * LDK;
    char* Bs = As + BM * LDK;
#pragma unroll
    for (int i = 0; i < AP; ++i) *(uint4*)(As + (rbase + i * ROWS) * LDK + chunk * 16) = keep_if(oka[i], ra[i]);
#pragma unroll
    for (int i = 0; i < BP; ++i)
      if (BN >= ROWS || rbase + i * ROWS < BN) *(uint4*)(Bs + (rbase + i * ROWS) * LDK + chunk * 16) = keep_if(okb[i], rb[i]);
  };

  f32x16_t acc[WN / 32][WM / 32];
#pragma unroll
  for (int j = 0; j < WN / 32; ++j)
#pragma unroll
    for (int i = 0; i < WM / 32; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;

  // S2: taps of the wrong parity are stepped over whole (Cx / BKE k-tiles at a time; the
  // position is the same for every thread of the workgroup up to the chunk offset)
  const int tiles_per_tap = S2 ? p.Cx / BKE : 1;
  auto tap_live = [&]() { return ((ch + p.pad - kr) & 1) == 0 && ((cw + p.pad - ks) & 1) == 0; };
  auto skip_dead_taps = [&]() {
    if (S2) {
      while (kr < p.R && !tap_live()) {
        kflat += p.Cx;
        if (++ks == p.S) { ks = 0; ++kr; }
      }
    }
  };
  int nk = (p.Ktot + BKE - 1) / BKE;
  if (S2) {
    int nr = 0, ns = 0;
    for (int r = 0; r < p.R; ++r) nr += ((ch + p.pad - r) & 1) == 0;
    for (int q = 0; q < p.S; ++q) ns += ((cw + p.pad - q) & 1) == 0;
    nk = nr * ns * tiles_per_tap;
  }
  const int nk1 = nk;  // k-tiles of the layer itself; the folded shortcut follows
  if (S2 && p.x2 != nullptr && cls == 0) nk += p.Cx2 / BKE;
  auto load_tile = [&](int kt) {
    if (S2 && kt >= nk1) {
      load_global2();
    } else {
      skip_dead_taps();
      load_global();
    }
  };
  if (nk > 0) {
    load_tile(0);
    store_lds(0);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load_tile(kt + 1);
    const char* As = smem + buf * (BM + BN) * LDK + wave_m * WM * LDK;
    const char* Bs = smem + buf * (BM + BN) * LDK + BM * LDK + wave_n * WN * LDK;
    // weights are the MFMA A operand so that a lane ends up with 4 consecutive output
    // channels of one pixel (one vector access per operand in the epilogue)
    mma_step<T, WN, WM, BKB>(Bs, As, lane, acc);
    if (kt + 1 < nk) store_lds(buf ^ 1);
    __syncthreads();
  }

  // lane holds pixel m = lane%32 and channels 8*g + 4*(lane/32) + (0..3), g = 0..3, of each 32x32 tile
  const int nb = n0 + wave_n * WN + 4 * (lane >> 5);
  float bias[WN / 32][4][4];
  load_bias_groups<WN / 32>(p, nb, bias);
#pragma unroll
  for (int i = 0; i < WM / 32; ++i) {
    const int m = m0 + wave_m * WM + i * 32 + (lane & 31);
    size_t pix = (size_t)m;
    if (S2) {
      int img, oh, ow;
      row_pixel(m < Mc ? m : 0, img, oh, ow);
      pix = ((size_t)img * p.Ho + oh) * p.Wo + ow;
    }
    epilogue_tile<T, WN / 32, WM / 32>(p, acc, i, m < Mc, pix, nb, bias);
  }
}

// ------------------------------------------------------------------ 3x3 stride-1 forward / dgrad, asynchronous LDS fills
// The workgroup owns BM consecutive pixels of the flattened (image, row, column) index and BN output channels. In that
// index the nine taps of a pixel are the pixels at distance -W-1 .. W+1, so the input patch of a tile is BM + 2W + 2
// consecutive pixels whatever the image size: its copies are contiguous, need no table and no division, and no tile
// holds padding (a rectangle of 8 x 32 pixels plus halo is 340 rows and fits few image sizes; four 8 x 8 images with
// their halos are 400 rows against 274). Taps that leave the image read a block of zeros instead: one lane mask per
// image edge and fragment, combined on the scalar unit. Per KB-byte channel chunk the patch is staged in LDS ONCE and
// all nine taps read their MFMA operands from it at shifted rows. Every operand byte travels global -> LDS
// with global_load_lds_dwordx4 (no staging registers, lane L of a wave fills bytes
// [16L, 16L+16) of a 1 KiB LDS block), issued two pipeline stages (tap, channel chunk)
// ahead of its use: weight tiles rotate through three LDS slots and the next channel
// chunk's patch is fetched in slices spread over taps 0..6 of the current one. The
// compiler does not model these copies, so their completion is counted by hand: loads
// retire in order, every stage issues a fixed number per lane, and each stage waits
// until only the younger ones are outstanding, then crosses one workgroup barrier.
// LDS rows are KB unpadded bytes; the 16-byte column c of row r lives at column c ^ f(r), f(r) = (r * KB / 256) mod
// (KB/16), applied by choosing which global column a lane fetches. A 16-byte-per-lane LDS read is
// served 16 lanes per cycle from 64 four-byte banks, and the 16 lanes of one cycle are the
// four-lane quads q = lane/4 of a 32-lane half whose index has even (or odd) bit parity:
// {0,3,5,6} and {1,2,4,7} (measured). Any 16 consecutive rows hit 16 different 16-byte bank groups under f; the
// pixels of a 32-pixel fragment are dealt to lanes so that one cycle's lanes hold 16 consecutive ones, and a lane
// whose tap is outside the image reads the zero block at the bank group it would have used.
// Bound by the matrix unit and by one barrier per stage. Measured against rectangular tiles with halos (only images
// whose sides are powers of two; 8 x 32 pixels + halo), alone: 512 images of 32 x 32 x 64 58.9 -> 56.5 us, 128 -> 128
// channels at 16 x 16 unchanged at 45 us (860 TFLOP/s); per 8 iterations ResNet-20 in one module 5.77 -> 5.55 ms,
// ResNet-56 23.0 -> 22.5 ms, and 28 x 28 images, which ran on conv_gemm_kernel, 3.08 -> 2.72 ms.
// End of a workgroup of the asynchronous kernels: every copy has landed in this wave, acc holds its WM x WN tile.
// The residual / mask tiles are staged in the first `room` bytes of LDS (the operand buffers are free now) so that the
// epilogue pays one global round trip instead of one per 32-pixel column, and the output tile leaves from there in
// whole rows. The 1 KiB behind them holds alpha * bias. pixel(row): output pixel of a tile row, -1 past the end.
// act (wave-uniform): false for waves beyond the tile's own, which only keep the barriers.
template <typename T, int BM, int BN, int WM, int WN, typename Pixel>
__device__ __forceinline__ void tile_out(const ConvParams& p, const f32x16_t (&acc)[WN / 32][WM / 32],
                                         const uint32_t (&mb)[WM / 32][WN / 32], char* smem, int room, int n0, int wave,
                                         int wave_m, int wave_n, int lane, int lpix, Pixel pixel, bool act = true) {
  constexpr int ES = sizeof(T);
  constexpr int NW = (BM / WM) * (BN / WN), NI = WM / 32, NJ = WN / 32;
  constexpr int ROWB = BN * ES;        // bytes per tile row
  constexpr int NCOL = ROWB / 16;      // 16-byte columns per row
  constexpr int RPF = 64 / NCOL;       // rows per wave fill
  constexpr int FPW = BM / RPF / NW;    // fills per wave
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  int res_off = -1, mask_off = -1, nregions = 0;
  const int ab_off = room;
  float* ab_lds = (float*)(smem + ab_off);
  wg_barrier();
  if ((int)threadIdx.x < BN) {
    const int n = n0 + threadIdx.x;
    ab_lds[threadIdx.x] = (p.bias != nullptr && n < p.Nout) ? p.alpha * p.bias[n] : 0.f;
  }
  if (p.res || p.mask) {
    int region = 0;
    auto stage_tile = [&](const void* src_tensor) -> int {
      if ((region + 1) * BM * ROWB > room) return -1;
      const int rbase = region * BM * ROWB;
      if (act)
#pragma unroll
      for (int u = 0; u < FPW; ++u) {
        const int f = wave + NW * u;
        const int row = f * RPF + lane / NCOL, slot = lane % NCOL;
        const int gc = (slot ^ row) & (NCOL - 1);
        const int n = n0 + gc * (16 / ES);
        const int pix = pixel(row);
        const bool ok = pix >= 0 && n < p.ldy;
        const char* src = ok ? (const char*)src_tensor + ((size_t)pix * p.ldy + n) * ES : (const char*)p.zeros;
        dma16(src, lds0 + rbase + f * 1024);
      }
      ++region;
      return rbase;
    };
    if (p.mask) mask_off = stage_tile(p.mask);
    if (p.res) res_off = stage_tile(p.res);
    wait_vm<0>();
    nregions = region;
  }
  // Output tile in LDS: the residual tile's bytes if there is one, else the next free region.
  int out_off = res_off >= 0 ? res_off : ((nregions + 1) * BM * ROWB <= room ? nregions * BM * ROWB : -1);
  if (p.out_f32) out_off = -1;
  __syncthreads();  // also orders the plain LDS stores of alpha * bias

  const int nb = n0 + wave_n * WN + 4 * (lane >> 5);
  float bias[NJ][4][4] = {};
  if (act)
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = wave_m * WM + i * 32 + lpix;
    const int pix = pixel(m);
    epilogue_tile<T, NJ, NI>(p, acc, i, pix >= 0, (size_t)max(pix, 0), nb, bias, (const char DDS_LDS_AS*)smem, res_off, mask_off, m, ROWB,
                             wave_n * WN + 4 * (lane >> 5), ab_off, mb[i], out_off);
  }
  if (out_off >= 0) {
    // write the tile out: a wave stores RPF whole tile rows per instruction, 16 bytes per lane
    __syncthreads();
    if (act)
#pragma unroll
    for (int u = 0; u < FPW; ++u) {
      const int f = wave + NW * u;
      const int row = f * RPF + lane / NCOL, slot = lane % NCOL;
      const int gc = (slot ^ row) & (NCOL - 1);
      const int n = n0 + gc * (16 / ES);
      const int pix = pixel(row);
      const u32x4_t v = *(const u32x4_t DDS_LDS_AS*)((const char DDS_LDS_AS*)smem + out_off + f * 1024 + lane * 16);
      if (pix >= 0 && n < p.ldy) *(u32x4_t*)((char*)p.y + ((size_t)pix * p.ldy + n) * ES) = v;
    }
  }
}

// The two halves of a workgroup's waves hold partial sums of the same tile: the second half's meet the first half's in
// LDS (4 KiB per 32 x 32 block and wave, at the start of LDS) and end there.
template <int NI, int NJ>
__device__ __forceinline__ void add_halves(f32x16_t (&acc)[NJ][NI], char* smem, int khalf, int wave, int lane) {
  __syncthreads();  // the operands have been read
  f32x16_t* buf = (f32x16_t*)smem + (size_t)wave * NJ * NI * 64 + lane;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (khalf == 1) buf[(j * NI + i) * 64] = acc[j][i];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (khalf == 0) acc[j][i] += buf[(j * NI + i) * 64];
}

constexpr int kPartsRow = 96;  // bytes of a pixel's sixteen channels, split: three rows of 32 bytes

struct DmaGeom {
  int patch_rows;   // BM + 2W + 2 rounded up to whole wave fills
  int out_bytes;    // bytes of LDS the epilogue may stage tiles in (everything below the dump block)
  int dgrad;        // tap (r, s) reads the patch at distance (1-r, 1-s) instead of (r-1, s-1)
  Divisor dW, dH;
};

// fp32 (but RES): a workgroup splits the patch once a chunk (split3), into rows of three 32-byte parts that all nine taps read, and every wave
// the weights of its own 32 channels as it reads them. Eight waves; a vector instruction in three of four MFMA cycles is hidden, more add up, so waves
// are 128 pixels tall (24 MFMAs for one fragment of weights) wherever the launch still fills the chip: 256 x 128 tiles of the fp32 CNN's layers against
// 128 x 128 ones of 64 x 32 a wave 10840 -> 9100 us per 8 steps. us a launch, fp32 unit / here, 19.3 GFLOP each: 155 / 111 (256 tiles
// of 128 x 128), 157 / 100, 166 / 117 (256 x 128, 256 and 512 tiles), 150 / 98 (512 x 64), 285 / 190 (128 tiles). The patch split by each wave as it read
// it: 128 us where this takes 111. Bound by matrix and vector unit, which take turns (766 and 720 cycles of 1400 a stage of 128 x 128).
// RES (one channel chunk only): the weights of all nine taps are resident beside the patch, so everything is requested
// at once and the taps run without a barrier between them.
// KS = 2: eight waves, each four of which have operand buffers of their own and walk half of the channel chunks.
template <typename T, int BM, int BN, int WM, int WN, int PS, int KB, bool RES = false, int KS = 1>
__global__ __launch_bounds__(64 * KS * (BM / WM) * (BN / WN), sizeof(T) == 4 && WM < 128 ? 4 : 2) void conv3x3_dma_kernel(ConvParams p_, DmaGeom g) {
  ConvParams p = p_;
  constexpr int ES = sizeof(T);
  constexpr int NW = (BM / WM) * (BN / WN);  // waves per workgroup (each owns a WM x WN sub-tile)
  constexpr int FROWS = 1024 / KB;     // LDS rows per wave fill (KB = bytes of channels per row: 64 or 128)
  constexpr int CPR = KB / 16;         // 16-byte columns per row
  constexpr int RG = BN / FROWS;       // fills of a weight tile (one tap, one chunk)
  constexpr int WL = RG >= NW ? RG / NW : 1;  // weight fills per lane per stage
  constexpr int NKS = KB / 32;         // MFMA k-steps per stage
  constexpr int RPL = KB == 128 ? 1 : 2;  // log2(rows per 256 bytes of LDS)
  static_assert(KB == 64 || KB == 128, "row depth");
  static_assert(RES ? PS == 0 && (RG >= NW || (RG % 2 == 0 && NW % RG == 0)) : RG >= NW || NW == 2 * RG, "fills of a weight tile per wave");
  constexpr int NI = WM / 32, NJ = WN / 32;
  static_assert((NW == 4 || (NW == 8 && ES == 4 && !RES)) && (KS == 1 || (KS == 2 && !RES)), "waves per tile");
  constexpr bool PLANES = ES == 4 && !RES;  // the patch is split once a chunk, into rows of three 32-byte parts behind it
  static_assert(!PLANES || (KB == 64 && KS == 1), "sixteen channels a chunk");
  extern __shared__ __align__(16) char smem[];
  const int prow = g.patch_rows;
  const int pbuf_bytes = prow * KB;
  const int wring_off = PLANES ? prow * (KB + kPartsRow) : (PS > 0 ? 2 : 1) * pbuf_bytes;
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const uint32_t lds_dump = lds0 + g.out_bytes;   // 1 KiB that absorbs surplus fills
  const int zero_off = g.out_bytes + 1024;        // 256 bytes of zeros
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: everything derived from it stays in SGPRs
  const int wave = wave_wg & (NW - 1), khalf = wave_wg / NW;
  const int buf0 = KS > 1 ? khalf * (wring_off + 3 * BN * KB) : 0;  // operand buffers of this half
  char* wring = smem + buf0 + wring_off;
  const uint32_t lds_pbuf = lds0 + buf0, lds_wring = lds_pbuf + wring_off;
  const int wave_m = wave % (BM / WM), wave_n = wave / (BM / WM);
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  if (p.nrep > 1) {  // the launcher made sure that the pixels of a tile belong to one data-group
    const int r = min(m0 / (p.M / p.nrep), p.nrep - 1);
    p.w = (const char*)p.w + (size_t)r * p.w_rep;
    if (p.bias) p.bias += (size_t)r * p.bias_rep;
  }
  const int nchunks = (p.Cx * ES) / KB / KS;  // channel chunks of this half
  const size_t pixbytes = (size_t)p.Cx * ES;
  const size_t chunk0 = (size_t)khalf * nchunks * KB;
  if (tid < (PLANES ? 32 : 16)) *(uint4*)(smem + zero_off + tid * 16) = make_uint4(0u, 0u, 0u, 0u);

  const int l8 = lane / CPR;  // row inside a fill
  const int pcol = lane % CPR;
  // global 16-byte column this lane fetches: (row / 2^RPL) mod CPR of a row whose fill index has the wave's parity
  const uint32_t c16 = (uint32_t)((pcol ^ (((l8 + (wave & 1) * FROWS) >> RPL) & (CPR - 1))) * 16);
  const int pw_total = prow / FROWS;  // wave fills in a patch
  // Patch fills of this wave: byte offset from the patch's first row. Rows before the tensor's first or after its
  // last pixel repeat that pixel (no tap inside an image reads them).
  constexpr int NPRO = (KB == 128 && PS == 0) ? 11 : 7;  // fills per wave that cover the largest patch
  const int first = m0 - p.W - 1;  // pixel of patch row 0
  const char* pbase = (const char*)p.x + (long long)first * (long long)pixbytes + chunk0;
  uint32_t poff[NPRO];
#pragma unroll
  for (int j = 0; j < NPRO; ++j) {
    const int row = (wave + NW * j) * FROWS + l8;
    poff[j] = (uint32_t)(min(max(row, -first), p.M - 1 - first)) * (uint32_t)pixbytes + c16;
  }
  auto patch_dst = [&](int j, int buf) {
    const int wl = wave + NW * j;
    return wl < pw_total ? lds_pbuf + (PLANES ? 0 : buf * pbuf_bytes) + wl * 1024 : lds_dump;
  };
  // weight rows: byte offset of this lane's 16 bytes inside the weight tensor at tap 0, chunk 0.
  // Rows past Nout repeat the last one: their output columns lie past ldy == Nout and are never stored.
  uint32_t wvo[WL];
#pragma unroll
  for (int u = 0; u < WL; ++u) {
    const int gn = n0 + (wave % RG + NW * u) * FROWS + l8;
    wvo[u] = (uint32_t)(gn < p.Nout ? gn : p.Nout - 1) * (uint32_t)(9 * pixbytes) + c16;
  }
  auto fill_w = [&](int chunk, int tap, int slot) {
    const char* base = (const char*)p.w + (size_t)tap * pixbytes + chunk0 + (size_t)chunk * KB;  // wave-uniform
#pragma unroll
    for (int u = 0; u < WL; ++u) dma16s(base, wvo[u], lds_wring + slot * (BN * KB) + (wave % RG + NW * u) * 1024);  // (twice the same where two waves share a fill)
  };

  // pixel of the 32-pixel fragment held by this lane: quads {0,3,5,6} -> pixels 0..15, {1,2,4,7} -> 16..31
  const int lq = (lane >> 2) & 7;
  const int lpix = ((__builtin_popcount(lq) & 1) << 4) | ((lq >> 1) << 2) | (lane & 3);
  // dgrad through a ReLU: the sign bits of this lane's outputs are fetched now (a few bytes per
  // pixel, the oldest loads of the kernel) so that the epilogue reads nothing but the accumulators
  uint32_t mb[NI][NJ] = {};
  if (p.maskbits) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int pix = m0 + wave_m * WM + i * 32 + lpix;
#pragma unroll
      for (int j = 0; j < NJ; ++j) mb[i][j] = load_bits32(p.maskbits, (size_t)pix, p.ldy, n0 + wave_n * WN + 32 * j, pix < p.M);
    }
  }

  // prologue: whole first patch, then the weight tiles of stages 0 and 1. Issued before the rest of
  // the set-up (fragment addresses, edge masks, accumulators) so that it runs under the copies' latency.
#pragma unroll
  for (int j = 0; j < NPRO; ++j)
    if (wave + NW * j < pw_total) dma16s(pbase, poff[j], patch_dst(j, 0));
  if (!RES) {
    fill_w(0, 0, 0);
    fill_w(0, 1, 1);
  } else if (RG >= NW) {
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) fill_w(0, tap, tap);
  } else {  // a tile is less than a fill per wave: the waves take the fills of consecutive taps
#pragma unroll
    for (int u = 0; u < (9 * RG + NW - 1) / NW; ++u) {
      const int f = wave + NW * u;
      if (f < 9 * RG) dma16s((const char*)p.w + (size_t)(f / RG) * pixbytes, wvo[0], lds_wring + f * 1024);
    }
  }

  // fragment addressing
  const int half = lane >> 5;
  // Patch operand of tap (r, s): row * KB + ((half ^ f(row)) << 4), row = tile pixel + (W + 1) +- ((r-1) W + (s-1))
  int rowb[NI];
  // is the neighbour that tap row 0 / 2 and tap column 0 / 2 read inside the image
  bool ok_r0[NI], ok_r2[NI], ok_s0[NI], ok_s2[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = wave_m * WM + i * 32 + lpix;
    rowb[i] = PLANES ? m + p.W + 1 : (m + p.W + 1) * KB + half * 16;
    const uint32_t pix = (uint32_t)(m0 + m);
    const int line = (int)(__umulhi(pix, g.dW.mul) >> g.dW.shift), w = (int)pix - line * p.W;
    const int h = line - (int)(__umulhi((uint32_t)line, g.dH.mul) >> g.dH.shift) * p.H;
    const bool up = h > 0, down = h < p.H - 1, left = w > 0, right = w < p.W - 1;
    ok_r0[i] = g.dgrad ? down : up;
    ok_r2[i] = g.dgrad ? up : down;
    ok_s0[i] = g.dgrad ? right : left;
    ok_s2[i] = g.dgrad ? left : right;
  }
  constexpr int ROW = PLANES ? 1 : KB;  // unit of rowb
  const int tap_w = (g.dgrad ? -p.W : p.W) * ROW, tap_1 = g.dgrad ? -ROW : ROW;
  int boff[NJ][NKS];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = wave_n * WN + j * 32 + (lane & 31);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) boff[j][ks] = n * KB + (((PLANES ? 2 * half + ks : 2 * ks + half) ^ ((n >> RPL) & (CPR - 1))) << 4);
  }
  f32x16_t acc[NJ][NI];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;

  // LDS offsets of this lane's patch operands at the tap about to be multiplied. They are formed behind the MFMAs of
  // the previous tap, before the barrier: after it only the LDS reads stand between a stage and its first MFMA.
  int a0[NI];
  auto address = [&](int chunk, int tap_r, int tap_s) {
    const int tapoff = (tap_r - 1) * tap_w + (tap_s - 1) * tap_1;  // wave-uniform
    const int pbuf = buf0 + (PS > 0 ? (chunk & 1) * pbuf_bytes : 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int rb = rowb[i];
      asm volatile("" : "+v"(rb));  // keeps the nine taps' addresses from being precomputed (and spilled)
      const int t = rb + tapoff;    // row * KB + half * 16; f(row) = bits 8.. of it
      const int a = PLANES ? (int)__umul24(t, kPartsRow) + pbuf_bytes + (((t >> 3 ^ half) & 1) << 4) : (t ^ ((t >> 4) & ((CPR - 1) << 4))) + pbuf;
      if (tap_r == 1 && tap_s == 1) {
        a0[i] = a;
      } else {
        const bool okr = tap_r == 0 ? ok_r0[i] : tap_r == 2 ? ok_r2[i] : true;
        const bool oks = tap_s == 0 ? ok_s0[i] : tap_s == 2 ? ok_s2[i] : true;
        a0[i] = okr && oks ? a : ((a & 0xf0) | zero_off);
      }
      asm volatile("" : "+v"(a0[i]));
    }
  };
  // fp32: sums of a chunk, which join the long ones behind its last tap
  f32x16_t inner[PLANES ? NJ : 1][PLANES ? NI : 1] = {};
  auto fold = [&]() {
    if constexpr (PLANES)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          acc[j][i] += inner[j][i];
          inner[j][i] = f32x16_t{};
        }
  };
  auto compute = [&](int slot) {
    const char* wb = wring + slot * (BN * KB);
    if constexpr (PLANES) {
      uint4 b[NJ][2];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int k = 0; k < 2; ++k) b[j][k] = *(const uint4*)(wb + boff[j][k]);
      constexpr int G = NI < 2 ? NI : 2;  // blocks of pixels at a time
      Parts a[G];
      auto read_a = [&](int i0) {
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
          for (int k = 0; k < 3; ++k) a[i].part[k] = *(const uint4*)(smem + a0[i0 + i] + 32 * k);
      };
      Parts w[NJ];
      read_a(0);
#pragma unroll
      for (int j = 0; j < NJ; ++j) w[j] = split3(b[j][0], b[j][1]);
#pragma unroll
      for (int i0 = 0; i0 < NI; i0 += G) {
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < G; ++i) mfma16B<bf16_t>(w[j].part[kPartA[k]], a[i].part[kPartB[k]], inner[j][i0 + i]);
        if (i0 + G < NI) read_a(i0 + G);
      }
      return;
    } else if constexpr (ES == 4) {
#pragma unroll
      for (int k2 = 0; k2 < NKS; k2 += 2) {
        uint4 a[NI][2], b[NJ][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
          for (int i = 0; i < NI; ++i) a[i][k] = *(const uint4*)(smem + (a0[i] ^ ((k2 + k) << 5)));
#pragma unroll
          for (int j = 0; j < NJ; ++j) b[j][k] = *(const uint4*)(wb + boff[j][k2 + k]);
        }
        Parts w[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) w[j] = split3(b[j][0], b[j][1]);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          f32x16_t* sums[NJ];
#pragma unroll
          for (int j = 0; j < NJ; ++j) sums[j] = &acc[j][i];
          mfma_split<NJ>(split3(a[i][0], a[i][1]), w, sums);
        }
      }
      return;
    }
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      uint4 a[NI], b[NJ];
#pragma unroll
      for (int i = 0; i < NI; ++i) a[i] = *(const uint4*)(smem + (a0[i] ^ (ks << 5)));
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[j] = *(const uint4*)(wb + boff[j][ks]);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) mfma16B<T>(b[j], a[i], acc[j][i]);
    }
  };

  auto split_patch = [&]() {
    for (int u = tid; u < 2 * prow; u += 64 * NW) {
      const int r = u >> 1, h = u & 1;
      const char* from = smem + r * KB;
      const int f = (r >> RPL) & (CPR - 1);
      const Parts t = split3(*(const uint4*)(from + (((2 * h) ^ f) << 4)), *(const uint4*)(from + (((2 * h + 1) ^ f) << 4)));
#pragma unroll
      for (int k = 0; k < 3; ++k) *(uint4*)(smem + pbuf_bytes + r * kPartsRow + 32 * k + (((r >> 3 ^ h) & 1) << 4)) = t.part[k];
    }
    wg_barrier();
  };

// One stage = one tap of one channel chunk. VM = fills per lane issued after the weight
// tile this stage consumes: one weight tile plus the patch slices of the two previous stages.
#define DDS_STAGE(TAP)                                                                              \
  {                                                                                                 \
    constexpr int VM = WL + PS * (((TAP) >= 2 && (TAP) <= 8 ? 1 : 0) + ((TAP) >= 1 && (TAP) <= 7 ? 1 : 0)); \
    wait_vm<VM>();                                                                                  \
    wg_barrier();                                                                                   \
    if constexpr (PLANES && (TAP) == 0) split_patch();                                              \
    {                                                                                               \
      int ct = chunk + ((TAP) + 2 >= 9 ? 1 : 0), tt = ((TAP) + 2) % 9;                             \
      if (ct >= nchunks) { ct = nchunks - 1; tt = 8; }                                              \
      fill_w(ct, tt, ((TAP) + 2) % 3);                                                              \
    }                                                                                               \
    if (PS > 0 && (TAP) < 7) {                                                                      \
      const int cn = chunk + 1 < nchunks ? chunk + 1 : chunk;                                       \
      _Pragma("unroll") for (int u = 0; u < PS; ++u)                                                \
        dma16s(pbase + (size_t)cn * KB, poff[((TAP) < 7 ? (TAP) : 0) * PS + u], patch_dst((TAP) * PS + u, (chunk + 1) & 1)); \
    }                                                                                               \
    compute((TAP) % 3);                                                                             \
    address(chunk + ((TAP) == 8 ? 1 : 0), ((TAP) + 1) % 9 / 3, ((TAP) + 1) % 3);                    \
  }

  address(0, 0, 0);

  if (RES) {
    wait_vm<0>();
    wg_barrier();
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      compute(tap);
      if (tap < 8) address(0, (tap + 1) / 3, (tap + 1) % 3);
    }
  } else
  for (int chunk = 0; chunk < nchunks; ++chunk) {
    DDS_STAGE(0) DDS_STAGE(1) DDS_STAGE(2) DDS_STAGE(3) DDS_STAGE(4) DDS_STAGE(5) DDS_STAGE(6) DDS_STAGE(7) DDS_STAGE(8)
    fold();
  }
#undef DDS_STAGE
  wait_vm<0>();

  if constexpr (ES == 4) {
    // No part of an infinity, or of what rounds to one, is a remainder: every sum that meets one is NaN here. A workgroup that finds a NaN
    // forms its sums again on the fp32 matrix unit, from the operands as they are.
    bool nan = false;
#pragma unroll
    for (int j = 0; j < NJ; ++j) nan |= any_nan(acc[j]);
    if (workgroup_any(nan, smem + g.out_bytes, wave_wg, NW)) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;
#pragma unroll 1
      for (int t = 0; t < 9 * nchunks; ++t) {
        const int chunk = t / 9, tap = t - 9 * chunk, r = tap / 3, c = tap - 3 * r;
        if (!RES) {
          wg_barrier();
          if (tap == 0)
#pragma unroll
            for (int j = 0; j < NPRO; ++j)
              if (wave + NW * j < pw_total) dma16s(pbase + (size_t)chunk * KB, poff[j], lds_pbuf + (wave + NW * j) * 1024);
          fill_w(chunk, tap, 0);
          wait_vm<0>();
          wg_barrier();
        }
        const char* wb = wring + (RES ? tap * (BN * KB) : 0);
        const int shift = (r - 1) * tap_w / ROW + (c - 1) * tap_1 / ROW;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int row = wave_m * WM + i * 32 + lpix + p.W + 1 + shift;
          const bool in = (r == 0 ? ok_r0[i] : r == 2 ? ok_r2[i] : true) && (c == 0 ? ok_s0[i] : c == 2 ? ok_s2[i] : true);
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks) {
            const int col = PLANES ? 2 * half + ks : 2 * ks + half;  // as boff
            const uint4 a = *(const uint4*)(smem + (in ? row * KB + ((col ^ ((row >> RPL) & (CPR - 1))) << 4) : zero_off));
#pragma unroll
            for (int j = 0; j < NJ; ++j) mfma16B<float>(*(const uint4*)(wb + boff[j][ks]), a, acc[j][i]);
          }
        }
      }
    }
  }

  if (KS > 1) add_halves<NI, NJ>(acc, smem, khalf, wave, lane);
  const auto pixel = [&](int row) { return m0 + row < p.M ? m0 + row : -1; };
  tile_out<T, BM, BN, WM, WN>(p, acc, mb, smem, g.out_bytes, n0, wave, wave_m, wave_n, lane, lpix, pixel, khalf == 0);
}

inline int ilog2_exact(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return (1 << l) == v ? l : -1;
}

template <typename T, int BM, int BN, int WM, int WN, int PS, int KB, bool RES = false, int KS = 1>
bool launch_dma_inst(const ConvParams& p, hipStream_t s) {
  constexpr int FROWS = 1024 / KB;
  constexpr int NW = (BM / WM) * (BN / WN);
  if (p.Cx * (int)sizeof(T) % KB != 0) return false;
  if (p.Cx * (int)sizeof(T) / KB % KS != 0) return false;
  const int nchunks = p.Cx * (int)sizeof(T) / KB / KS;
  DmaGeom g;
  g.patch_rows = (BM + 2 * p.W + 2 + FROWS - 1) / FROWS * FROWS;
  g.dgrad = p.dgrad;
  g.dW = make_divisor(p.W);
  g.dH = make_divisor(p.H);
  const int fills_per_wave = (g.patch_rows / FROWS + NW - 1) / NW;
  if (fills_per_wave > ((KB == 128 && PS == 0) ? 11 : 7)) return false;  // patch offsets kept per lane
  if (PS == 0 ? nchunks != 1 : (nchunks * KS < 2 || 7 * PS < fills_per_wave)) return false;
  constexpr bool PLANES = sizeof(T) == 4 && !RES;
  int operands = KS * (PLANES ? g.patch_rows * (KB + kPartsRow) : (PS > 0 ? 2 : 1) * g.patch_rows * KB) + KS * (RES ? 9 : 3) * BN * KB;
  constexpr int tile = BM * BN * (int)sizeof(T);  // the output tile is staged where the operands were, if two workgroups still fit a CU
  if (operands < tile && tile <= 72 * 1024) operands = tile;
  g.out_bytes = operands;
  const int smem = operands + 1024 + (PLANES ? 512 : 256);
  if (smem > 160 * 1024) return false;
  static DeviceOnce lds;
  allow_whole_lds(lds, (const void*)conv3x3_dma_kernel<T, BM, BN, WM, WN, PS, KB, RES, KS>);
  dim3 grid((p.M + BM - 1) / BM, (p.ldy + BN - 1) / BN);
  conv3x3_dma_kernel<T, BM, BN, WM, WN, PS, KB, RES, KS><<<grid, 64 * KS * NW, smem, s>>>(p, g);
  return true;
}

// Picks the tile for the asynchronous kernel; false if the problem is outside its range.
// Channel chunks are 64 bytes deep: the LDS footprint lets two or three workgroups share a
// CU and hide each other's prologue and epilogue, and with 16 rows per wave fill a patch of
// up to 448 rows needs at most 7 fills per wave, so one slice per tap (PS = 1) is enough.
template <typename T>
bool launch_dma(const ConvParams& p, hipStream_t s) {
  constexpr int KB = 64;
  if (p.R != 3 || p.S != 3 || p.stride != 1 || p.pad != 1 || p.H != p.Ho || p.W != p.Wo || p.out_f32) return false;
  if (p.H < 2 || p.W < 2 || p.zeros == nullptr) return false;  // dividing by one is beyond make_divisor
  // pad weight rows repeat row Nout-1 (columns past ldy are not stored); per-lane patch and weight offsets are 32-bit
  if (p.ldy != p.Nout) return false;
  if ((long long)p.Nout * 9 * p.Cx * (long long)sizeof(T) >= (1ll << 31)) return false;
  const int rowbytes = p.Cx * (int)sizeof(T);
  if (rowbytes % KB != 0 || rowbytes > (1 << 20)) return false;
  const int nchunks = rowbytes / KB;
  // At most 32 output channels of one chunk: 32-column tiles (a 64-column tile multiplies and stores half padding) of 128
  // pixels with all weights resident, four workgroups a CU. 32 -> 32 channels at 16 x 16, bf16, alone: 256 images
  // 21.5 -> 14.0 us, 194 images 9.8 -> 5.4 us (256-pixel tiles: 14.2 us and 776 workgroups 11.9 against 11.5 us).
  if (p.ldy <= 32 && rowbytes == 128 && launch_dma_inst<T, 128, 32, 32, 32, 0, 128, true>(p, s)) return true;
  if (p.ldy <= 32 && nchunks == 1 && launch_dma_inst<T, 128, 32, 32, 32, 0, KB, true>(p, s)) return true;
  // 64 bf16 (32 fp32) channels in and at most 64 out: one 128-byte chunk, i.e. whole cache lines per patch row,
  // nine stages instead of eighteen and the whole patch requested in the prologue (62.0 -> 59.4 us at 32 x 32 x 64).
  // Resident weights take 74 KB, one workgroup per CU: for launches that give no CU a second one (64 -> 64 channels at
  // 8 x 8, 194 images: 11.2 -> 5.5 us; with 776 workgroups 16.4 us against 10.5 us for the 256-pixel tiles).
  if (rowbytes == 128 && p.ldy <= 64) {
    if (p.M <= 64 * 256 && launch_dma_inst<T, 64, 64, 32, 32, 0, 128, true>(p, s)) return true;
    if constexpr (sizeof(T) == 2)
      if (launch_dma_inst<T, 256, 64, 64, 64, 0, 128>(p, s)) return true;
  }
  if (nchunks == 1) {
    if constexpr (sizeof(T) == 4) {
      if (p.ldy <= 64) return launch_dma_inst<T, 256, 64, 64, 32, 0, KB>(p, s);
      return launch_dma_inst<T, 128, 128, 64, 32, 0, KB>(p, s);
    } else {
      if (p.ldy <= 64) return launch_dma_inst<T, 256, 64, 64, 64, 0, KB>(p, s);
      return launch_dma_inst<T, 256, 128, 128, 64, 0, KB>(p, s);
    }
  }
  // small images: 128-pixel tiles give more workgroups. 256-pixel tiles from 256 workgroups up (one per CU: half the
  // weight copies per FLOP; with the other modules' kernels sharing the chip this beat two 128-pixel workgroups per
  // CU at 256 channels, 2.27 vs 2.31 ms per ResNet-18 step).
  // fp32, us per 8 steps on either side of the lines: fp32 CNN, 4 groups of 128, 128 x 128 tiles / 256 x 128 and 512 x 64 ones 10840 / 9100. Images
  // of any sides (conv_gather_kernel before, whose stages re-read every pixel for each tap): 28 x 28, 2 groups of 97 4240 / 3375, 30 x 30, 3 of 150 7794 /
  // 6685, 36 x 36, 4 of 200 16989 / 14513, 9 x 9, one of 16 1700 / 1732. Launches that leave three of four CUs without a 128 x 128 or 256 x 64 tile:
  // 64 x 64 ones, four waves: fp32 CNN, one group of 8 3050 / 1900, of 32 3215 / 2065, of 80 3630 / 2735, 2 of 64 3990 / 3360, ResNet-20 at 16 6470 / 5290,
  // at 194 11650 / 10590, 9 x 9, one of 16 1725 / 1250, 20 x 20, 2 of 97 2780 / 2354; up to 32768 pixels of 64 channels ResNet-20 at 500 and 512
  // 20630 / 21130 and 20830 / 21510, up to 128 tiles of 128 x 128 the fp32 CNN at 4 x 128 8910 / 9130.
  const long long tiles256 = (long long)((p.M + 255) / 256) * ((p.ldy + 127) / 128);
  if constexpr (sizeof(T) == 4) {
    if (p.ldy <= 64) {
      // (data-groups with weights of their own begin at multiples of 256 pixels)
      if (p.M >= 512 * 256 && (p.nrep <= 1 || p.M / p.nrep % 512 == 0) && launch_dma_inst<T, 512, 64, 128, 32, 1, KB>(p, s)) return true;
      if (p.M <= 64 * 256 && launch_dma_inst<T, 64, 64, 32, 32, 1, KB>(p, s)) return true;
      return launch_dma_inst<T, 256, 64, 64, 32, 1, KB>(p, s);
    }
    if (tiles256 >= 256 && launch_dma_inst<T, 256, 128, 128, 32, 1, KB>(p, s)) return true;
    if ((long long)((p.M + 127) / 128) * ((p.ldy + 127) / 128) <= 64 && launch_dma_inst<T, 64, 64, 32, 32, 1, KB>(p, s)) return true;
    return launch_dma_inst<T, 128, 128, 64, 32, 1, KB>(p, s);
  } else {
    if (tiles256 >= 256) {
      if (p.ldy <= 64 && launch_dma_inst<T, 256, 64, 64, 64, 1, KB>(p, s)) return true;
      if (launch_dma_inst<T, 256, 128, 128, 64, 1, KB>(p, s)) return true;
    }
    // Launches that would leave half of the CUs without a 128 x 128 tile: 64 x 64 tiles whose channel chunks two halves of
    // eight waves share, a quarter of the stages (and of whole cache lines). 64 images, alone: 512 channels at 4 x 4 47.6 ->
    // 19.2 us, 256 at 8 x 8 26.6 -> 12.0 us; 128 at 16 x 16 (128 tiles) 17.2 against 16.3 us and no faster in the step.
    if ((long long)((p.M + 127) / 128) * ((p.ldy + 127) / 128) < 128 && launch_dma_inst<T, 64, 64, 32, 32, 1, 128, false, 2>(p, s)) return true;
    return launch_dma_inst<T, 128, 128, 64, 64, 1, KB>(p, s);
  }
}

// ------------------------------------------------------------------ any other convolution with whole 64-byte channel chunks
// Strided, 1x1 and stride-2 input-gradient launches: the same implicit GEMM as conv_gemm_kernel, its operands copied
// global -> LDS as in conv3x3_dma_kernel. A stage is one (tap, 64-byte channel chunk): BM gathered pixels (zeros where
// the tap leaves the image) and BN weight rows, two stages ahead in three slots. Which pixel a tile row is, and where
// its taps start, is worked out once per workgroup into a table in LDS.
// S2 (dgrad of a stride-2 layer): output pixels are dealt to workgroups by parity class (h % 2, w % 2), blockIdx.x =
// turn * tiles_per_class + tile, the class with the most taps first; a class walks only the taps of its parity (4, 2, 2 and 1 of
// nine; 1, 0, 0 and 0 of a 1x1 kernel, whose one class with work launched last made its fp32 launch of 131072 x 256 outputs from 512
// channels 143 us instead of 109, the head's included), class (0, 0) also a folded 1x1 shortcut (x2, w2).
// Bound by the copies and the barrier of short reductions. Alone against conv_gemm_kernel (operands staged through
// registers, outputs stored 8 bytes at a time), ResNet-18 shapes, 512 images: input gradients of the stride-2 layers
// 91 / 67 / 71 -> 54 / 42 / 46 us, their forward passes with the 1x1 shortcuts 50 / 40 / 58 -> 40 / 33 / 39 us.
struct GatherGeom {
  int tiles_per_class;
  int out_bytes;  // bytes of LDS below the row table: operand slots, then the epilogue's tiles
};

// KS = 2: eight waves, each four of which have operand slots of their own and walk half of the stages.
template <typename T, int BM, int BN, int WM, int WN, bool S2, int KS>
__global__ __launch_bounds__(256 * KS, 2) void conv_gather_kernel(ConvParams p_, GatherGeom g) {
  ConvParams p = p_;
  constexpr int ES = sizeof(T);
  constexpr int KB = 64, FROWS = 16, NKS = 2;  // bytes of a row (four 16-byte columns), rows of a 1 KiB fill, k-steps
  constexpr int AP = BM / FROWS / 4;                     // fills per wave and stage: gathered rows ...
  constexpr int RG = BN / FROWS, WL = RG >= 4 ? RG / 4 : 1;  // ... and weight rows (two waves copy the same ones if RG < 4)
  constexpr int SLOT = (BM + BN) * KB;
  constexpr int NI = WM / 32, NJ = WN / 32;
  static_assert((BM / WM) * (BN / WN) == 4, "four waves");
  static_assert(AP >= 1 && (RG >= 4 || RG == 2), "fills per wave");
  extern __shared__ __align__(16) char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  int* rowpix = (int*)(smem + g.out_bytes + 1024);  // output pixel of a tile row, -1 past the end
  int2* rowsrc = (int2*)(rowpix + BM);               // pixel of x at tap offset (0, 0); its row << 16 | column, signed

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave_wg & 3, khalf = wave_wg >> 2;
  const int wave_m = wave % (BM / WM), wave_n = wave / (BM / WM);
  const int turn = S2 ? (int)blockIdx.x / g.tiles_per_class : 0;
  const int cls = S2 ? (p.pad & 1 ? 3 - turn : turn) : 0;  // most taps first: odd rows and columns if pad is odd
  const int ch = cls >> 1, cw = cls & 1;
  const int Hc = S2 ? (p.Ho - ch + 1) >> 1 : p.Ho, Wc = S2 ? (p.Wo - cw + 1) >> 1 : p.Wo;  // this class's output grid
  const int Mc = p.Nimg * Hc * Wc;
  const int m0 = ((int)blockIdx.x - turn * g.tiles_per_class) * BM, n0 = blockIdx.y * BN;
  if (m0 >= Mc) return;  // the classes of an odd-sized grid differ
  if (p.nrep > 1) {  // the launcher made sure that a tile never straddles two data-groups
    const int r = min(m0 / (Mc / p.nrep), p.nrep - 1);
    p.w = (const char*)p.w + (size_t)r * p.w_rep;
    if (p.bias) p.bias += (size_t)r * p.bias_rep;
    if (p.w2) p.w2 = (const char*)p.w2 + (size_t)r * p.w2_rep;
  }
  if (tid < BM) {
    const int m = min(m0 + tid, Mc - 1);
    const int line = m / Wc, ow = m - line * Wc;
    const int img = line / Hc, oh = line - img * Hc;
    const int h = S2 ? oh : p.dgrad ? oh + p.pad : oh * p.stride - p.pad;
    const int w = S2 ? ow : p.dgrad ? ow + p.pad : ow * p.stride - p.pad;
    const int pix = S2 ? (img * p.Ho + 2 * oh + ch) * p.Wo + 2 * ow + cw : m;
    rowpix[tid] = m0 + tid < Mc ? pix : -1;
    rowsrc[tid] = make_int2((img * p.H + h) * p.W + w, (int)((uint32_t)h << 16 | (uint32_t)(w & 0xffff)));
  }
  __syncthreads();

  const int l4 = lane >> 2;
  const uint32_t c16 = (uint32_t)(((lane & 3) ^ ((l4 >> 2) & 3)) * 16);  // column c of row r lives at c ^ (r / 4) % 4
  int a_pix[AP], a_h[AP], a_w[AP];
#pragma unroll
  for (int j = 0; j < AP; ++j) {
    const int2 t = rowsrc[(wave + 4 * j) * FROWS + l4];
    a_pix[j] = t.x;
    a_h[j] = t.y >> 16;
    a_w[j] = (int)(int16_t)(t.y & 0xffff);
  }
  const char* zsrc = (const char*)p.zeros + c16;
  // weight rows past Nout repeat the last one: their columns are never stored
  uint32_t wvo[WL], wvo2[S2 ? WL : 1];
#pragma unroll
  for (int u = 0; u < WL; ++u) {
    const int n = min(n0 + (wave % RG + 4 * u) * FROWS + l4, p.Nout - 1);
    wvo[u] = (uint32_t)n * (uint32_t)(p.Ktot * ES) + c16;
    if (S2) wvo2[u] = (uint32_t)n * (uint32_t)(p.Cx2 * ES) + c16;
  }
  const int pixbytes = p.Cx * ES;
  const int nchunks = pixbytes / KB;
  // taps of this launch or class: r = r0, r0 + step, ...; likewise s
  const int step = S2 ? 2 : 1;
  const int r0 = S2 ? (ch + p.pad) & 1 : 0, s0 = S2 ? (cw + p.pad) & 1 : 0;
  const int ntr = p.R > r0 ? (p.R - r0 + step - 1) / step : 0, nts = p.S > s0 ? (p.S - s0 + step - 1) / step : 0;
  const int nk1 = ntr * nts * nchunks;  // stages of the layer itself; a folded shortcut's follow
  const int nk = nk1 + (S2 && p.x2 != nullptr && cls == 0 ? p.Cx2 * ES / KB : 0);

  const int per_half = (nk + KS - 1) / KS;
  const int kt0 = khalf * per_half;                  // first stage of this half
  const int own = min(nk - kt0, per_half);           // and how many it has
  // position of the next stage to be copied
  const int tap0 = KS > 1 ? kt0 / nchunks : 0;
  int fc = KS > 1 ? kt0 - tap0 * nchunks : 0;
  int fr = KS > 1 && nts > 0 ? r0 + step * (tap0 / nts) : r0, fs = KS > 1 && nts > 0 ? s0 + step * (tap0 % nts) : s0;
  auto fill = [&](int t, int slot) {
    const uint32_t base = lds0 + (khalf * 3 + slot) * SLOT;
    const int kt = kt0 + t;
    if (S2 && kt >= nk1) {  // the shortcut reads the pixel itself from its own tensor
      const int off = (kt - nk1) * KB;
      const char* x = (const char*)p.x2 + off;
#pragma unroll
      for (int j = 0; j < AP; ++j)
        dma16(x + (size_t)(uint32_t)a_pix[j] * (uint32_t)(p.Cx2 * ES) + c16, base + (wave + 4 * j) * 1024);
#pragma unroll
      for (int u = 0; u < WL; ++u)
        dma16s((const char*)p.w2 + off, wvo2[u], base + BM * KB + (wave % RG + 4 * u) * 1024);
      return;
    }
    // distance of the tap in x: forward (r, s), dgrad (-r, -s), S2 (ch + pad - r) / 2
    const int dr = S2 ? (ch + p.pad - fr) / 2 : p.dgrad ? -fr : fr, ds = S2 ? (cw + p.pad - fs) / 2 : p.dgrad ? -fs : fs;
    const int dp = dr * p.W + ds;
    const char* x = (const char*)p.x + fc * KB;
#pragma unroll
    for (int j = 0; j < AP; ++j) {
      const bool ok = (unsigned)(a_h[j] + dr) < (unsigned)p.H && (unsigned)(a_w[j] + ds) < (unsigned)p.W;
      const char* src = x + (size_t)(uint32_t)(a_pix[j] + dp) * (uint32_t)pixbytes + c16;
      dma16(ok ? src : zsrc, base + (wave + 4 * j) * 1024);
    }
    const char* w = (const char*)p.w + (size_t)(fr * p.S + fs) * pixbytes + fc * KB;
#pragma unroll
    for (int u = 0; u < WL; ++u) dma16s(w, wvo[u], base + BM * KB + (wave % RG + 4 * u) * 1024);
    if (++fc == nchunks) {
      fc = 0;
      fs += step;
      if (fs >= p.S) { fs = s0; fr += step; }
    }
  };
  const int lq = (lane >> 2) & 7;
  const int lpix = ((__builtin_popcount(lq) & 1) << 4) | ((lq >> 1) << 2) | (lane & 3);  // see conv3x3_dma_kernel
  const int half = lane >> 5;
  uint32_t mb[NI][NJ] = {};
  if (p.maskbits) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int pix = rowpix[wave_m * WM + i * 32 + lpix];
#pragma unroll
      for (int j = 0; j < NJ; ++j) mb[i][j] = load_bits32(p.maskbits, (size_t)max(pix, 0), p.ldy, n0 + wave_n * WN + 32 * j, pix >= 0);
    }
  }
  if (own > 0) fill(0, 0);
  if (own > 1) fill(1, 1);
  int aoff[NI], boff[NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = wave_m * WM + i * 32 + lpix;
    aoff[i] = m * KB + ((half ^ ((m >> 2) & 3)) << 4);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = wave_n * WN + j * 32 + (lane & 31);
    boff[j] = BM * KB + n * KB + ((half ^ ((n >> 2) & 3)) << 4);
  }
  f32x16_t acc[NJ][NI];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;

  int cur = 0, nxt = 2;  // slots of this stage and of the one two ahead
  for (int kt = 0; kt < per_half; ++kt) {
    if (kt + 1 < own) wait_vm<AP + WL>();  // only the next stage's copies are younger
    else wait_vm<0>();
    wg_barrier();
    if (KS > 1 && kt >= own) continue;
    if (kt + 2 < own) fill(kt + 2, nxt);
    const char* sb = smem + (khalf * 3 + cur) * SLOT;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      uint4 a[NI], b[NJ];
#pragma unroll
      for (int i = 0; i < NI; ++i) a[i] = *(const uint4*)(sb + (aoff[i] ^ (ks << 5)));
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[j] = *(const uint4*)(sb + (boff[j] ^ (ks << 5)));
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) mfma16B<T>(b[j], a[i], acc[j][i]);
    }
    cur = cur == 2 ? 0 : cur + 1;
    nxt = nxt == 2 ? 0 : nxt + 1;
  }
  wait_vm<0>();
  if (KS > 1) add_halves<NI, NJ>(acc, smem, khalf, wave, lane);
  const auto pixel = [&](int row) { return rowpix[row]; };
  tile_out<T, BM, BN, WM, WN>(p, acc, mb, smem, g.out_bytes, n0, wave, wave_m, wave_n, lane, lpix, pixel, khalf == 0);
}

template <typename T, int BM, int BN, int WM, int WN, bool S2, int KS = 1>
bool launch_gather_inst(const ConvParams& p, hipStream_t s) {
  GatherGeom g;
  const int mc = S2 ? p.Nimg * ((p.Ho + 1) / 2) * ((p.Wo + 1) / 2) : p.M;  // class (0, 0) is the largest
  g.tiles_per_class = (mc + BM - 1) / BM;
  constexpr int slots = KS * 3 * (BM + BN) * 64, tile = BM * BN * (int)sizeof(T);
  g.out_bytes = slots < tile && tile <= 72 * 1024 ? tile : slots;
  const int smem = g.out_bytes + 1024 + BM * 12;
  static DeviceOnce lds;
  allow_whole_lds(lds, (const void*)conv_gather_kernel<T, BM, BN, WM, WN, S2, KS>);
  dim3 grid((S2 ? 4 : 1) * g.tiles_per_class, (p.ldy + BN - 1) / BN);
  conv_gather_kernel<T, BM, BN, WM, WN, S2, KS><<<grid, 256 * KS, smem, s>>>(p, g);
  return true;
}

template <typename T, bool S2>
bool launch_gather_t(const ConvParams& p, hipStream_t s) {
  if (p.ldy <= 32) return launch_gather_inst<T, 128, 32, 32, 32, S2>(p, s);
  if (p.ldy <= 64) return launch_gather_inst<T, 128, 64, 64, 32, S2>(p, s);
  // few tiles: as in launch_dma (64 images of ResNet-18: 36 / 20 / 33 -> 19 / 12 / 19 us; with a line at 300 tiles the full
  // batch went from 17.1 to 17.3 ms per 8 steps)
  if (sizeof(T) == 2 && (long long)((p.M + 127) / 128) * ((p.ldy + 127) / 128) < 128)
    return launch_gather_inst<T, 64, 64, 32, 32, S2, 2>(p, s);
  return launch_gather_inst<T, 128, 128, 64, 64, S2>(p, s);
}

// False: not a launch of conv_gather_kernel, nothing launched.
template <typename T>
bool launch_gather(const ConvParams& p, hipStream_t s) {
  constexpr int KE = 64 / (int)sizeof(T);
  if (p.Cx % KE != 0 || p.ldy != p.Nout || p.zeros == nullptr || p.R < 1 || p.S < 1) return false;
  if (p.Ktot != p.R * p.S * p.Cx || p.stride < 1 || p.stride > 2) return false;
  // table entries hold a row and a column in 16 bits each; pixel numbers, weight offsets and bytes of a pixel are 32-bit
  if (p.H > 30000 || p.W > 30000 || p.R > 1000 || p.S > 1000) return false;
  if ((long long)p.Nimg * p.H * p.W >= (1ll << 30) || (long long)p.Nout * p.Ktot * (long long)sizeof(T) >= (1ll << 31)) return false;
  if (!p.dgrad || p.stride == 1) return p.x2 == nullptr && launch_gather_t<T, false>(p, s);
  if (p.x2 != nullptr && (p.Cx2 % KE != 0 || (long long)p.Nout * p.Cx2 * (long long)sizeof(T) >= (1ll << 31))) return false;
  return launch_gather_t<T, true>(p, s);
}

// ------------------------------------------------------------------ wgrad
// 16-byte chunks loaded along the channel axis for CE consecutive pixels are
// transposed in registers so that LDS rows run along the pixel (reduction) axis.
template <typename T> __device__ __forceinline__ void transpose_chunks(const uint4* in, uint4* out);
__device__ __forceinline__ uint32_t pack_lo(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }
template <> __device__ __forceinline__ void transpose_chunks<bf16_t>(const uint4* in, uint4* out) {
  // out[e] = element e of in[0..7]
  out[0] = make_uint4(pack_lo(in[0].x, in[1].x), pack_lo(in[2].x, in[3].x), pack_lo(in[4].x, in[5].x), pack_lo(in[6].x, in[7].x));
  out[1] = make_uint4(pack_hi(in[0].x, in[1].x), pack_hi(in[2].x, in[3].x), pack_hi(in[4].x, in[5].x), pack_hi(in[6].x, in[7].x));
  out[2] = make_uint4(pack_lo(in[0].y, in[1].y), pack_lo(in[2].y, in[3].y), pack_lo(in[4].y, in[5].y), pack_lo(in[6].y, in[7].y));
  out[3] = make_uint4(pack_hi(in[0].y, in[1].y), pack_hi(in[2].y, in[3].y), pack_hi(in[4].y, in[5].y), pack_hi(in[6].y, in[7].y));
  out[4] = make_uint4(pack_lo(in[0].z, in[1].z), pack_lo(in[2].z, in[3].z), pack_lo(in[4].z, in[5].z), pack_lo(in[6].z, in[7].z));
  out[5] = make_uint4(pack_hi(in[0].z, in[1].z), pack_hi(in[2].z, in[3].z), pack_hi(in[4].z, in[5].z), pack_hi(in[6].z, in[7].z));
  out[6] = make_uint4(pack_lo(in[0].w, in[1].w), pack_lo(in[2].w, in[3].w), pack_lo(in[4].w, in[5].w), pack_lo(in[6].w, in[7].w));
  out[7] = make_uint4(pack_hi(in[0].w, in[1].w), pack_hi(in[2].w, in[3].w), pack_hi(in[4].w, in[5].w), pack_hi(in[6].w, in[7].w));
}
template <typename T> __device__ __forceinline__ uint4 one_chunk();
template <> __device__ __forceinline__ uint4 one_chunk<bf16_t>() { return make_uint4(0x3f80u, 0, 0, 0); }

template <typename T, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(256, 2) void wgrad_gemm_kernel(WgradParams p) {
  constexpr int ES = sizeof(T);
  constexpr int CE = 16 / ES;
  constexpr int BKB = 128;
  constexpr int BKE = BKB / ES;    // pixels per tile
  constexpr int KG = BKE / CE;     // pixel groups per tile (each CE pixels)
  constexpr int LDK = BKB + 16;
  constexpr int A_BLOCKS = (BM / CE) * KG, B_BLOCKS = (BN / CE) * KG;
  constexpr int NBLK = (A_BLOCKS + B_BLOCKS + 255) / 256;  // blocks per thread
  static_assert((BM / WM) * (BN / WN) == 4, "four waves");
  __shared__ __align__(16) char smem[2 * (BM + BN) * LDK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave % (BM / WM), wave_n = wave / (BM / WM);
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int z = blockIdx.z;
  const int pz0 = z * p.pix_per_split;
  const int pz1 = min(p.P, pz0 + p.pix_per_split);
  const int HoWo = p.Ho * p.Wo;

  // static description of this thread's blocks
  bool isA[NBLK], okc[NBLK], isBias[NBLK];
  int row0[NBLK], kg[NBLK], bh[NBLK], bw[NBLK], coff[NBLK];
#pragma unroll
  for (int b = 0; b < NBLK; ++b) {
    int id = tid + b * 256;
    isA[b] = id < A_BLOCKS;
    isBias[b] = false;
    if (id >= A_BLOCKS + B_BLOCKS) {  // spare loader slot: contributes nothing
      okc[b] = false;
      row0[b] = -1;
      kg[b] = bh[b] = bw[b] = coff[b] = 0;
    } else if (isA[b]) {
      int mc = id % (BM / CE);
      kg[b] = id / (BM / CE);
      row0[b] = mc * CE;
      int m = m0 + mc * CE;
      okc[b] = m < p.ldy;
      coff[b] = m;
      bh[b] = bw[b] = 0;
    } else {
      id -= A_BLOCKS;
      int nc = id % (BN / CE);
      kg[b] = id / (BN / CE);
      row0[b] = BM + nc * CE;
      int n = n0 + nc * CE;
      okc[b] = n < p.NK;
      isBias[b] = n == p.NK;
      int nn = okc[b] ? n : 0;
      int tap = nn / p.Cx;
      coff[b] = nn - tap * p.Cx;
      int r = tap / p.S;
      bh[b] = r - p.pad;
      bw[b] = (tap - r * p.S) - p.pad;
    }
  }

  // unconditional loads from clamped addresses; validity is applied when the data is parked in LDS
  uint4 regs[NBLK][CE];
  uint32_t okmask[NBLK], onemask[NBLK];
  auto load_global = [&](int ptile) {
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
      okmask[b] = 0;
      onemask[b] = 0;
#pragma unroll
      for (int g = 0; g < CE; ++g) {
        const int pix = ptile + kg[b] * CE + g;
        const bool inr = pix < pz1;
        const char* src = (const char*)p.dy;
        bool ok = false;
        if (isA[b]) {
          ok = inr && okc[b];
          if (ok) src = (const char*)p.dy + ((size_t)pix * p.ldy + coff[b]) * ES;
        } else if (okc[b]) {
          const int pp = inr ? pix : 0;
          int img = pp / HoWo;
          int rem = pp - img * HoWo;
          int oh = rem / p.Wo, ow = rem - oh * p.Wo;
          int hi = oh * p.stride + bh[b], wi = ow * p.stride + bw[b];
          ok = inr && (unsigned)hi < (unsigned)p.H && (unsigned)wi < (unsigned)p.W;
          if (ok) src = (const char*)p.x + (((size_t)img * p.H + hi) * p.W + wi) * p.Cx * ES + (size_t)coff[b] * ES;
        } else if (isBias[b] && inr) {
          onemask[b] |= 1u << g;
        }
        okmask[b] |= (ok ? 1u : 0u) << g;
        regs[b][g] = *(const uint4*)src;
      }
    }
  };
  auto store_lds = [&](int buf) {
    char* base = smem + buf * (BM + BN) * LDK;
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
      if (row0[b] < 0) continue;
      uint4 sel[CE], t[CE];
#pragma unroll
      for (int g = 0; g < CE; ++g) {
        sel[g] = keep_if((okmask[b] >> g) & 1u, regs[b][g]);
        if ((onemask[b] >> g) & 1u) sel[g] = one_chunk<T>();
      }
      transpose_chunks<T>(sel, t);
#pragma unroll
      for (int e = 0; e < CE; ++e) *(uint4*)(base + (row0[b] + e) * LDK + kg[b] * 16) = t[e];
    }
  };

  f32x16_t acc[WM / 32][WN / 32];
#pragma unroll
  for (int i = 0; i < WM / 32; ++i)
#pragma unroll
    for (int j = 0; j < WN / 32; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const int nk = (pz1 - pz0 + BKE - 1) / BKE;
  if (nk > 0) {
    load_global(pz0);
    store_lds(0);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load_global(pz0 + (kt + 1) * BKE);
    const char* As = smem + buf * (BM + BN) * LDK + wave_m * WM * LDK;
    const char* Bs = smem + buf * (BM + BN) * LDK + BM * LDK + wave_n * WN * LDK;
    mma_step<T, WM, WN, BKB>(As, Bs, lane, acc);
    if (kt + 1 < nk) store_lds(buf ^ 1);
    __syncthreads();
  }

  float* out = p.partial + (size_t)z * p.Pl;
#pragma unroll
  for (int j = 0; j < WN / 32; ++j) {
    const int n = n0 + wave_n * WN + j * 32 + (lane & 31);
    if (n > p.NK) continue;
#pragma unroll
    for (int i = 0; i < WM / 32; ++i) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + wave_m * WM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (m >= p.Mout) continue;
        const float v = p.alpha * acc[i][j][e];
        if (n < p.NK) out[(size_t)m * p.NK + n] = v;
        else out[(size_t)p.Mout * p.NK + m] = v;
      }
    }
  }
}

// ------------------------------------------------------------------ 3x3 stride-1 wgrad, asynchronous LDS fills + LDS transpose reads (bf16)
// dW[k][tap][c] = sum over pixels p of dY[p][k] * X[p + tap][c]. The workgroup owns a
// 64(k) x 64(c) block for ALL nine taps and walks its split of the pixel axis in tiles of
// 128 pixels (rows of one image, or whole small images): per tile the dY rows and the X
// patch with halo are copied global -> LDS in their natural [pixel][channel] order (two
// slots: the next tile is copied while this one is multiplied) and the nine taps reuse them. The reduction
// index of this GEMM is the pixel, which is the slow axis of both operands in memory:
// ds_read_b64_tr_b16 hands each lane four pixels of one channel from a 4 x 16 block, so
// no register or LDS transposition is needed. 16-byte LDS columns are XOR-ed with
// 2*(row & 3) so that the four rows of such a block sit on different banks.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 lds_tr16(const char* p) {
  s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t DDS_LDS_AS*)p);
  return __builtin_bit_cast(uint2, v);
}

// Geometry the host passes along with WgradParams.
struct WgradGeom {
  int cblocks;     // 64-channel blocks of the real input tensor
  int sub[4];      // wgrad_flat_body<true>: sub-pixel (dy * 2 + dx) served by block row / cblocks
  int rmap[2][2];  // wgrad_flat_body<true>: real kernel row for (virtual row R', dy), -1 if none; the same table serves columns
  // wgrad_dma_body, wgrad_s2_dma_body
  int tiles_h;     // tiles per image (a power of two; 1 when a tile holds whole images)
  // wgrad_flat_body, wgrad_s2_flat_body
  int Q;           // position pitch of an image row, Wo + 1
  int imgs_rep;    // images per data-group
  int rep_tiles;   // tiles per data-group
  int patch_rows;  // of a tile, whole 8-row fills
  Divisor dQ, dH;  // by Q and by Ho + 1 (wgrad_rows_body: by Wo and by Ho)
};

__device__ __forceinline__ uint2 lds_tr16_at(uint32_t lds_byte_address) {
  s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t DDS_LDS_AS*)(size_t)lds_byte_address);
  return __builtin_bit_cast(uint2, v);
}

// Waves: four per tap group, each owning a 32(k) x 32(c) quarter of the block; three
// tap groups (one per kernel row, 12 waves, three per SIMD) so that the LDS reads of one wave
// hide behind the MFMAs of the others; a group's row shift is folded into its lanes' base addresses.
template <int TWLOG, int THLOG>
__device__ __forceinline__ void wgrad_dma_body(const WgradParams& p, const WgradGeom& wg, char* smem, int bx, int by, int z) {
  constexpr int TW = 1 << TWLOG, TH = 1 << THLOG, PW = TW + 2, PP = (TH + 2) * PW;
  constexpr int IMGS = 128 / (TW * TH);
  static_assert(IMGS >= 1 && IMGS * TW * TH == 128, "a tile is 128 pixels");
  constexpr int NWV = 12;                         // waves per workgroup
  constexpr int PROW = (IMGS * PP + 7) / 8 * 8;   // patch rows, whole 8-row fills
  constexpr int FY = (16 + NWV - 1) / NWV;        // dY fills per wave (16 per tile)
  constexpr int PF = (PROW / 8 + NWV - 1) / NWV;  // patch fills per wave
  constexpr int NT = 3;                           // taps accumulated by one wave
  // Two slots: tiles in flight in LDS (the next one is copied while this one is multiplied) keep a workgroup at 84 KB,
  // so that a conv workgroup of another module fits on the same CU; a third slot (copies two tiles ahead,
  // 126 KB) was 1-2 % slower per training step on every configuration although each launch alone was not.
  constexpr int SLOT = 16384 + PROW * 128;
  const uint32_t lds_ring = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = (wave >> 1) & 1;
  const int tg = wave >> 2;  // tap group: kernel row of this wave's three taps
  const int k0 = bx * 64;
  const int c0 = by * 64;
  // Split z = (data-group, j): the data-group's tiles are dealt to its q splits as evenly as whole
  // tiles allow (tile counts differ by at most one), so a split never mixes two data-groups.
  const int q = p.nsplit / p.nrep, rep_tiles = (p.P >> 7) / p.nrep;
  const int zr = z / q, zj = z - zr * q;
  const int tile0 = zr * rep_tiles + (int)(((long long)zj * rep_tiles) / q);
  const int ntiles = zr * rep_tiles + (int)(((long long)(zj + 1) * rep_tiles) / q) - tile0;
  const size_t ybytes = (size_t)p.ldy * 2, xbytes = (size_t)p.Cx * 2;

  // A tile is 128 consecutive pixels of the flattened (image, row, column) index of the output
  // grid, so the source address of every fill advances by a constant from tile to tile; what is
  // kept per lane and fill is the byte offset of its patch row relative to the tile origin and
  // the row / column facts that decide whether that row is padding.
  const int l8 = lane >> 3;
  const int c16 = ((lane & 7) ^ ((l8 & 3) << 1)) * 16;  // global 16-byte column for LDS slot lane&7 of a row with row&3 == l8&3
  const char* zsrc = (const char*)p.zeros + c16;
  constexpr int pw_total = PROW >> 3;
  const bool ycol_ok = k0 + (c16 >> 1) < p.ldy;   // this lane's 8 output channels exist
  const bool xcol_ok = c0 + (c16 >> 1) < p.Cx;    // ... and its 8 input channels (tensors narrower than a 64-channel block)
  const size_t tile_ybytes = 128 * ybytes, tile_xbytes = 128 * xbytes;
  const char* ysrc0 = (const char*)p.dy + ((size_t)tile0 * 128 + (size_t)(wave * 8 + l8)) * ybytes + (size_t)k0 * 2 + c16;
  const char* xsrc0 = (const char*)p.x + (size_t)tile0 * tile_xbytes + (size_t)c0 * 2 + c16;
  int prel[PF], pflag[PF];  // byte offset from the tile origin; yy | column valid << 8
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int row = (wave + NWV * u) * 8 + l8;
    int rel = 0, flag = 0;
    if (row < IMGS * PP) {
      const int im = row / PP, rem = row - im * PP;
      const int yy = rem / PW, xx = rem - yy * PW;
      rel = (int)((((long long)im * p.H + yy - 1) * p.W + (xx - 1)) * (long long)xbytes);
      flag = yy | (((unsigned)(xx - 1) < (unsigned)p.Wo ? 1 : 0) << 8);
    }
    prel[u] = rel;
    pflag[u] = flag;
  }
  const int tile_in_img_mask = wg.tiles_h - 1;
  auto fill_tile = [&](int t, int slot) {  // t: tile index inside this split (fills nothing real past the end)
    const bool live_t = t < ntiles;
    const int tt = live_t ? t : 0;
    const int h0 = ((tile0 + tt) & tile_in_img_mask) << THLOG;
    const uint32_t base = lds_ring + slot * SLOT;
    const char* ysrc = ysrc0 + (size_t)tt * tile_ybytes;
    const char* xsrc = xsrc0 + (size_t)tt * tile_xbytes;
    const bool yok = live_t && ycol_ok;
#pragma unroll
    for (int u = 0; u < FY; ++u) {  // dY rows: tile pixel 8*(wave + NWV u) + l8
      if (!(live_t && wave + NWV * u < 16)) continue;  // wave-uniform
      dma16(yok ? ysrc + (size_t)u * (NWV * 8) * ybytes : zsrc, base + (wave + NWV * u) * 1024);
    }
#pragma unroll
    for (int u = 0; u < PF; ++u) {  // patch rows
      const int wl = wave + NWV * u;
      if (!(live_t && wl < pw_total)) continue;  // wave-uniform
      const int gh = h0 + (pflag[u] & 255) - 1;
      const bool ok = xcol_ok && (pflag[u] >> 8) && (unsigned)gh < (unsigned)p.Ho;
      dma16(ok ? xsrc + prel[u] : zsrc, base + 16384 + wl * 1024);
    }
  };

  // the first tile is requested before the rest of the set-up, which runs under its latency
  fill_tile(0, 0);

  // fragment addressing (see lds_tr16): lane -> (16-lane group, row inside the 4-row block, 8-byte segment)
  const int lq = lane & 15, grp16 = (lane >> 4) & 1, khalf = lane >> 5;
  const int rsub = lq >> 2, seg = lq & 3;
  // A (dY): rows are tile pixels; row & 3 == rsub for every block this lane reads
  const int a_c = 4 * wave_m + 2 * grp16 + (seg >> 1);
  const int a_lane = (8 * khalf + rsub) * 128 + ((a_c ^ (rsub << 1)) << 4) + 8 * (seg & 1);
  // B (patch): k-step ks covers tile pixels 16 ks + ql, ql = 8 khalf + rsub + 4 hh for this
  // lane's two 4-pixel blocks hh. The patch row of such a pixel splits into a per-lane part
  // (kept in registers, one copy per value v of (row + tap offset) & 3 that the column
  // swizzle depends on) and a part that only depends on (ks, tap): a compile-time offset.
  const int b_c = 4 * wave_n + 2 * grp16 + (seg >> 1);
  int baddr[2][4];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int ql = 8 * khalf + rsub + 4 * hh;
    const int rl = (ql >> TWLOG) * PW + (ql & (TW - 1)) + tg * PW;
#pragma unroll
    for (int v = 0; v < 4; ++v) baddr[hh][v] = rl * 128 + ((b_c ^ (((rl + v) & 3) << 1)) << 4) + 8 * (seg & 1);
  }
  f32x16_t acc[NT], accb;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) accb[e] = 0.f;
  const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  // narrow layers (at most 32 output or input channels): the waves of the empty half-blocks skip the arithmetic
  const bool idle_wave = k0 + wave_m * 32 >= p.Mout || c0 + wave_n * 32 >= p.Cx;

  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill_tile(t + 1, (t + 1) & 1);
    uint32_t ybuf = lds_ring + (t & 1) * SLOT + a_lane;
    uint32_t bp[2][4];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        bp[hh][v] = lds_ring + (t & 1) * SLOT + 16384 + baddr[hh][v];
        // opaque: otherwise every (lane part + compile-time part) sum is precomputed outside the
        // tile loop, one register each, instead of riding in the instruction's offset field
        asm volatile("" : "+v"(bp[hh][v]));
      }
    asm volatile("" : "+v"(ybuf));
    // Fragments of k-step ks + 1 (16 pixels each) are read into the other register set while the
    // MFMAs of k-step ks run, so only the first k-step of a tile waits for LDS.
    uint4 af[2], bf[2][NT];
    auto load_frags = [&](int ks, int set) {  // ks is a constant after unrolling
      const int q0 = ks * 16;
      const int rc = (q0 >> (TWLOG + THLOG)) * PP + ((q0 >> TWLOG) & (TH - 1)) * PW + (q0 & (TW - 1));
      const uint2 a0 = lds_tr16_at(ybuf + ks * 2048);
      const uint2 a1 = lds_tr16_at(ybuf + ks * 2048 + 512);
      af[set] = make_uint4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
      for (int tap = 0; tap < NT; ++tap) {
        const int v = (rc + tap) & 3;  // the row shift sits in the base
        const uint2 b0 = lds_tr16_at(bp[0][v] + (rc + tap) * 128);
        const uint2 b1 = lds_tr16_at(bp[1][v] + (rc + tap) * 128);
        bf[set][tap] = make_uint4(b0.x, b0.y, b1.x, b1.y);
      }
    };
    if (idle_wave) continue;  // its 32 x 32 block lies past the real channels: fills and barriers only
    load_frags(0, 0);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      if (ks + 1 < 8) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
      for (int tap = 0; tap < NT; ++tap) mfma16B<bf16_t>(af[ks & 1], bf[ks & 1][tap], acc[tap]);
      if (wave_n == 0 && by == 0 && tg == 1) mfma16B<bf16_t>(af[ks & 1], ones, accb);  // bias gradient: column sums of dY
    }
  }
  wait_vm<0>();

  float* out = p.partial + (size_t)z * p.Pl;
  const int cin = c0 + wave_n * 32 + (lane & 31);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int k = k0 + wave_m * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (k >= p.Mout) continue;
    if (cin < p.Cx) {
#pragma unroll
      for (int tap = 0; tap < NT; ++tap)
        out[(size_t)k * p.NK + (tg * 3 + tap) * p.Cx + cin] = p.alpha * acc[tap][e];
    }
    if (wave_n == 0 && (lane & 31) == 0 && by == 0 && tg == 1) out[(size_t)p.Mout * p.NK + k] = p.alpha * accb[e];
  }
}

// ------------------------------------------------------------------ 3x3 stride-2 pad-1 weight gradients (bf16)
// Output pixel (oy, ox) and tap r read input row 2 oy + r - 1: of the input regrouped into 2x2 sub-pixels (dy, dx), tap rows 0 and 2 read dy =
// 1 of super-rows oy - 1 and oy, tap row 1 dy = 0 of oy; columns likewise. A tile is 64 output pixels, its patch four planes, one per
// sub-pixel (gathered at pixel stride 2 by the copies), in which consecutive output pixels are consecutive rows; otherwise as at stride
// 1: 64(k) x 64(c) for all nine taps, twelve waves, a kernel row per four of them, and in the launch of the stride-1 layers.
// Bound by the copies (46 KB for 144 MFMAs) and the barrier of a tile. Before, a workgroup of four waves took one sub-pixel of 128-pixel tiles
// with the 1, 2, 2 or 4 taps that meet it, so dY was copied four times and the workgroups' work differed as much. ResNet-18, 512 images, serial
// time of all weight gradients of a step but the stem's: 810 -> 595 us (the three stride-2 layers with their shortcuts took 265 in launches of their
// own); steps of 512 images 2.065 -> 2.02 ms, of 64 0.482 -> 0.460, ResNet-20 in one module 0.300 -> 0.291, ResNet-56 1.65 -> 1.60.
struct S2Acc {
  f32x16_t tap[3], bias;
};
__device__ __forceinline__ void wgrad_s2_store(const WgradParams& p, const S2Acc& acc, int k0, int c0, int z, int wave_m, int wave_n, int tg, int lane, bool bias_wave) {
  float* out = p.partial + (size_t)z * p.Pl;
  const int cin = c0 + wave_n * 32 + (lane & 31);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int k = k0 + wave_m * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (k >= p.Mout) continue;
    if (cin < p.Cx) {
#pragma unroll
      for (int s = 0; s < 3; ++s) out[(size_t)k * p.NK + (tg * 3 + s) * p.Cx + cin] = p.alpha * acc.tap[s][e];
    }
    if (bias_wave && (lane & 31) == 0) out[(size_t)p.Mout * p.NK + k] = p.alpha * acc.bias[e];
  }
}

// Input of 2 Ho x 2 Wo with Ho and Wo powers of two, whole 64-pixel tiles of rows of one image or of whole images: every address in the loop is
// a register plus a constant. ALL: an image's plane has a row above it whether dy needs one or not (tiles of several images, whose
// distance in a plane is a constant then).
template <int TWLOG, int THLOG>
struct S2Tile {
  static constexpr int TW = 1 << TWLOG, TH = 1 << THLOG, IMGS = 64 / (TW * TH);
  static constexpr bool ALL = IMGS > 1;
  static_assert(IMGS >= 1 && IMGS * TW * TH == 64, "a tile is 64 pixels");
  static constexpr int height(int dy) { return TH + (ALL ? 1 : dy); }
  static constexpr int rows(int d) { return (IMGS * height(d >> 1) * (TW + (d & 1)) + 7) / 8 * 8; }
  static constexpr int base(int d) { return d == 0 ? 0 : base(d - 1) + rows(d - 1); }  // of the planes (0,0), (0,1), (1,0), (1,1)
  static constexpr int patch = base(3) + rows(3);
};
template <int TWLOG, int THLOG>
__device__ __forceinline__ void wgrad_s2_dma_body(const WgradParams& p, const WgradGeom& wg, char* smem, int bx, int by, int z) {
  typedef S2Tile<TWLOG, THLOG> T;
  constexpr int TW = T::TW, TH = T::TH, NWV = 12;
  constexpr int PF = (T::patch / 8 + NWV - 1) / NWV;  // patch fills per wave
  constexpr int SLOT = 8192 + T::patch * 128;
  const uint32_t lds_ring = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = (wave >> 1) & 1, tg = wave >> 2;
  const int k0 = bx * 64, c0 = by * 64;
  const int q = p.nsplit / p.nrep, rep_tiles = (p.P >> 6) / p.nrep;
  const int zr = z / q, zj = z - zr * q;
  const int tile0 = zr * rep_tiles + (int)(((long long)zj * rep_tiles) / q);
  const int ntiles = zr * rep_tiles + (int)(((long long)(zj + 1) * rep_tiles) / q) - tile0;
  const size_t ybytes = (size_t)p.ldy * 2, xbytes = (size_t)p.Cx * 2;

  const int l8 = lane >> 3;
  const int c16 = ((lane & 7) ^ ((l8 & 3) << 1)) * 16;  // global 16-byte column for LDS slot lane&7 of a row with row&3 == l8&3
  const char* zsrc = (const char*)p.zeros + c16;
  const bool ycol_ok = k0 + (c16 >> 1) < p.ldy, xcol_ok = c0 + (c16 >> 1) < p.Cx;
  const size_t tile_ybytes = 64 * ybytes, tile_xbytes = 256 * xbytes;
  const char* ysrc0 = (const char*)p.dy + ((size_t)tile0 * 64 + (size_t)(wave * 8 + l8)) * ybytes + (size_t)k0 * 2 + c16;
  const char* xsrc0 = (const char*)p.x + (size_t)tile0 * tile_xbytes + (size_t)c0 * 2 + c16;
  int prel[PF], pflag[PF];  // byte offset from the tile's first input pixel; super-row from the tile's first, -2 where the column is none
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int row = (wave + NWV * u) * 8 + l8;
    const int d = row < T::base(1) ? 0 : row < T::base(2) ? 1 : row < T::base(3) ? 2 : 3;
    const int dy = d >> 1, dx = d & 1, pw = TW + dx, ph = T::ALL ? TH + 1 : TH + dy;
    const int r = row - (d == 0 ? 0 : d == 1 ? T::base(1) : d == 2 ? T::base(2) : T::base(3));
    const int im = r / (pw * ph), rem = r - im * (pw * ph), yy = rem / pw, xx = rem - yy * pw;
    const int sy = yy - (T::ALL ? 1 : dy), sx = xx - dx;
    prel[u] = (int)((((long long)im * p.H + 2 * sy + dy) * p.W + 2 * sx + dx) * (long long)xbytes);
    pflag[u] = im < T::IMGS && sx >= 0 ? sy : -2;
  }
  auto fill_tile = [&](int t, int slot) {
    if (t >= ntiles) return;
    const int h0 = ((tile0 + t) & (wg.tiles_h - 1)) << THLOG;
    const uint32_t base = lds_ring + slot * SLOT;
    if (wave < 8) dma16(ycol_ok ? ysrc0 + (size_t)t * tile_ybytes : zsrc, base + wave * 1024);
    const char* xsrc = xsrc0 + (size_t)t * tile_xbytes;
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int f = wave + NWV * u;
      if (f >= T::patch / 8) continue;  // wave-uniform
      const bool ok = xcol_ok && pflag[u] >= -1 && h0 + pflag[u] >= 0;
      dma16(ok ? xsrc + prel[u] : zsrc, base + 8192 + f * 1024);
    }
  };
  fill_tile(0, 0);

  const int lq = lane & 15, grp16 = (lane >> 4) & 1, khalf = lane >> 5;  // fragment addressing as in wgrad_dma_body
  const int rsub = lq >> 2, seg = lq & 3;
  const int a_c = 4 * wave_m + 2 * grp16 + (seg >> 1), b_c = 4 * wave_n + 2 * grp16 + (seg >> 1);
  const int a_lane = (8 * khalf + rsub) * 128 + ((a_c ^ (rsub << 1)) << 4) + 8 * (seg & 1);
  // patch rows: a lane's part for each plane of its kernel row and each value of the constant part mod 4 (the column swizzle depends on it)
  const int dy = tg == 1 ? 0 : 1, ys = T::ALL ? (tg == 0 ? 0 : 1) : tg == 2 ? 1 : 0;
  int baddr[2][2][4];
#pragma unroll
  for (int dx = 0; dx < 2; ++dx)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int ql = 8 * khalf + rsub + 4 * hh;
      const int plane = dy ? (dx ? T::base(3) : T::base(2)) : (dx ? T::base(1) : T::base(0));
      const int rl = plane + ((ql >> TWLOG) + ys) * (TW + dx) + (ql & (TW - 1));
#pragma unroll
      for (int v = 0; v < 4; ++v) baddr[dx][hh][v] = 8192 + rl * 128 + ((b_c ^ (((rl + v) & 3) << 1)) << 4) + 8 * (seg & 1);
    }
  S2Acc acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc.tap[0][e] = acc.tap[1][e] = acc.tap[2][e] = acc.bias[e] = 0.f;
  const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  const bool idle_wave = k0 + wave_m * 32 >= p.Mout || c0 + wave_n * 32 >= p.Cx;
  const bool bias_wave = wave_n == 0 && by == 0 && tg == 1;

  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill_tile(t + 1, (t + 1) & 1);
    if (idle_wave) continue;
    uint32_t base = lds_ring + (t & 1) * SLOT;
    asm volatile("" : "+s"(base));
    uint32_t bp[2][2][4];
#pragma unroll
    for (int dx = 0; dx < 2; ++dx)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          bp[dx][hh][v] = base + baddr[dx][hh][v];
          asm volatile("" : "+v"(bp[dx][hh][v]));  // constants ride in the instructions' offsets (see wgrad_dma_body)
        }
    uint32_t ybuf = base + a_lane;
    asm volatile("" : "+v"(ybuf));
    uint4 af[2], bf[2][3];
    auto load_frags = [&](int ks, int set) {  // ks is a constant after unrolling
      const int q0 = ks * 16;
      const uint2 a0 = lds_tr16_at(ybuf + ks * 2048), a1 = lds_tr16_at(ybuf + ks * 2048 + 512);
      af[set] = make_uint4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const int dx = s == 1 ? 0 : 1, pw = TW + dx;
        const int rc = (q0 >> (TWLOG + THLOG)) * ((TH + 1) * pw) + ((q0 >> TWLOG) & (TH - 1)) * pw + (q0 & (TW - 1)) + (s == 2 ? 1 : 0);
        const uint2 b0 = lds_tr16_at(bp[dx][0][rc & 3] + rc * 128), b1 = lds_tr16_at(bp[dx][1][rc & 3] + rc * 128);
        bf[set][s] = make_uint4(b0.x, b0.y, b1.x, b1.y);
      }
    };
    load_frags(0, 0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks + 1 < 4) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
      for (int s = 0; s < 3; ++s) mfma16B<bf16_t>(af[ks & 1], bf[ks & 1][s], acc.tap[s]);
      if (bias_wave) mfma16B<bf16_t>(af[ks & 1], ones, acc.bias);  // bias gradient: column sums of dY
    }
  }
  wait_vm<0>();
  wgrad_s2_store(p, acc, k0, c0, z, wave_m, wave_n, tg, lane, bias_wave);
}

// ------------------------------------------------------------------ the same weight gradients for any image size (bf16)
// wgrad_dma_body wants images whose sides are powers of two and data-groups of whole 128-pixel tiles. Everything
// else 3x3 stride 1 or 2 comes here. The pixels of a data-group are numbered with a row pitch of Wo + 1 and one
// extra row above every image, so that each row's padding is the extra column before it and each image's the extra
// row: a tile is 128 consecutive such positions, dY and X are copied with zeros at the extra ones, and the taps are
// constant distances (-Q-1 .. Q+1, Q = Wo + 1) with nothing to test in the inner loop. Price: (Ho+1)(Wo+1) / (Ho Wo)
// of the arithmetic (1.07 at 28 x 28) and two multiply-high divisions per copied row. Otherwise as above: a workgroup owns
// 64(k) x 64(c) for all taps; S2: one sub-pixel of the input at a time, its taps R', S' in {-1, 0}.
// Bound, as there, by the barrier and the LDS reads around a tile's MFMAs. 64 -> 64 channels at 14 x 14, 194 images, with
// 196 workgroups of wgrad_gemm_kernel (operands transposed in registers) 62 us, here 12 us; 32 -> 64 at stride 2 from
// 28 x 28 42 -> 16 us.
template <bool S2>
__device__ __forceinline__ void wgrad_flat_body(const WgradParams& p, const WgradGeom& wg, char* smem, int bx, int by, int z) {
  constexpr int NWV = S2 ? 4 : 12;  // waves: four per tap group, each a 32(k) x 32(c) quarter; stride 1: one group per kernel row
  constexpr int NT = S2 ? 4 : 3;    // taps accumulated by one wave
  const uint32_t lds_ring = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int slot_bytes = 16384 + wg.patch_rows * 128;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = (wave >> 1) & 1;
  const int tg = wave >> 2;
  const int k0 = bx * 64;
  const int sub = S2 ? wg.sub[by / wg.cblocks] : 0;
  const int sdy = sub >> 1, sdx = sub & 1;
  const int c0 = (S2 ? by % wg.cblocks : by) * 64;
  const int q = p.nsplit / p.nrep;
  const int zr = z / q, zj = z - zr * q;
  const int tile0 = (int)(((long long)zj * wg.rep_tiles) / q);
  const int ntiles = (int)(((long long)(zj + 1) * wg.rep_tiles) / q) - tile0;

  const int l8 = lane >> 3;
  const int c16 = ((lane & 7) ^ ((l8 & 3) << 1)) * 16;  // global 16-byte column for LDS slot lane&7 of a row with row&3 == l8&3
  const char* zsrc = (const char*)p.zeros + c16;
  const bool ycol_ok = k0 + (c16 >> 1) < p.ldy, xcol_ok = c0 + (c16 >> 1) < p.Cx;
  const char* ybase = (const char*)p.dy + (size_t)k0 * 2 + c16;
  const char* xbase = (const char*)p.x + (size_t)c0 * 2 + c16;
  const uint32_t ybytes = (uint32_t)p.ldy * 2, xbytes = (uint32_t)p.Cx * 2;
  const int img0 = zr * wg.imgs_rep;
  // position in the data-group -> image of the group, row, column of the output grid; false on the extra rows and columns
  auto locate = [&](int u, int& im, int& h, int& w) {
    const uint32_t uu = (uint32_t)max(u, 0);
    const int line = (int)(__umulhi(uu, wg.dQ.mul) >> wg.dQ.shift);
    w = (int)uu - line * wg.Q;
    im = (int)(__umulhi((uint32_t)line, wg.dH.mul) >> wg.dH.shift);
    h = line - im * (p.Ho + 1) - 1;
    return u >= 0 && w < p.Wo && h >= 0 && im < wg.imgs_rep;
  };
  auto fill_tile = [&](int t, int slot) {
    if (t >= ntiles) return;
    const int u0 = (tile0 + t) * 128;
    const uint32_t base = lds_ring + slot * slot_bytes;
    for (int f = wave; f < 16 + (wg.patch_rows >> 3); f += NWV) {  // 16 fills of dY rows, then the patch: eight rows each
      int im, h, w;
      const char* src = zsrc;
      if (f < 16) {
        const bool ok = locate(u0 + f * 8 + l8, im, h, w) && ycol_ok;
        if (ok) src = ybase + (size_t)((uint32_t)(((img0 + im) * p.Ho + h) * p.Wo + w)) * ybytes;
      } else {
        bool ok = locate(u0 - wg.Q - 1 + (f - 16) * 8 + l8, im, h, w) && xcol_ok;
        const int hi = S2 ? 2 * h + sdy : h, wi = S2 ? 2 * w + sdx : w;
        if (S2) ok = ok && hi < p.H && wi < p.W;
        if (ok) src = xbase + (size_t)((uint32_t)(((img0 + im) * p.H + hi) * p.W + wi)) * xbytes;
      }
      dma16(src, base + f * 1024);
    }
  };
  fill_tile(0, 0);

  // fragment addressing as in wgrad_dma_body; the patch row of tile position u at tap (R, S) is u + R Q + S
  const int lq = lane & 15, grp16 = (lane >> 4) & 1, khalf = lane >> 5;
  const int rsub = lq >> 2, seg = lq & 3;
  const int a_c = 4 * wave_m + 2 * grp16 + (seg >> 1);
  const int a_lane = (8 * khalf + rsub) * 128 + ((a_c ^ (rsub << 1)) << 4) + 8 * (seg & 1);
  const int b_c = 4 * wave_n + 2 * grp16 + (seg >> 1);
  int baddr[2][NT];
  bool live[NT];
  int tapreal[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int toff = S2 ? (t >> 1) * wg.Q + (t & 1) : tg * wg.Q + t;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int row = 8 * khalf + rsub + 4 * hh + toff;
      baddr[hh][t] = 16384 + row * 128 + ((b_c ^ ((row & 3) << 1)) << 4) + 8 * (seg & 1);
    }
    if (S2) {
      const int rr = wg.rmap[t >> 1][sdy], ss = wg.rmap[t & 1][sdx];
      live[t] = rr >= 0 && ss >= 0;
      tapreal[t] = rr * p.S + ss;
    } else {
      live[t] = true;
      tapreal[t] = tg * 3 + t;
    }
  }
  f32x16_t acc[NT], accb;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) accb[e] = 0.f;
  const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  const bool idle_wave = k0 + wave_m * 32 >= p.Mout || c0 + wave_n * 32 >= p.Cx;
  const bool bias_wave = wave_n == 0 && by == 0 && tg == (S2 ? 0 : 1);

  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill_tile(t + 1, (t + 1) & 1);
    if (idle_wave) continue;
    const uint32_t base = lds_ring + (t & 1) * slot_bytes;
    const uint32_t ybuf = base + a_lane;
    uint32_t bp[2][NT];
#pragma unroll
    for (int tap = 0; tap < NT; ++tap) { bp[0][tap] = base + baddr[0][tap]; bp[1][tap] = base + baddr[1][tap]; }
    uint4 af[2], bf[2][NT];
    auto load_frags = [&](int ks, int set) {  // 16 positions; fragments of step ks + 1 are read while step ks is multiplied
      const uint2 a0 = lds_tr16_at(ybuf + ks * 2048), a1 = lds_tr16_at(ybuf + ks * 2048 + 512);
      af[set] = make_uint4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
      for (int tap = 0; tap < NT; ++tap) {
        const uint2 b0 = lds_tr16_at(bp[0][tap] + ks * 2048), b1 = lds_tr16_at(bp[1][tap] + ks * 2048);
        bf[set][tap] = make_uint4(b0.x, b0.y, b1.x, b1.y);
      }
    };
    load_frags(0, 0);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      if (ks + 1 < 8) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
      for (int tap = 0; tap < NT; ++tap)
        if (!S2 || live[tap]) mfma16B<bf16_t>(af[ks & 1], bf[ks & 1][tap], acc[tap]);
      if (bias_wave) mfma16B<bf16_t>(af[ks & 1], ones, accb);  // bias gradient: column sums of dY
    }
  }
  wait_vm<0>();

  float* out = p.partial + (size_t)z * p.Pl;
  const int cin = c0 + wave_n * 32 + (lane & 31);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int k = k0 + wave_m * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (k >= p.Mout) continue;
    if (cin < p.Cx) {
#pragma unroll
      for (int tap = 0; tap < NT; ++tap)
        if (live[tap]) out[(size_t)k * p.NK + tapreal[tap] * p.Cx + cin] = p.alpha * acc[tap][e];
    }
    if (bias_wave && (lane & 31) == 0) out[(size_t)p.Mout * p.NK + k] = p.alpha * accb[e];
  }
}

// The same for any image size, on positions as in wgrad_flat_body: a plane of a tile holds the positions from 64 before ... the tile's first, less
// one row of Q if dy (tap row 0) and less one if dx (tap column 0), on.
struct S2Flat {
  int rows[4], base[4], total;  // of the planes (dy, dx) = (0,0), (0,1), (1,0), (1,1)
};
__host__ __device__ inline S2Flat s2_flat(int Q) {
  S2Flat f;
  f.total = 0;
  for (int d = 0; d < 4; ++d) {
    f.rows[d] = (64 + (d >> 1) * Q + (d & 1) + 7) / 8 * 8;
    f.base[d] = f.total;
    f.total += f.rows[d];
  }
  return f;
}
__device__ __forceinline__ void wgrad_s2_flat_body(const WgradParams& p, const WgradGeom& wg, char* smem, int bx, int by, int z) {
  constexpr int NWV = 12;
  const uint32_t lds_ring = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const S2Flat pl = s2_flat(wg.Q);
  const int slot_bytes = 8192 + pl.total * 128;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = (wave >> 1) & 1, tg = wave >> 2;
  const int k0 = bx * 64, c0 = by * 64;
  const int q = p.nsplit / p.nrep;
  const int zr = z / q, zj = z - zr * q;
  const int tile0 = (int)(((long long)zj * wg.rep_tiles) / q);
  const int ntiles = (int)(((long long)(zj + 1) * wg.rep_tiles) / q) - tile0;

  const int l8 = lane >> 3;
  const int c16 = ((lane & 7) ^ ((l8 & 3) << 1)) * 16;  // global 16-byte column for LDS slot lane&7 of a row with row&3 == l8&3
  const char* zsrc = (const char*)p.zeros + c16;
  const bool ycol_ok = k0 + (c16 >> 1) < p.ldy, xcol_ok = c0 + (c16 >> 1) < p.Cx;
  const char* ybase = (const char*)p.dy + (size_t)k0 * 2 + c16;
  const char* xbase = (const char*)p.x + (size_t)c0 * 2 + c16;
  const uint32_t ybytes = (uint32_t)p.ldy * 2, xbytes = (uint32_t)p.Cx * 2;
  const int img0 = zr * wg.imgs_rep;
  auto fill_tile = [&](int t, int slot) {
    if (t >= ntiles) return;
    const int u0 = (tile0 + t) * 64;
    const uint32_t base = lds_ring + slot * slot_bytes;
    for (int f = wave; f < 8 + (pl.total >> 3); f += NWV) {  // eight fills of dY rows, then the planes: eight rows each
      const int r = (f - 8) * 8;
      const int d = r < pl.base[1] ? 0 : r < pl.base[2] ? 1 : r < pl.base[3] ? 2 : 3;  // wave-uniform
      const int dy = f < 8 ? 0 : d >> 1, dx = f < 8 ? 0 : d & 1;
      const int u = u0 + (f < 8 ? f * 8 : r - (d == 0 ? 0 : d == 1 ? pl.base[1] : d == 2 ? pl.base[2] : pl.base[3]) - dy * wg.Q - dx) + l8;
      // position in the data-group -> image of the group, row, column of the output grid; none on the extra rows and columns
      const uint32_t uu = (uint32_t)max(u, 0);
      const int line = (int)(__umulhi(uu, wg.dQ.mul) >> wg.dQ.shift), w = (int)uu - line * wg.Q;
      const int im = (int)(__umulhi((uint32_t)line, wg.dH.mul) >> wg.dH.shift), h = line - im * (p.Ho + 1) - 1;
      bool ok = u >= 0 && w < p.Wo && h >= 0 && im < wg.imgs_rep;
      const char* src = zsrc;
      if (f < 8) {
        if (ok && ycol_ok) src = ybase + (size_t)((uint32_t)(((img0 + im) * p.Ho + h) * p.Wo + w)) * ybytes;
      } else {
        const int hi = 2 * h + dy, wi = 2 * w + dx;
        ok = ok && xcol_ok && hi < p.H && wi < p.W;
        if (ok) src = xbase + (size_t)((uint32_t)(((img0 + im) * p.H + hi) * p.W + wi)) * xbytes;
      }
      dma16(src, base + f * 1024);
    }
  };
  fill_tile(0, 0);

  const int lq = lane & 15, grp16 = (lane >> 4) & 1, khalf = lane >> 5;  // fragment addressing as in wgrad_dma_body
  const int rsub = lq >> 2, seg = lq & 3;
  const int a_c = 4 * wave_m + 2 * grp16 + (seg >> 1), b_c = 4 * wave_n + 2 * grp16 + (seg >> 1);
  const int a_lane = (8 * khalf + rsub) * 128 + ((a_c ^ (rsub << 1)) << 4) + 8 * (seg & 1);
  int baddr[2][3];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int plane = tg == 1 ? (s == 1 ? pl.base[0] : pl.base[1]) : (s == 1 ? pl.base[2] : pl.base[3]);
      const int row = plane + 8 * khalf + rsub + 4 * hh + (tg == 2 ? wg.Q : 0) + (s == 2 ? 1 : 0);
      baddr[hh][s] = 8192 + row * 128 + ((b_c ^ ((row & 3) << 1)) << 4) + 8 * (seg & 1);
    }
  S2Acc acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc.tap[0][e] = acc.tap[1][e] = acc.tap[2][e] = acc.bias[e] = 0.f;
  const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  const bool idle_wave = k0 + wave_m * 32 >= p.Mout || c0 + wave_n * 32 >= p.Cx;
  const bool bias_wave = wave_n == 0 && by == 0 && tg == 1;

  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill_tile(t + 1, (t + 1) & 1);
    if (idle_wave) continue;
    const uint32_t base = lds_ring + (t & 1) * slot_bytes;
    uint32_t bp[2][3];
#pragma unroll
    for (int s = 0; s < 3; ++s) { bp[0][s] = base + baddr[0][s]; bp[1][s] = base + baddr[1][s]; }
    uint4 af[2], bf[2][3];
    auto load_frags = [&](int ks, int set) {
      const uint2 a0 = lds_tr16_at(base + a_lane + ks * 2048), a1 = lds_tr16_at(base + a_lane + ks * 2048 + 512);
      af[set] = make_uint4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const uint2 b0 = lds_tr16_at(bp[0][s] + ks * 2048), b1 = lds_tr16_at(bp[1][s] + ks * 2048);
        bf[set][s] = make_uint4(b0.x, b0.y, b1.x, b1.y);
      }
    };
    load_frags(0, 0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks + 1 < 4) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
      for (int s = 0; s < 3; ++s) mfma16B<bf16_t>(af[ks & 1], bf[ks & 1][s], acc.tap[s]);
      if (bias_wave) mfma16B<bf16_t>(af[ks & 1], ones, acc.bias);  // bias gradient: column sums of dY
    }
  }
  wait_vm<0>();
  wgrad_s2_store(p, acc, k0, c0, z, wave_m, wave_n, tg, lane, bias_wave);
}

// Linear layers and 1x1 convolutions of stride 1 and 2 (bf16): no taps; tiles of 128 output pixels, four waves, the rest as above. Against
// operands transposed in registers (wgrad_gemm_kernel), each launch alone, a net of three linear layers: 512 -> 512 in the middle at
// 16 / 512 / 4096 rows 32 / 44 / 58 -> 22 / 23 / 33 us, 2048 -> 32 at 16384 rows 120 -> 65 us. A head shares the launch of its module's
// shortcuts, where the old kernel took 11 to 16 us with one to twelve workgroups.
__device__ __forceinline__ void wgrad_rows_body(const WgradParams& p, const WgradGeom& wg, char* smem, int bx, int by, int z) {
  constexpr int SLOT = 32768;
  const uint32_t lds_ring = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = wave >> 1;
  const int k0 = bx * 64, c0 = by * 64;
  const int q = p.nsplit / p.nrep;
  const int zr = z / q, zj = z - zr * q;
  const int tile0 = (int)(((long long)zj * wg.rep_tiles) / q);
  const int ntiles = (int)(((long long)(zj + 1) * wg.rep_tiles) / q) - tile0;
  const int rows_rep = p.P / p.nrep, row0 = zr * rows_rep;

  const int l8 = lane >> 3;
  const int c16 = ((lane & 7) ^ ((l8 & 3) << 1)) * 16;  // global 16-byte column for LDS slot lane&7 of a row with row&3 == l8&3
  const char* zsrc = (const char*)p.zeros + c16;
  const bool ycol_ok = k0 + (c16 >> 1) < p.ldy, xcol_ok = c0 + (c16 >> 1) < p.Cx;
  const char* ybase = (const char*)p.dy + (size_t)k0 * 2 + c16;
  const char* xbase = (const char*)p.x + (size_t)c0 * 2 + c16;
  auto fill_tile = [&](int t, int slot) {
    if (t >= ntiles) return;
    const uint32_t base = lds_ring + slot * SLOT;
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // eight rows of each operand
      const int f = wave + 4 * u, row = (tile0 + t) * 128 + f * 8 + l8;
      const bool ok = row < rows_rep;
      const uint32_t r = (uint32_t)(row0 + row);
      uint32_t rx = r;  // row of X: the pixel itself, or the one at twice its row and column
      if (p.stride == 2) {
        const uint32_t line = p.Wo > 1 ? __umulhi(r, wg.dQ.mul) >> wg.dQ.shift : r, im = p.Ho > 1 ? __umulhi(line, wg.dH.mul) >> wg.dH.shift : line;
        rx = (im * p.H + 2 * (line - im * p.Ho)) * p.W + 2 * (r - line * p.Wo);
      }
      dma16(ok && ycol_ok ? ybase + (size_t)r * (uint32_t)(p.ldy * 2) : zsrc, base + f * 1024);
      dma16(ok && xcol_ok ? xbase + (size_t)rx * (uint32_t)(p.Cx * 2) : zsrc, base + 16384 + f * 1024);
    }
  };
  fill_tile(0, 0);

  const int lq = lane & 15, grp16 = (lane >> 4) & 1, khalf = lane >> 5;  // fragment addressing as in wgrad_dma_body
  const int rsub = lq >> 2, seg = lq & 3;
  const int a_c = 4 * wave_m + 2 * grp16 + (seg >> 1), b_c = 4 * wave_n + 2 * grp16 + (seg >> 1);
  const int lrow = (8 * khalf + rsub) * 128 + 8 * (seg & 1);
  const int a_lane = lrow + ((a_c ^ (rsub << 1)) << 4), b_lane = lrow + 16384 + ((b_c ^ (rsub << 1)) << 4);
  f32x16_t acc, accb;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = accb[e] = 0.f;
  const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  const bool idle_wave = k0 + wave_m * 32 >= p.Mout || c0 + wave_n * 32 >= p.Cx;
  const bool bias_wave = wave_n == 0 && by == 0;

  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill_tile(t + 1, (t + 1) & 1);
    if (idle_wave) continue;
    const uint32_t base = lds_ring + (t & 1) * SLOT;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint2 a0 = lds_tr16_at(base + a_lane + ks * 2048), a1 = lds_tr16_at(base + a_lane + ks * 2048 + 512);
      const uint2 b0 = lds_tr16_at(base + b_lane + ks * 2048), b1 = lds_tr16_at(base + b_lane + ks * 2048 + 512);
      const uint4 a = make_uint4(a0.x, a0.y, a1.x, a1.y);
      mfma16B<bf16_t>(a, make_uint4(b0.x, b0.y, b1.x, b1.y), acc);
      if (bias_wave) mfma16B<bf16_t>(a, ones, accb);  // bias gradient: column sums of dY
    }
  }
  wait_vm<0>();

  float* out = p.partial + (size_t)z * p.Pl;
  const int cin = c0 + wave_n * 32 + (lane & 31);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int k = k0 + wave_m * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (k >= p.Mout) continue;
    if (cin < p.Cx) out[(size_t)k * p.NK + cin] = p.alpha * acc[e];
    if (bias_wave && (lane & 31) == 0) out[(size_t)p.Mout * p.NK + k] = p.alpha * accb[e];
  }
}

// One launch takes several layers (3x3 ones of either stride, or 1x1 ones and those of stride 2 with long rows): workgroup -> (layer, k-block,
// sub-pixel / c-block, split). Every (k, c) block of one split reads the same dY rows and X patches, so they should meet in one L2: workgroups are
// handed to the eight XCDs round-robin in launch order, hence launch index i lands on XCD i % 8 as the (i / 8)-th workgroup
// of that XCD. Where the split count is a multiple of eight, XCD x takes the splits z = x (mod 8) and runs all blocks of
// a split back to back, so they are resident together and walk the pixel tiles at the same pace (a layer's workgroups start at a
// multiple of eight).
struct WgradLayer {
  WgradParams p;
  WgradGeom g;
  int tiling;  // 0..3: wgrad_dma_body for rows of 32, 16, 8, 4 pixels; 4: wgrad_flat_body; 5: wgrad_rows_body; 6..9: wgrad_s2_dma_body, 10: wgrad_s2_flat_body
  int first;   // first workgroup
  int gx, gy;  // k-blocks, (sub-pixel, c-block) pairs
};
struct WgradGroup {
  int n;
  WgradLayer layer[kWgradGroupMax];
};
static_assert(sizeof(WgradGroup) <= 4096, "kernel arguments");

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 2 : 1) void wgrad_tiles_kernel(WgradGroup grp) {
  extern __shared__ __align__(16) char smem[];
  int li = 0;
  while (li + 1 < grp.n && (int)blockIdx.x >= grp.layer[li + 1].first) ++li;
  const WgradLayer& l = grp.layer[li];
  const int lin = blockIdx.x - l.first, nblk = l.gx * l.gy;
  if (lin >= nblk * l.p.nsplit) return;
  const int xcds = (l.p.nsplit & 7) == 0 ? 3 : 0;  // log2
  const int j = lin >> xcds;
  const int z = ((j / nblk) << xcds) + (lin & ((1 << xcds) - 1)), blk = j % nblk;
  const int bx = blk % l.gx, by = blk / l.gx;
  if (WAVES == 4) {
    if (l.tiling == 4) wgrad_flat_body<true>(l.p, l.g, smem, bx, by, z);
    else wgrad_rows_body(l.p, l.g, smem, bx, by, z);
    return;
  }
  switch (l.tiling) {
    case 0: wgrad_dma_body<5, 2>(l.p, l.g, smem, bx, by, z); break;
    case 1: wgrad_dma_body<4, 3>(l.p, l.g, smem, bx, by, z); break;
    case 2: wgrad_dma_body<3, 3>(l.p, l.g, smem, bx, by, z); break;
    case 3: wgrad_dma_body<2, 2>(l.p, l.g, smem, bx, by, z); break;
    case 4: wgrad_flat_body<false>(l.p, l.g, smem, bx, by, z); break;
    case 6: wgrad_s2_dma_body<5, 1>(l.p, l.g, smem, bx, by, z); break;
    case 7: wgrad_s2_dma_body<4, 2>(l.p, l.g, smem, bx, by, z); break;
    case 8: wgrad_s2_dma_body<3, 3>(l.p, l.g, smem, bx, by, z); break;
    case 9: wgrad_s2_dma_body<2, 2>(l.p, l.g, smem, bx, by, z); break;
    case 10: wgrad_s2_flat_body(l.p, l.g, smem, bx, by, z); break;
  }
}

// ------------------------------------------------------------------ wgrad, fp32
// partial[z][m][n] = alpha * sum over the pixels of split z of dY[p][m] * X(p; n), n = (tap, c). Both operands are used as they lie
// in memory: panels of 32 pixels x 32 channels, [pixel][128 bytes], copied global -> LDS (two slots), of which 32 consecutive lanes read 32
// consecutive channels of a pixel with no conflict and a constant offset per step; a lane reads eight pixels of one channel, splits them
// into bf16 parts (split3) and has a fragment of v_mfma_f32_32x32x16_bf16. Lane l of wave w always copies pixel 8 w + l / 8 of a tile,
// 16 bytes of one tap per panel: one image position per lane and tile, stepped without a division. Any kernel size,
// stride, image size and batch; linear layers are the 1x1 case. The bias gradient is the product with a column of ones,
// in the first column of workgroups: each of its waves adds one 32-row block of it to its four (two) products. The sums of two tiles join the long
// ones together, on the vector unit. Bound by the split (176 vector instructions of a wave for 24 MFMAs of 64 x 64). The wide layers of the fp32 CNN,
// 512 images, alone, v_mfma_f32_32x32x2_f32 (64 cycles per 4 kFLOP) / parts: 256 / 174, 246 / 168, 206 / 137 us, the 3-channel stem 86 / 71.
struct Wgrad32Geom {
  int sw, sh, si;         // 32 pixels = si images + sh rows + sw columns of the output grid
};

template <int BM, int BN>
__global__ __launch_bounds__(256, 2) void wgrad_f32_kernel(WgradParams p, Wgrad32Geom g) {
  constexpr int AP = BM / 32, BP = BN / 32;           // panels
  constexpr int NI = BM / 64, NJ = BN / 64;           // 32 x 32 blocks of a wave: a quarter of the tile
  constexpr int SLOT = (AP + BP) * 4096;
  __shared__ __align__(16) char smem[2 * SLOT];
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = wave >> 1;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN, z = blockIdx.z;
  const int first = z * p.pix_per_split, end = first + p.pix_per_split;  // the last tile may be a partial one
  const int ntiles = (p.pix_per_split + 31) / 32;

  const int l8 = lane >> 3, c4 = (lane & 7) * 4;  // pixel of a fill, first channel of this lane's 16 bytes
  int pix, ow, oh, img, filled;
  auto start = [&]() {
    pix = first + wave * 8 + l8;
    const int line = pix / p.Wo;
    ow = pix - line * p.Wo;
    img = line / p.Ho;
    oh = line - img * p.Ho;
    filled = 0;
  };
  start();
  bool n_ok[BP];
  int n_r[BP], n_s[BP], n_off[BP];  // tap and element offset of this lane's columns in every panel
#pragma unroll
  for (int b = 0; b < BP; ++b) {
    const int n = n0 + 32 * b + c4;
    n_ok[b] = n < p.NK;
    const int tap = (n_ok[b] ? n : 0) / p.Cx, c = (n_ok[b] ? n : 0) - tap * p.Cx;
    n_r[b] = tap / p.S;
    n_s[b] = tap - n_r[b] * p.S;
    n_off[b] = (n_r[b] * p.W + n_s[b]) * p.Cx + c;
  }
  const float* zsrc = (const float*)p.zeros + c4;
  auto fill = [&](int slot) {  // the next tile
    if (filled++ >= ntiles) return;
    const uint32_t base = lds0 + slot * SLOT + wave * 1024;
    const bool live = pix < end;
    const float* dy = (const float*)p.dy + (long long)pix * p.ldy + m0 + c4;
#pragma unroll
    for (int a = 0; a < AP; ++a) dma16(live && m0 + 32 * a + c4 < p.ldy ? dy + 32 * a : zsrc, base + a * 4096);
    const int h = oh * p.stride - p.pad, w = ow * p.stride - p.pad;
    const float* x = (const float*)p.x + ((long long)(img * p.H + h) * p.W + w) * p.Cx;
#pragma unroll
    for (int b = 0; b < BP; ++b) {
      const bool ok = live && n_ok[b] && (unsigned)(h + n_r[b]) < (unsigned)p.H && (unsigned)(w + n_s[b]) < (unsigned)p.W;
      dma16(ok ? x + n_off[b] : zsrc, base + (AP + b) * 4096);
    }
    pix += 32;
    ow += g.sw;
    if (ow >= p.Wo) { ow -= p.Wo; ++oh; }
    oh += g.sh;
    if (oh >= p.Ho) { oh -= p.Ho; ++img; }
    img += g.si;
  };
  fill(0);

  const int l32 = (lane >> 5) * 512 + (lane & 31) * 4;  // steps pair pixels 8 i + j and 8 i + 4 + j; channel lane % 32
  const int bias_block = NI > 1 ? wave_n : 0;  // the 32-row block whose bias gradient this wave sums
  const bool bias_wave = blockIdx.y == 0 && wave_n < NI;
  f32x16_t acc[NI][NJ] = {}, inner[NI][NJ] = {}, accb = {};
  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill((t + 1) & 1);
    const char* sa = smem + (t & 1) * SLOT + wave_m * NI * 4096 + l32;
    const char* sb = smem + (t & 1) * SLOT + (AP + wave_n * NJ) * 4096 + l32;
#pragma unroll
    for (int g = 0; g < 2; ++g) {  // sixteen pixels
      float a[NI][8], b[NJ][8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int at = (2 * g + (k >> 2)) * 1024 + (k & 3) * 128;
#pragma unroll
        for (int i = 0; i < NI; ++i) a[i][k] = *(const float*)(sa + i * 4096 + at);
#pragma unroll
        for (int j = 0; j < NJ; ++j) b[j][k] = *(const float*)(sb + j * 4096 + at);
      }
      Parts x[NJ], y[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) y[i] = split3(a[i]);
#pragma unroll
      for (int j = 0; j < NJ; ++j) x[j] = split3(b[j]);
      // (Ahead of the products, not behind them: the compiler counts no wait from a product to an addition of its sums across the end of this branch.)
      if (bias_wave) {
        const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
#pragma unroll
        for (int k = 2; k >= 0; --k) {
          if (bias_block == 0) mfma16B<bf16_t>(y[0].part[k], ones, accb);
          else mfma16B<bf16_t>(y[NI - 1].part[k], ones, accb);
        }
      }
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) mfma16B<bf16_t>(y[i].part[kPartA[k]], x[j].part[kPartB[k]], inner[i][j]);
      __builtin_amdgcn_sched_barrier(0);  // (the fragments of both groups at once would not fit the registers)
    }
    if ((t & 1) || t + 1 == ntiles) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          acc[i][j] += inner[i][j];
          inner[i][j] = f32x16_t{};
        }
    }
  }
  wait_vm<0>();

  bool nan = any_nan(acc[0]) | any_nan(acc[NI - 1]);
  if (bias_wave) nan |= any_nan<1>({accb});
  if (workgroup_any(nan, smem, wave, 4)) {  // (as in conv3x3_dma_kernel)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x16_t{};
    accb = f32x16_t{};
    start();
#pragma unroll 1
    for (int t = 0; t < ntiles; ++t) {
      wg_barrier();
      fill(0);
      wait_vm<0>();
      wg_barrier();
      const char* sa = smem + wave_m * NI * 4096 + l32;
      const char* sb = smem + (AP + wave_n * NJ) * 4096 + l32;
#pragma unroll 4
      for (int ks = 0; ks < 16; ++ks) {
        float a[NI], b[NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) a[i] = *(const float*)(sa + i * 4096 + (ks >> 2) * 1024 + (ks & 3) * 128);
#pragma unroll
        for (int j = 0; j < NJ; ++j) b[j] = *(const float*)(sb + j * 4096 + (ks >> 2) * 1024 + (ks & 3) * 128);
        if (bias_wave) accb = __builtin_amdgcn_mfma_f32_32x32x2f32(bias_block == 0 ? a[0] : a[NI - 1], 1.f, accb, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    }
  }

  float* out = p.partial + (size_t)z * p.Pl;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int mb = m0 + (wave_m * NI + i) * 32;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + (wave_n * NJ + j) * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = mb + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (m < p.Mout && n < p.NK) out[(size_t)m * p.NK + n] = p.alpha * acc[i][j][e];
      }
    }
  }
  if (bias_wave && (lane & 31) == 0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = m0 + (wave_m * NI + bias_block) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      if (m < p.Mout) out[(size_t)p.Mout * p.NK + m] = p.alpha * accb[e];
    }
  }
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Problem of data-group r alone (see ConvParams::nrep): its images, outputs and weights.
template <typename T>
ConvParams replica_slice(const ConvParams& p, int r) {
  constexpr size_t ES = sizeof(T);
  ConvParams q = p;
  const size_t Nr = (size_t)(p.Nimg / p.nrep);
  const size_t in_pix = r * Nr * p.H * p.W, out_el = r * Nr * p.Ho * p.Wo * p.ldy;
  q.x = (const char*)p.x + in_pix * p.Cx * ES;
  q.y = (char*)p.y + out_el * (p.out_f32 ? 4 : ES);
  if (p.res) q.res = (const char*)p.res + out_el * ES;
  if (p.mask) q.mask = (const char*)p.mask + out_el * ES;
  if (p.bits_out) q.bits_out = (char*)p.bits_out + out_el / 8;
  if (p.maskbits) q.maskbits = (const char*)p.maskbits + out_el / 8;
  if (p.x2) q.x2 = (const char*)p.x2 + in_pix * p.Cx2 * ES;
  q.w = (const char*)p.w + (size_t)r * p.w_rep;
  if (p.w2) q.w2 = (const char*)p.w2 + (size_t)r * p.w2_rep;
  if (p.bias) q.bias = p.bias + (size_t)r * p.bias_rep;
  q.Nimg = (int)Nr;
  q.M = p.M / p.nrep;
  q.nrep = 1;
  return q;
}

// True if no tile of any kernel variant (at most 256 rows) can hold pixels of two data-groups.
inline bool replicas_tile_aligned(const ConvParams& p) {
  const int Nr = p.Nimg / p.nrep;
  if (p.dgrad && p.stride == 2) {  // rows are enumerated per parity class of the output grid
    for (int cls = 0; cls < 4; ++cls) {
      const int Hc = (p.Ho - (cls >> 1) + 1) >> 1, Wc = (p.Wo - (cls & 1) + 1) >> 1;
      if ((Nr * Hc * Wc) % 256 != 0) return false;
    }
  }
  return (Nr * p.Ho * p.Wo) % 256 == 0;
}

template <typename T>
int launch_conv_one(const ConvParams& p, hipStream_t s);

template <typename T>
int launch_conv_t(const ConvParams& p, hipStream_t s) {
  if (launch_linear(sizeof(T) == 4 ? DT_F32 : DT_BF16, p, s)) return 0;
  if (p.nrep > 1 && (p.Nimg % p.nrep != 0 || !replicas_tile_aligned(p))) {
    int family = 1;  // one launch per data-group
    for (int r = 0; r < p.nrep; ++r) family &= launch_conv_one<T>(replica_slice<T>(p, r), s);
    return family;
  }
  return launch_conv_one<T>(p, s);
}

template <typename T>
int launch_conv_one(const ConvParams& p, hipStream_t s) {
  constexpr int BKB = 64;
  if (p.nrep <= 1 && launch_linear(sizeof(T) == 4 ? DT_F32 : DT_BF16, p, s)) return 0;  // a data-group's slice
  if (sizeof(T) == 2 && launch_conv_narrow(p, s)) return p.Cx == 16;
  if (launch_dma<T>(p, s)) return 1;
  if (launch_gather<T>(p, s)) return 0;
  // dgrad of a stride-2 convolution: workgroups per parity class (class (0,0) is the largest)
  const bool s2 = p.dgrad && p.stride == 2 && p.Cx % (BKB / (int)sizeof(T)) == 0 &&
                  (p.x2 == nullptr || p.Cx2 % (BKB / (int)sizeof(T)) == 0);
  const int mc = p.Nimg * ((p.Ho + 1) / 2) * ((p.Wo + 1) / 2);
  if (p.ldy <= 32 && !s2) {  // narrow layers (16 / 32 output channels): half the padded columns
    dim3 grid(cdiv(p.M, 256), 1);
    if (p.dgrad) conv_gemm_kernel<T, 256, 32, 64, 32, BKB, true><<<grid, 256, 0, s>>>(p, 0);
    else conv_gemm_kernel<T, 256, 32, 64, 32, BKB, false><<<grid, 256, 0, s>>>(p, 0);
  } else if (p.ldy <= 64) {
    const int tpc = cdiv(mc, 256);
    dim3 grid(s2 ? 4 * tpc : cdiv(p.M, 256), cdiv(p.ldy, 64));
    if (s2) conv_gemm_kernel<T, 256, 64, 64, 64, BKB, true, true><<<grid, 256, 0, s>>>(p, tpc);
    else if (p.dgrad) conv_gemm_kernel<T, 256, 64, 64, 64, BKB, true><<<grid, 256, 0, s>>>(p, 0);
    else conv_gemm_kernel<T, 256, 64, 64, 64, BKB, false><<<grid, 256, 0, s>>>(p, 0);
  } else {
    const int tpc = cdiv(mc, 128);
    dim3 grid(s2 ? 4 * tpc : cdiv(p.M, 128), cdiv(p.ldy, 128));
    if (s2) conv_gemm_kernel<T, 128, 128, 64, 64, BKB, true, true><<<grid, 256, 0, s>>>(p, tpc);
    else if (p.dgrad) conv_gemm_kernel<T, 128, 128, 64, 64, BKB, true><<<grid, 256, 0, s>>>(p, 0);
    else conv_gemm_kernel<T, 128, 128, 64, 64, BKB, false><<<grid, 256, 0, s>>>(p, 0);
  }
  return 0;
}

// bf16 problems of whole tiles (128 pixels, 64 at stride 2) per data-group (nrep of them) go to wgrad_dma_body (3x3 stride 1 pad 1) and
// wgrad_s2_dma_body (3x3 stride 2 pad 1 on even-sized images). Returns the tiling, -1 if it is none of them.
int wgrad_dma_tiling(const WgradParams& p, int nrep, int* tiles_h) {
  const bool s1 = p.R == 3 && p.S == 3 && p.stride == 1 && p.pad == 1 && p.H == p.Ho && p.W == p.Wo;
  const bool s2 = p.R == 3 && p.S == 3 && p.stride == 2 && p.pad == 1 && p.H == 2 * p.Ho && p.W == 2 * p.Wo;
  if (!s1 && !s2) return -1;
  const int tile_log = s2 ? 6 : 7;
  if (nrep < 1 || p.P % ((1 << tile_log) * nrep) != 0) return -1;
  if (p.Cx % 8 != 0 || (p.Cx > 64 && p.Cx % 64 != 0) || p.zeros == nullptr) return -1;
  // byte offsets of patch rows relative to the tile origin are 32-bit
  if ((long long)(128 + 2 * p.W + 4) * 4 * p.Cx * 2 >= (1ll << 31) || p.Cx * 2 + 256 > kZeroBytes) return -1;
  const int lw = ilog2_exact(p.Wo), lh = ilog2_exact(p.Ho);
  if (lw < 2 || lh < 0 || p.Wo > 32) return -1;
  int th_log;  // rows of a tile
  if (lw + lh >= tile_log) { th_log = tile_log - lw; *tiles_h = p.Ho >> th_log; }
  else { th_log = lh; *tiles_h = 1; }
  const int want = s2 ? (lw == 5 ? 1 : lw == 4 ? 2 : lw == 3 ? 3 : 2) : (lw == 5 ? 2 : lw == 4 ? 3 : lw == 3 ? 3 : 2);
  if (th_log != want) return -1;
  return (s2 ? 6 : 0) + 5 - lw;
}

// Sub-pixels of a 3x3 stride-2 layer in launch order and the real tap of (virtual tap, sub-pixel offset): rows 2oy-1, 2oy, 2oy+1
int wgrad_s2_taps(int (&sub)[4], int (&rmap)[2][2]) {
  rmap[0][0] = -1; rmap[0][1] = 0; rmap[1][0] = 1; rmap[1][1] = 2;
  for (int s = 3; s >= 0; --s) sub[3 - s] = s;  // heaviest sub-pixels first: (1,1) accumulates four taps, (0,0) one
  return 4;
}

// 3x3 pad 1, stride 1 and 2, of any image size: wgrad_flat_body, wgrad_s2_flat_body. Returns the tiling, -1: not one of them.
int wgrad_flat_geometry(const WgradParams& p, int nrep, WgradGeom& wg, int* slot) {
  const bool s1 = p.R == 3 && p.S == 3 && p.stride == 1 && p.pad == 1 && p.H == p.Ho && p.W == p.Wo;
  const bool s2 = p.R == 3 && p.S == 3 && p.stride == 2 && p.pad == 1 && p.Ho == (p.H + 1) / 2 && p.Wo == (p.W + 1) / 2;
  if ((!s1 && !s2) || nrep < 1 || p.Nimg % nrep != 0 || p.Cx % 8 != 0 || p.ldy % 8 != 0) return -1;
  if (p.zeros == nullptr) return -1;
  wg.Q = p.Wo + 1;
  wg.imgs_rep = p.Nimg / nrep;
  const long long positions = (long long)wg.imgs_rep * (p.Ho + 1) * wg.Q;
  if (positions + 128 + 2 * wg.Q >= (1ll << 31) || (long long)p.Nimg * p.H * p.W >= (1ll << 31)) return -1;
  wg.dQ = make_divisor(wg.Q);
  wg.dH = make_divisor(p.Ho + 1);
  // Four planes of a tile in two slots: rows of at most 151 output pixels at stride 2. Longer ones are taken a sub-pixel at a time, where dY is copied
  // for each but a tile's rows above the image row are a quarter.
  if (s2 && 2 * (8192 + s2_flat(wg.Q).total * 128) <= 160 * 1024) {
    wg.patch_rows = s2_flat(wg.Q).total;
    wg.rep_tiles = (int)((positions + 63) / 64);
    *slot = 8192 + wg.patch_rows * 128;
    return 10;
  }
  wg.rep_tiles = (int)((positions + 127) / 128);
  wg.patch_rows = (128 + (s2 ? wg.Q + 1 : 2 * wg.Q + 2) + 7) / 8 * 8;
  *slot = 16384 + wg.patch_rows * 128;
  return 2 * *slot <= 160 * 1024 ? 4 : -1;  // rows of at most 190 (stride 2: 382) output pixels
}

// The layer's part of a launch of wgrad_tiles_kernel but for its place in it (p.nrep is looked at, p.nsplit and the pointers but
// for `zeros` are not); false: not a layer of this kernel. rep_tiles: 128-position tiles of a data-group; smem: LDS.
bool wgrad_layer(const WgradParams& p, WgradLayer& l, int* rep_tiles, int* smem) {
  l.p = p;
  l.g.cblocks = cdiv(p.Cx, 64);
  l.gx = cdiv(p.Mout, 64);
  l.gy = l.g.cblocks;
  if (p.R == 1 && p.S == 1 && p.pad == 0 && (p.stride == 1 || (p.stride == 2 && p.Ho == (p.H + 1) / 2 && p.Wo == (p.W + 1) / 2))) {
    if (p.nrep < 1 || p.P % p.nrep != 0 || p.Cx % 8 != 0 || p.ldy % 8 != 0 || p.zeros == nullptr) return false;
    if ((long long)p.Nimg * p.H * p.W >= (1ll << 31)) return false;
    l.tiling = 5;
    l.g.dQ = make_divisor(p.Wo > 1 ? p.Wo : 2);
    l.g.dH = make_divisor(p.Ho > 1 ? p.Ho : 2);
    *rep_tiles = l.g.rep_tiles = cdiv(p.P / p.nrep, 128);
    *smem = 2 * 32768;
    return true;
  }
  l.tiling = wgrad_dma_tiling(p, p.nrep, &l.g.tiles_h);
  int slot;
  switch (l.tiling) {
    case 6: slot = 8192 + S2Tile<5, 1>::patch * 128; break;
    case 7: slot = 8192 + S2Tile<4, 2>::patch * 128; break;
    case 8: slot = 8192 + S2Tile<3, 3>::patch * 128; break;
    case 9: slot = 8192 + S2Tile<2, 2>::patch * 128; break;
    case -1:
      l.tiling = wgrad_flat_geometry(p, p.nrep, l.g, &slot);
      if (l.tiling < 0) return false;
      break;
    default: {
      const int tw = p.Wo, th = p.Ho * p.Wo >= 128 ? 128 / tw : p.Ho;
      slot = 16384 + ((128 / (tw * th)) * (th + 2) * (tw + 2) + 7) / 8 * 8 * 128;
    }
  }
  if (l.tiling == 4 || l.tiling == 10) *rep_tiles = l.g.rep_tiles;
  else *rep_tiles = p.P / ((l.tiling < 4 ? 128 : 64) * p.nrep);
  *smem = 2 * slot;
  if (l.tiling == 4 && p.stride == 2) l.gy *= wgrad_s2_taps(l.g.sub, l.g.rmap);
  return true;
}

// Waves of a workgroup: which of the two kernels takes the layer.
inline int wgrad_waves(const WgradParams& p, const WgradLayer& l) { return l.tiling == 5 || (l.tiling == 4 && p.stride == 2) ? 4 : 12; }

// False: not taken, nothing launched.
bool launch_wgrad_tiles(const WgradParams* p, int n, hipStream_t s) {
  if (n < 1 || n > kWgradGroupMax) return false;
  WgradGroup g{};
  int wgs = 0, smem = 0;
  for (int i = 0; i < n; ++i) {
    WgradLayer& l = g.layer[i];
    int tiles = 0, need = 0;
    if (p[i].nrep < 1 || p[i].nsplit % p[i].nrep != 0 || !wgrad_layer(p[i], l, &tiles, &need) || wgrad_waves(p[i], l) != wgrad_waves(p[0], g.layer[0])) return false;
    const int q = p[i].nsplit / p[i].nrep;
    if (q < 1 || q > tiles) return false;  // no empty split
    l.first = wgs;
    wgs += (l.gx * l.gy * p[i].nsplit + 7) / 8 * 8;
    smem = smem > need ? smem : need;
  }
  g.n = n;
  static DeviceOnce lds[2];
  if (wgrad_waves(p[0], g.layer[0]) == 4) {
    allow_whole_lds(lds[1], (const void*)wgrad_tiles_kernel<4>);
    wgrad_tiles_kernel<4><<<wgs, 256, smem, s>>>(g);
  } else {
    allow_whole_lds(lds[0], (const void*)wgrad_tiles_kernel<12>);
    wgrad_tiles_kernel<12><<<wgs, 768, smem, s>>>(g);
  }
  return true;
}

void launch_wgrad_f32(const WgradParams& p, hipStream_t s) {
  const int BM = p.Mout <= 64 ? 64 : 128, BN = p.Mout <= 64 && p.NK <= 64 ? 64 : 128;
  Wgrad32Geom g;
  g.sw = 32 % p.Wo;
  g.sh = 32 / p.Wo % p.Ho;
  g.si = 32 / p.Wo / p.Ho;
  dim3 grid(cdiv(p.Mout, BM), cdiv(p.NK, BN), p.nsplit);
  if (BM == 128) wgrad_f32_kernel<128, 128><<<grid, 256, 0, s>>>(p, g);
  else if (BN == 128) wgrad_f32_kernel<64, 128><<<grid, 256, 0, s>>>(p, g);
  else wgrad_f32_kernel<64, 64><<<grid, 256, 0, s>>>(p, g);
}

int launch_wgrad_bf16(const WgradParams* pp, int n, hipStream_t s) {
  if (launch_wgrad_slim(pp, n, s) || launch_wgrad_tiles(pp, n, s)) return 1;
  const WgradParams& p = pp[0];
  if (n != 1 || (long long)p.nsplit * p.pix_per_split != p.P) return -1;  // no layer shares wgrad_gemm_kernel, whose splits are equal
  if (p.Mout <= 64 && p.NK + 8 <= 128) {  // few input channels and taps, e.g. a 3x3 stem without padding
    dim3 grid(cdiv(p.Mout, 64), 1, p.nsplit);
    wgrad_gemm_kernel<bf16_t, 64, 128, 32, 64><<<grid, 256, 0, s>>>(p);
  } else if (p.Mout <= 64) {
    dim3 grid(cdiv(p.Mout, 64), cdiv(p.NK + 8, 256), p.nsplit);
    wgrad_gemm_kernel<bf16_t, 64, 256, 64, 64><<<grid, 256, 0, s>>>(p);
  } else {
    dim3 grid(cdiv(p.Mout, 128), cdiv(p.NK + 8, 128), p.nsplit);
    wgrad_gemm_kernel<bf16_t, 128, 128, 64, 64><<<grid, 256, 0, s>>>(p);
  }
  return 0;
}

}  // namespace

void allow_whole_lds(DeviceOnce& once, const void* kernel) {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return;
  once(device, [kernel] { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess; });
}

int launch_conv(int dt, const ConvParams& p, hipStream_t s) {
  return dt == DT_F32 ? launch_conv_t<float>(p, s) : launch_conv_t<bf16_t>(p, s);
}

int launch_wgrad(int dt, const WgradParams* p, int n, hipStream_t s) {
  if (dt != DT_F32) return launch_wgrad_bf16(p, n, s);
  for (int i = 0; i < n; ++i) launch_wgrad_f32(p[i], s);
  return 0;
}

WgradWork wgrad_work(int dt, const WgradParams& shape) {
  WgradWork w{};
  if (dt == DT_F32) return w;
  int smem = 0;
  WgradLayer l;
  if (const int tiles = wgrad_slim_tiles(shape, shape.nrep, &w.key)) {
    w.blocks = 1;
    w.tiles = tiles;
    w.key += 4;
  } else if (wgrad_layer(shape, l, &w.tiles, &smem)) {
    w.blocks = l.gx * l.gy;
    w.key = wgrad_waves(shape, l) == 4 ? 2 : 1;
  }
  return w;
}

// Split count of the kernels that take any layer.
static int wgrad_generic_split(int dt, const WgradParams& shape) {
  const int Mout = shape.Mout, NK = shape.NK, W = shape.nrep;
  const int per_replica = shape.P / W;  // pixels of one replica's mini-batch
  const int ce = dtype_ce(dt);
  const int bke = 128 / dtype_size(dt);
  int tiles = (Mout <= 64) ? cdiv(Mout, 64) * cdiv(NK + ce, 256) : cdiv(Mout, 128) * cdiv(NK + ce, 128);
  // about 1024 workgroups of wgrad_gemm_kernel's tiles; in fp32, too, whose launches have other tiles, so that a sum is split as it
  // always was (fp32 CNN: 512 and 256 the same within 0.5 %)
  int q = cdiv(1024, tiles * W);
  int qmax = per_replica / (2 * bke);  // at least two k-tiles per split
  if (qmax < 1) qmax = 1;
  if (q > qmax) q = qmax;
  if (q * W > 256) q = 256 / W;
  if (q < 1) q = 1;
  while (q > 1 && per_replica % q != 0) --q;  // splits never straddle replicas
  return W * q;
}

void wgrad_choose_splits(int dt, const WgradParams* shapes, int n, bool one_module, int* nsplit) {
  const WgradWork w0 = wgrad_work(dt, shapes[0]);
  if (w0.key == 0) {
    for (int i = 0; i < n; ++i) nsplit[i] = wgrad_generic_split(dt, shapes[i]);
    return;
  }
  long long total = 0;
  for (int i = 0; i < n; ++i) {
    const WgradWork w = wgrad_work(dt, shapes[i]);
    total += (long long)w.blocks * w.tiles * shapes[i].nrep;
  }
  bool one_per_cu = false;  // by LDS
  for (int i = 0; i < n && w0.key == 2; ++i) {
    WgradLayer l;
    int tiles = 0, lds = 0;
    wgrad_layer(shapes[i], l, &tiles, &lds);
    one_per_cu = one_per_cu || lds > 80 * 1024;
  }
  // Workgroups of the launch. The partial sums cost HBM traffic in proportion to the split counts (written here, read by the
  // update), and a workgroup of the wide kernel keeps others of its kind off the CU: half of the chip, three quarters where each
  // has 32 tiles all the same. ms per 8 steps with 128 / 192 / 256: ResNet-18 in four modules 17.3 / 17.0 / 17.4, 64 images of it 4.3 /
  // 4.4 / 4.6; ResNet-20 in one module 3.50 / 3.58 / 3.59. A workgroup of 1x1 layers has four waves where one of 3x3 layers has twelve, and of
  // stride-2 layers of long rows the four sub-pixels carry 4 : 2 : 2 : 1 taps: twice as many, or two rounds where rows are so long that one takes
  // more than half of a CU's LDS and 384 would be one and a half (128 -> 128 channels from 512 x 512 pixels, two images, 453 -> 270 us). A stride-1 layer that
  // shares its launch with no other has no launch to save its partial sums for: the chip (3 -> 256 channels at 32 x 32, 62
  // images, 128 / 256: 30.7 / 19.0 us), but not where other modules want it too (a net of 32 and 64 channels in two modules, us per 8
  // steps, 128 / 256: 400 images of 32 x 32 2025 / 2099, 256 of them 1603 / 1676, 300 of 28 x 28 1571 / 1560). Narrow layers: two or three share a CU
  // (256 / 384 / 512: ResNet-56 in eight modules 18.6 / 18.3 / 18.2, ResNet-20 in one 3.56 / 3.50 / 3.48, its normalised form in two
  // 11.9 / 11.7 / 11.5; 768 for layers of up to 16 channels, three of whose workgroups fit a CU: ResNet-20 in one 3.02 / 3.01, in one with
  // normalisation 12.2 / 12.3, ResNet-56 the same), less an eighth: tiles of images and batches of powers of two make every one of 512
  // workgroups, and the update of so many splits and other modules' launches lose more than this one gains (512 / 448 / 384: ResNet-20
  // in two modules, four data-groups of 64 2.67 / 2.61 / 2.62, of 128 4.00 / 3.89 / 3.93, of 194 5.18 / 5.22 / 5.28, in one, 256 images, 3.36 /
  // 3.32 / 3.33; ResNet-56, four of 64, 5.39 / 5.31 / 5.28).
  int target_wgs = w0.key > 4 ? 448 : total >= 192 * 32 ? 192 : 128;
  if (w0.key == 2) target_wgs = one_per_cu && target_wgs == 192 ? 512 : 2 * target_wgs;
  if (w0.key == 1 && n == 1 && one_module) target_wgs = 256;
  const long long per_wg = (total + target_wgs - 1) / target_wgs;  // tiles a workgroup walks
  for (int i = 0; i < n; ++i) {
    const WgradWork w = wgrad_work(dt, shapes[i]);
    long long q = (w.tiles + per_wg - 1) / per_wg;
    if (q * shapes[i].nrep > 512) q = 512 / shapes[i].nrep;
    nsplit[i] = shapes[i].nrep * (int)(q < 1 ? 1 : q);
  }
}

}  // namespace dds
