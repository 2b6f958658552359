// Plain matrix products of few rows (linear layers, 1x1 stride-1 convolutions on small images), forward and dgrad:
//   y[m, n] = epilogue( sum_k x[m, k] * w[n, k] )
// The tiled kernels of gemm.hip hand such a product to a handful of workgroups that walk the whole reduction, one
// memory round trip and barrier per k-tile: the 3072 -> 256 layer of the perceptron (64 rows, fp32) kept two
// workgroups busy for 192 k-tiles. Here a tile is 16 x 16. In bf16 the eight waves of a workgroup split its reduction once
// each has a k-step of its own: 15 -> 4.3 us for a ResNet's 512 -> 10 head. In fp32 one wave walks it, twelve k-steps
// requested ahead, in the order of the tiled kernels: every sum is theirs bit for bit, and the perceptron's 8 iterations take
// 0.75-0.80 ms instead of 2.38 (a split over eight waves: 0.70-0.75 ms, but other sums). Bound by latency, past one or two
// tiles per CU by L2.
#include "kernels.h"

namespace dds {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

struct bf16_t { uint16_t v; };

template <typename T> __device__ __forceinline__ f32x4_t mfma16x16(const uint4& a, const uint4& b, f32x4_t c);
template <> __device__ __forceinline__ f32x4_t mfma16x16<bf16_t>(const uint4& a, const uint4& b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
// fp32 products are added in the order of the tiled kernels of gemm.hip (0, 4, 1, 5, 2, 6, 3, 7 of every eight), so that a
// layer's sums do not depend on which kernel its row count selects: swapping half-waves between neighbouring
// components puts k = 0 4 1 5, 2 6 3 7, 8 12 9 13 and 10 14 11 15 of the 16 in the four lane groups of one instruction each.
__device__ __forceinline__ void swap_halves(uint32_t& lo, uint32_t& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
  lo = r[0];
  hi = r[1];
}
template <> __device__ __forceinline__ f32x4_t mfma16x16<float>(const uint4& a_, const uint4& b_, f32x4_t c) {
  uint4 a = a_, b = b_;
  swap_halves(a.x, a.y); swap_halves(a.z, a.w);
  swap_halves(b.x, b.y); swap_halves(b.z, b.w);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
template <typename T> __device__ __forceinline__ void load4(const void* p, size_t i, float (&v)[4]);
template <> __device__ __forceinline__ void load4<float>(const void* p, size_t i, float (&v)[4]) {
  const float4 t = *(const float4*)((const float*)p + i);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ __forceinline__ void load4<bf16_t>(const void* p, size_t i, float (&v)[4]) {
  const uint2 t = *(const uint2*)((const uint16_t*)p + i);
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
}

// NW waves; KS of them share one 16 x 16 tile (NW / KS tiles along n per workgroup). Weights are the MFMA A operand
// (rows n), activations the B operand (columns m): lane l = 16 g + j supplies the 16 bytes g of a 64-byte k-step of
// weight row j and of activation row j, and ends with output channels 4 g .. 4 g + 3 of row j. Loads go straight from
// global memory (a k-step reads 64 contiguous bytes of 16 rows), UN k-steps ahead of their use; the partial tiles
// of the KS waves meet in LDS and are added in a fixed order by the tile's first wave.
template <typename T, int KS, int NW>
__global__ __launch_bounds__(64 * NW) void linear_kernel(ConvParams p) {
  constexpr int ES = sizeof(T), TILES = NW / KS, UN = sizeof(T) == 4 ? 12 : 4;
  __shared__ f32x4_t red[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int ks = wave % KS;
  const int m0 = blockIdx.x * 16, n0 = (blockIdx.y * TILES + wave / KS) * 16;
  const char* wbase = (const char*)p.w;
  const float* bias = p.bias;
  if (p.nrep > 1) {  // the launcher made sure that 16 rows never straddle two data-groups
    const int r = min(m0 / (p.M / p.nrep), p.nrep - 1);
    wbase += (size_t)r * p.w_rep;
    if (bias) bias += (size_t)r * p.bias_rep;
  }
  const int rowbytes = p.Cx * ES;              // a multiple of 16
  const int steps = (rowbytes + 63) >> 6;
  const int s0 = steps * ks / KS, s1 = steps * (ks + 1) / KS;
  const bool mok = m0 + j < p.M, nok = n0 + j < p.Nout;
  const char* xrow = (const char*)p.x + (size_t)(mok ? m0 + j : 0) * rowbytes;
  const char* wrow = wbase + (size_t)(nok ? n0 + j : 0) * rowbytes;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  uint4 xa[UN], wa[UN];
  // unconditional loads from clamped addresses; what lies past a row's end or past the last row is zeroed
  auto load = [&](int s) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int off = (s + u) * 64 + g * 16;
      const bool ok = s + u < s1 && off < rowbytes;
      const uint4 a = *(const uint4*)(wrow + (ok ? off : 0)), b = *(const uint4*)(xrow + (ok ? off : 0));
      const uint32_t ka = ok && nok ? 0xffffffffu : 0u, kb = ok && mok ? 0xffffffffu : 0u;
      wa[u] = make_uint4(a.x & ka, a.y & ka, a.z & ka, a.w & ka);
      xa[u] = make_uint4(b.x & kb, b.y & kb, b.z & kb, b.w & kb);
    }
  };
  if (s0 < s1) load(s0);
  for (int s = s0; s < s1; s += UN) {
    uint4 xc[UN], wc[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) { xc[u] = xa[u]; wc[u] = wa[u]; }
    if (s + UN < s1) load(s + UN);
#pragma unroll
    for (int u = 0; u < UN; ++u) acc = mfma16x16<T>(wc[u], xc[u], acc);
  }
  if (KS > 1) {
    red[wave][lane] = acc;
    __syncthreads();
    if (ks != 0) return;
#pragma unroll
    for (int k = 1; k < KS; ++k) acc += red[wave + k][lane];
  }

  // epilogue of four consecutive channels n .. n + 3 of row m
  const int m = m0 + j, n = n0 + 4 * g;
  const bool ok = m < p.M && n < p.ldy;
  const size_t o = ok ? (size_t)m * p.ldy + n : 0;
  float rs[4] = {0.f, 0.f, 0.f, 0.f};
  uint32_t keep = 0xfu;
  if (p.res) load4<T>(p.res, o, rs);
  if (p.maskbits) {
    keep = (uint32_t)((const uint8_t*)p.maskbits)[o >> 3] >> (n & 4);
  } else if (p.mask) {
    float mk[4];
    load4<T>(p.mask, o, mk);
    keep = (mk[0] > 0.f ? 1u : 0u) | (mk[1] > 0.f ? 2u : 0u) | (mk[2] > 0.f ? 4u : 0u) | (mk[3] > 0.f ? 8u : 0u);
  }
  const float lower = p.relu ? 0.f : -__builtin_inff();
  float v[4];
  uint32_t signs = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float b = bias != nullptr && n + e < p.Nout ? p.alpha * bias[n + e] : 0.f;
    float t = fmaf(p.alpha, acc[e], b) + rs[e];
    t = __builtin_amdgcn_fmed3f(t, lower, __builtin_inff());
    v[e] = ((keep >> e) & 1u) ? t : 0.f;
    signs |= (v[e] > 0.f ? 1u : 0u) << e;
  }
  if (ok) {
    if (sizeof(T) == 4 || p.out_f32) *(float4*)((float*)p.y + o) = make_float4(v[0], v[1], v[2], v[3]);
    else *(uint2*)((uint16_t*)p.y + o) = make_uint2(pack_bf16_rne(v[0], v[1]), pack_bf16_rne(v[2], v[3]));
  }
  if (p.bits_out) {  // ldy is a multiple of 8: lane groups 2 i and 2 i + 1 hold the two nibbles of a byte
    const uint32_t other = (uint32_t)__shfl_xor((int)signs, 16, 64);
    if (ok && (g & 1) == 0) ((uint8_t*)p.bits_out)[o >> 3] = (uint8_t)(signs | (other << 4));
  }
}

template <typename T>
bool launch_linear_t(const ConvParams& p, hipStream_t s) {
  const int steps = (p.Cx * (int)sizeof(T) + 63) / 64;
  if constexpr (sizeof(T) == 4) linear_kernel<T, 1, 1><<<dim3((p.M + 15) / 16, (p.ldy + 15) / 16), 64, 0, s>>>(p);
  // eight waves per tile once each has a k-step of its own, else a tile per wave
  else if (steps >= 8) linear_kernel<T, 8, 8><<<dim3((p.M + 15) / 16, (p.ldy + 15) / 16), 512, 0, s>>>(p);
  else linear_kernel<T, 1, 8><<<dim3((p.M + 15) / 16, (p.ldy + 127) / 128), 512, 0, s>>>(p);
  return true;
}

// Where the 16 x 16 tiles pay. A tile reads its 16 weight and 16 activation rows from L2, so past one or two tiles per CU
// the time grows with tiles x (trips of the load loop), while a tiled kernel of gemm.hip takes the time of one workgroup's
// reduction, whatever the number of rows, until it has a workgroup for every CU: its k-steps times the cost of a stage,
// which the width of its tile sets (32, 64 or 128 columns). Both sides were timed on 1298 shapes a type (16 to 24576 rows, 32 to
// 2048 deep, 16 to 2048 columns). The lines below are where they meet: the side taken is the faster one or within 22 % of it
// (bf16 of 160 to 224 channels takes 6.3 us where the tiled kernel takes 5.2).
// us, linear / conv_gather_kernel / conv_gemm_kernel, columns x depth x rows:
//   bf16 128 x 1024 x 512 4.5 / 9.3 / 23, x 1024 6.3 / 9.4 / 23, x 2048 9.9 / 9.4 / 23, x 8192 33 / 9.9 / 23
//   bf16 64 x 256 x 2048 6.3 / 6.9 / 12, x 4096 9.9 / 6.9 / 12
//   fp32 128 x 512 x 2048 12 / 42 / 47, x 8192 39 / 43 / 48, x 16384 73 / 43 / 48; 64 x 32 x 4096 6.2 / 6.3 / 9.8, x 8192 9.2 / 6.5 / 10
// conv_gemm_kernel takes the channel counts that conv_gather_kernel refuses, at 1.1 to 2.5 times its time, and has lines of
// its own (within 30 %, at the shortest reductions 53 %).
bool few_tiles(int dt, const ConvParams& p, int steps) {
  const bool gather = p.Cx % (64 / dtype_size(dt)) == 0 && p.ldy == p.Nout;
  const int width = p.ldy <= 32 ? 0 : p.ldy <= 64 ? 1 : 2;  // column tile of the alternative
  const long long rows = (p.M + 15) / 16, tiles = rows * ((p.ldy + 15) / 16);
  if (dt == DT_F32) {  // one wave a tile, twelve steps a trip
    const int line[2][3] = {{3000, 4500, 4500}, {1800, 2500, 4200}};
    return tiles * ((steps + 11) / 12 * 12 + 8) <= (long long)line[gather][width] * (steps + 8);
  }
  if (steps < 8) return rows * ((p.ldy + 127) / 128) * ((steps + 3) / 4) <= (!gather ? 768 : width < 2 ? 512 : 256);
  const int slope[2][3] = {{90, 90, 90}, {38, 45, 24}};
  return tiles * ((steps + 31) / 32) <= 128 + slope[gather][width] * steps;
}

}  // namespace

// True if the launch was taken: a plain product (1x1, stride 1, no padding) of few rows and columns.
bool launch_linear(int dt, const ConvParams& p, hipStream_t s) {
  if (p.R != 1 || p.S != 1 || p.stride != 1 || p.pad != 0 || p.x2 != nullptr) return false;
  const long long tiles = (long long)((p.M + 127) / 128) * ((p.ldy + 127) / 128);
  if (tiles > 128 || (p.ldy + 15) / 16 > 65535) return false;
  if (!few_tiles(dt, p, (p.Cx * dtype_size(dt) + 63) / 64)) return false;
  if (p.nrep > 1 && (p.M % p.nrep != 0 || (p.M / p.nrep) % 16 != 0)) return false;
  return dt == DT_F32 ? launch_linear_t<float>(p, s) : launch_linear_t<bf16_t>(p, s);
}

}  // namespace dds
