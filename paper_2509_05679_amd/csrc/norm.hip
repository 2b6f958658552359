// Training-mode batch normalisation for gfx950, forward and backward, with statistics per
// data-group (each group normalises over its own B*H*W values per channel). HBM-bound: every
// kernel streams [rows][ld] NHWC tensors once. Reductions run in fp64 registers inside a
// workgroup and are combined across workgroups in a fixed order, so results are reproducible.
//
//   forward : mu, var over the group's rows; xhat = (x - mu) * rstd; v = alpha * (gamma * xhat + beta) + res;
//             y = relu ? max(v, 0) : v   (+ sign plane of y)
//   backward: g = alpha * dy;  dbeta = sum g;  dgamma = sum g * xhat;
//             dx = gamma * rstd * (g - dbeta / m - xhat * dgamma / m),  m = rows per group
// The backward uses the mean, rstd and gamma that the forward of the same mini-batch stored.
#include "norm_fold.h"

namespace dds {
namespace {

struct bf16_t { uint16_t v; };

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
// two floats -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
// 0x00010001 where both halves of a packed bf16 pair are > 0, 0 / 1 per half otherwise
__device__ __forceinline__ uint32_t positive_pair(uint32_t w) {
  typedef short s16x2_t __attribute__((ext_vector_type(2)));
  const s16x2_t one = {1, 1}, zero = {0, 0};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_elementwise_min(__builtin_bit_cast(s16x2_t, w), one), zero));
}

// Eight consecutive channels of one row. Channel strides are multiples of 8 (bf16) or 4 (fp32):
// `full` is false for the last group of an fp32 row whose stride is 4 mod 8 (upper half absent).
template <typename T>
__device__ __forceinline__ void load8(const void* base, size_t elem, bool full, float (&f)[8]) {
  if (sizeof(T) == 2) {
    const uint4 v = *(const uint4*)((const char*)base + elem * 2);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[2 * i] = bf2f((uint16_t)(w[i] & 0xffffu)); f[2 * i + 1] = bf2f((uint16_t)(w[i] >> 16)); }
  } else {
    const float4 a = *(const float4*)((const char*)base + elem * 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    if (full) {
      const float4 b = *(const float4*)((const char*)base + elem * 4 + 16);
      f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    } else {
      f[4] = f[5] = f[6] = f[7] = 0.f;
    }
  }
}

// Stores eight channels and returns their sign byte (bit i = stored value i > 0).
template <typename T>
__device__ __forceinline__ uint32_t store8(void* base, size_t elem, bool full, const float (&f)[8]) {
  if (sizeof(T) == 2) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack_bf16(f[2 * i], f[2 * i + 1]);
    *(uint4*)((char*)base + elem * 2) = make_uint4(w[0], w[1], w[2], w[3]);
    // pair i's low half belongs to bit 2 i, its high half (bit 16) to bit 2 i + 1
    uint32_t t = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) t |= positive_pair(w[i]) << (2 * i);
    return (t | (t >> 15)) & 0xffu;
  } else {
    *(float4*)((char*)base + elem * 4) = make_float4(f[0], f[1], f[2], f[3]);
    if (full) *(float4*)((char*)base + elem * 4 + 16) = make_float4(f[4], f[5], f[6], f[7]);
    uint32_t t = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) t |= (f[i] > 0.f ? 1u : 0u) << i;
    return t;
  }
}

// Thread layout shared by the four kernels: 256 threads = rpp rows x cg channel groups of 8.
struct Lane {
  int tg, tr, rpp, c0;
  bool active, full;
  long long row_lo, row_hi;  // this workgroup's rows (absolute)
};

__device__ __forceinline__ Lane make_lane(const BnParams& p, long long rows_per_split) {
  Lane l;
  const int cg = (p.ld + 7) / 8;
  l.rpp = 256 / cg;
  l.tg = threadIdx.x % cg;
  l.tr = threadIdx.x / cg;
  l.active = l.tr < l.rpp;
  l.c0 = 8 * l.tg;
  l.full = l.c0 + 8 <= p.ld;
  const int split = blockIdx.x, rep = blockIdx.y;
  const long long lo = (long long)split * rows_per_split;
  const long long hi = lo + rows_per_split < p.rows_per_rep ? lo + rows_per_split : p.rows_per_rep;
  l.row_lo = (long long)rep * p.rows_per_rep + lo;
  l.row_hi = (long long)rep * p.rows_per_rep + hi;
  return l;
}

// this thread's eight entries of a per-channel table row (16-byte aligned, ld is a multiple of 4)
__device__ __forceinline__ void load_coef(const float* row, const Lane& l, float (&f)[8]) {
  const int c0 = l.active ? l.c0 : 0;
  const float4 a = *(const float4*)(row + c0);
  const float4 b = *(const float4*)(row + (l.full ? c0 + 4 : c0));
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}

// Second half of the workgroup reduction. red[v * 256 + thread] holds quantity v (0-7: first sum of the
// thread's eight channels, 8-15: second sum) of every thread; thread = row-thread t * cg + channel group g.
// `parts` neighbouring threads (a power of two) share an output (v, g): each adds every parts-th row-thread in order, so that
// no chain of dependent LDS reads and fp64 additions is longer than 16 for rows of 8, 16, 32, ... channels (one thread per output
// walked 128 row-threads of a 16-channel row); a tree joins them. scale * total goes to out[channel * 2 + (v >> 3)],
// channel = 8 g + (v & 7).
__device__ __forceinline__ void fold_rows(const double* red, int cg, int rpp, int ld, double scale, double* out) {
  const int outputs = 16 * cg;
  int plog = 0;
  while ((outputs << (plog + 1)) <= 256) ++plog;
  const int parts = 1 << plog, part = threadIdx.x & (parts - 1);
  for (int o = threadIdx.x >> plog; o < outputs; o += 256 >> plog) {
    const int v = o / cg, g = o - v * cg;
    const int c = 8 * g + (v & 7);
    double a = 0.0;
#pragma unroll 4
    for (int t = part; t < rpp; t += parts) a += red[v * 256 + t * cg + g];
    for (int d = 1; d < parts; d <<= 1) a += __shfl_xor(a, d, 64);  // the partners have the same o
    if (part == 0 && c < ld) out[c * 2 + (v >> 3)] = scale * a;
  }
}

// ------------------------------------------------------------------ forward
// grid (nsums, W). scratch[((rep * nsums + split) * ld + c) * 2 + {0, 1}] = sum x, sum x^2 over the split's rows.
template <typename T>
__global__ __launch_bounds__(256) void bn_fwd_stats_kernel(BnParams p) {
  const Lane l = make_lane(p, p.rows_per_sum);
  const int cg = (p.ld + 7) / 8;
  double s[8], ss[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) s[i] = ss[i] = 0.0;
  if (l.active) {
    // four rows per trip: four independent 16-byte loads in flight per thread
    long long r = l.row_lo + l.tr;
    for (; r + 3 * l.rpp < l.row_hi; r += 4 * l.rpp) {
      float f[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) load8<T>(p.x, (size_t)(r + u * l.rpp) * p.ld + l.c0, l.full, f[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) { s[i] += (double)f[u][i]; ss[i] += (double)f[u][i] * (double)f[u][i]; }
    }
    for (; r < l.row_hi; r += l.rpp) {
      float f[8];
      load8<T>(p.x, (size_t)r * p.ld + l.c0, l.full, f);
#pragma unroll
      for (int i = 0; i < 8; ++i) { s[i] += (double)f[i]; ss[i] += (double)f[i] * (double)f[i]; }
    }
  }
  __shared__ double red[16 * 256];
#pragma unroll
  for (int i = 0; i < 8; ++i) { red[i * 256 + threadIdx.x] = s[i]; red[(8 + i) * 256 + threadIdx.x] = ss[i]; }
  __syncthreads();
  fold_rows(red, cg, l.rpp, p.ld, 1.0, p.scratch + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * p.ld * 2);
}

// grid (ld / 4, W), 256 threads = 64 split lanes x 4 channels (ld is a multiple of four): folds the nsums partial sums of a
// channel (lane j takes splits j, j+64, ...; a tree over the sixteen lanes of a wave, then the four waves in order) once per
// data-group and leaves the per-channel factors of the streaming kernel in coef[rep][.][ld], so that each of its
// threads starts with a few 16-byte loads instead of dozens of scalar ones.
template <bool BWD>
__global__ __launch_bounds__(256) void bn_finalize_kernel(BnParams p) {
  const int rep = blockIdx.y, lane4 = threadIdx.x >> 2;
  const int c = blockIdx.x * 4 + (threadIdx.x & 3);
  const ChannelInputs in = channel_inputs<BWD>(p, rep, c);
  double a = 0.0, b = 0.0;
#pragma unroll 4
  for (int sp = lane4; sp < p.nsums; sp += 64) {
    const double2 v = *(const double2*)(p.scratch + (((size_t)rep * p.nsums + sp) * p.ld + c) * 2);
    a += v.x;
    b += v.y;
  }
#pragma unroll
  for (int d = 4; d < 64; d <<= 1) {
    a += __shfl_xor(a, d, 64);
    b += __shfl_xor(b, d, 64);
  }
  __shared__ double red[2][4][4];
  if ((threadIdx.x & 63) < 4) {
    red[0][threadIdx.x >> 6][threadIdx.x & 3] = a;
    red[1][threadIdx.x >> 6][threadIdx.x & 3] = b;
  }
  __syncthreads();
  if (threadIdx.x >= 4) return;
  a = b = 0.0;
  for (int j = 0; j < 4; ++j) { a += red[0][j][threadIdx.x]; b += red[1][j][threadIdx.x]; }
  channel_factors<BWD>(p, in, rep, c, a, b, true, p.coef + (size_t)rep * kBnCoefRows * p.ld + c, p.ld);
}

// grid (nsplit, W): streams its rows; FOLD: the factors are made here, from the splits' sums. HBM-bound (reads x and the residual,
// writes y and 1/16 of it in sign bits); the rows of a trip are requested before anything is computed, the first ones
// before the per-channel factors, and stores and sign bits are packed conversions. Average over the ResNet-18 shapes at
// 4 x 128 (33 MB tensors): 16 us, 5.2 TB/s; with 32 scalar loads of statistics in front of the first row and
// conversions in integer arithmetic it was 30 us (backward: 15.5 against 25 us).
template <typename T, bool FOLD>
__global__ __launch_bounds__(256) void bn_fwd_apply_kernel(BnParams p) {
  Lane l = make_lane(p, p.rows_per_split);
  __shared__ __align__(16) float cf[FOLD ? 2 * kBnFoldLd : 4];
  const bool active = l.active;
  if (!active) {
    if (!FOLD) return;
    l.tg = l.tr = l.c0 = 0;  // reads with the first thread and takes part in the fold
    l.full = p.ld >= 8;
  }
  const float* coef = FOLD ? cf : p.coef + (size_t)blockIdx.y * kBnCoefRows * p.ld;
  const int stride = FOLD ? kBnFoldLd : p.ld;
  float scale[8], shift[8];
  auto load_rows = [&](long long r, float (&f)[4][8], float (&q)[4][8]) {  // rows past the end read the last one again
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long ru = r + u * l.rpp < l.row_hi ? r + u * l.rpp : l.row_hi - 1;
      load8<T>(p.x, (size_t)ru * p.ld + l.c0, l.full, f[u]);
      if (p.res) load8<T>(p.res, (size_t)ru * p.ld + l.c0, l.full, q[u]);
    }
  };
  float f[4][8], q[4][8];
  long long r = l.row_lo + l.tr;
  SplitFold<false, 256> fold;
  __shared__ double red[FOLD ? SplitFold<false, 256>::kDoubles : 1];
  if (FOLD) fold.request(p, blockIdx.y);
  load_rows(r, f, q);
  if (FOLD) fold.finish(p, blockIdx.y, blockIdx.x == 0, red, cf);
  if (!active) return;
  load_coef(coef, l, scale);
  load_coef(coef + stride, l, shift);
  for (;;) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long ru = r + u * l.rpp;
      if (ru >= l.row_hi) break;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float v = fmaf(f[u][i], scale[i], shift[i]);
        if (p.res) v += q[u][i];
        if (p.relu) v = v > 0.f ? v : 0.f;
        f[u][i] = v;
      }
      const uint32_t bits = store8<T>(p.y, (size_t)ru * p.ld + l.c0, l.full, f[u]);
      // the sign of the stored (rounded) value, as the convolution epilogues define the plane
      if (p.bits_out) ((uint8_t*)p.bits_out)[(size_t)ru * (p.ld / 8) + l.tg] = (uint8_t)bits;
    }
    r += 4 * l.rpp;
    if (r >= l.row_hi) break;
    load_rows(r, f, q);
  }
}

// ------------------------------------------------------------------ backward
// grid (nsums, W). scratch[((rep * nsums + split) * ld + c) * 2 + {0, 1}] = sum g, sum g * xhat over the split's
// rows, g = alpha * dy.
template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_stats_kernel(BnParams p) {
  const Lane l = make_lane(p, p.rows_per_sum);
  const int cg = (p.ld + 7) / 8;
  const int rep = blockIdx.y;
  const float* st = p.stats + (size_t)rep * 3 * p.ld;
  float mean[8], rstd[8];
  load_coef(st, l, mean);
  load_coef(st + p.ld, l, rstd);
  double s[8], ss[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) s[i] = ss[i] = 0.0;
  if (l.active) {
    long long r = l.row_lo + l.tr;
    for (; r + 3 * l.rpp < l.row_hi; r += 4 * l.rpp) {
      float f[4][8], g[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t e = (size_t)(r + u * l.rpp) * p.ld + l.c0;
        load8<T>(p.x, e, l.full, f[u]);
        load8<T>(p.dy, e, l.full, g[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float xh = (f[u][i] - mean[i]) * rstd[i];
          s[i] += (double)g[u][i];
          ss[i] += (double)g[u][i] * (double)xh;
        }
    }
    for (; r < l.row_hi; r += l.rpp) {
      const size_t e = (size_t)r * p.ld + l.c0;
      float f[8], g[8];
      load8<T>(p.x, e, l.full, f);
      load8<T>(p.dy, e, l.full, g);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float xh = (f[i] - mean[i]) * rstd[i];
        s[i] += (double)g[i];
        ss[i] += (double)g[i] * (double)xh;
      }
    }
  }
  __shared__ double red[16 * 256];
#pragma unroll
  for (int i = 0; i < 8; ++i) { red[i * 256 + threadIdx.x] = s[i]; red[(8 + i) * 256 + threadIdx.x] = ss[i]; }
  __syncthreads();
  fold_rows(red, cg, l.rpp, p.ld, (double)p.alpha, p.scratch + ((size_t)rep * gridDim.x + blockIdx.x) * p.ld * 2);
}

// grid (nsplit, W): streams dx from dy, x and the per-channel factors, laid out as the forward streaming kernel.
template <typename T, bool FOLD>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(BnParams p) {
  Lane l = make_lane(p, p.rows_per_split);
  __shared__ __align__(16) float cf[FOLD ? 5 * kBnFoldLd : 4];
  const bool active = l.active;
  if (!active) {
    if (!FOLD) return;
    l.tg = l.tr = l.c0 = 0;  // reads with the first thread and takes part in the fold
    l.full = p.ld >= 8;
  }
  const float* coef = FOLD ? cf : p.coef + (size_t)blockIdx.y * kBnCoefRows * p.ld;
  const int stride = FOLD ? kBnFoldLd : p.ld;
  float mean[8], rstd[8], k0[8], k1[8], k2[8];
  auto load_rows = [&](long long r, float (&f)[4][8], float (&g)[4][8]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long ru = r + u * l.rpp < l.row_hi ? r + u * l.rpp : l.row_hi - 1;
      load8<T>(p.x, (size_t)ru * p.ld + l.c0, l.full, f[u]);
      load8<T>(p.dy, (size_t)ru * p.ld + l.c0, l.full, g[u]);
    }
  };
  float f[4][8], g[4][8];
  long long r = l.row_lo + l.tr;
  SplitFold<true, 256> fold;
  __shared__ double red[FOLD ? SplitFold<true, 256>::kDoubles : 1];
  if (FOLD) fold.request(p, blockIdx.y);
  load_rows(r, f, g);
  if (FOLD) fold.finish(p, blockIdx.y, blockIdx.x == 0, red, cf);
  if (!active) return;
  load_coef(coef, l, mean);
  load_coef(coef + stride, l, rstd);
  load_coef(coef + 2 * stride, l, k0);
  load_coef(coef + 3 * stride, l, k1);
  load_coef(coef + 4 * stride, l, k2);
  for (;;) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long ru = r + u * l.rpp;
      if (ru >= l.row_hi) break;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float xh = (f[u][i] - mean[i]) * rstd[i];
        f[u][i] = k0[i] * g[u][i] - k1[i] - xh * k2[i];
      }
      (void)store8<T>(p.dx, (size_t)ru * p.ld + l.c0, l.full, f[u]);
    }
    r += 4 * l.rpp;
    if (r >= l.row_hi) break;
    load_rows(r, f, g);
  }
}

}  // namespace

// Row splits. Sums: about 32 KiB of the tensor each, at most 512 of a data-group. For rows of at most kBnFoldLd channels the
// streaming kernel can fold the splits itself: 2 us of it (16 channels, 776 images of 32 x 32: 9.8 -> 11.9 us) for a launch of 4 us
// and the gap before it. A lane folds eight splits, so there are fewer of them then (kBnFoldSums / ld), and streaming workgroups have at
// least twice the bytes that they fold, as long as there is one per CU. Not where that would leave fewer than half of the workgroups that
// sum and CUs without one (64 channels, 128 images of 32 x 32 each: 512 splits -> 32). Steps of normalised ResNet-20, with the
// launch / here: one data-group of 194 in one module 0.962 / 0.889 ms, in two 0.690 / 0.607, four in one 1.660 / 1.538, in
// two 1.292 / 1.231.
BnPlan bn_plan(int W, long long rows_per_rep, int ld, int es) {
  BnPlan b;
  const long long bytes = rows_per_rep * ld * es;
  auto clamp = [](long long v, long long lo, long long hi) { return v < lo ? lo : v > hi ? hi : v; };
  auto rows = [&](long long splits) { return (rows_per_rep + splits - 1) / splits; };
  long long sums = clamp(bytes / 32768, 1, 512), splits = sums;
  const long long few = clamp(512 / W, 1, kBnFoldSums / (ld > 32 ? 64 : ld > 16 ? 32 : ld > 8 ? 16 : 8));
  b.fold = ld <= kBnFoldLd && (2 * few >= sums || W * few >= 256);
  if (b.fold) {
    if (sums > few) sums = few;
    splits = clamp(splits, 1, clamp(bytes / (32ll * sums * ld), (256 + W - 1) / W, 512));
  }
  b.rows_per_sum = rows(sums);
  b.rows_per_split = rows(splits);
  b.nsums = (int)((rows_per_rep + b.rows_per_sum - 1) / b.rows_per_sum);
  b.nsplit = (int)((rows_per_rep + b.rows_per_split - 1) / b.rows_per_split);
  return b;
}

#define DDS_BN_DISPATCH(dt, KERNEL, ...)               \
  do {                                                 \
    if ((dt) == DT_F32) KERNEL<float> __VA_ARGS__;     \
    else KERNEL<bf16_t> __VA_ARGS__;                   \
  } while (0)
#define DDS_BN_DISPATCH_FOLD(dt, fold, KERNEL, ...)                                      \
  do {                                                                                   \
    if ((dt) == DT_F32) { if (fold) KERNEL<float, true> __VA_ARGS__; else KERNEL<float, false> __VA_ARGS__; }   \
    else { if (fold) KERNEL<bf16_t, true> __VA_ARGS__; else KERNEL<bf16_t, false> __VA_ARGS__; }                \
  } while (0)

void launch_bn_forward(int dt, const BnParams& p, hipStream_t s) {
  DDS_BN_DISPATCH(dt, bn_fwd_stats_kernel, <<<dim3(p.nsums, p.W), 256, 0, s>>>(p));
  if (p.streamed_later) return;
  if (!p.fold) bn_finalize_kernel<false><<<dim3(p.ld / 4, p.W), 256, 0, s>>>(p);
  DDS_BN_DISPATCH_FOLD(dt, p.fold, bn_fwd_apply_kernel, <<<dim3(p.nsplit, p.W), 256, 0, s>>>(p));
}

void launch_bn_backward(int dt, const BnParams& p, hipStream_t s) {
  DDS_BN_DISPATCH(dt, bn_bwd_stats_kernel, <<<dim3(p.nsums, p.W), 256, 0, s>>>(p));
  if (p.streamed_later) return;
  if (!p.fold) bn_finalize_kernel<true><<<dim3(p.ld / 4, p.W), 256, 0, s>>>(p);
  DDS_BN_DISPATCH_FOLD(dt, p.fold, bn_bwd_apply_kernel, <<<dim3(p.nsplit, p.W), 256, 0, s>>>(p));
}

}  // namespace dds
