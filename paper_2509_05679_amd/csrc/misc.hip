// Bandwidth-bound kernels for gfx950: batch ingest (layout + precision change),
// pooling, softmax cross-entropy, the fused replica-mean + SGD update, weight
// snapshots and parameter layout conversion. All tensors are NHWC with a channel
// stride that is a multiple of one 16-byte chunk.
#include "kernels.h"

namespace dds {
namespace {

struct bf16_t { uint16_t v; };

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// A 16-byte chunk viewed as CE floats.
template <typename T> struct Chunk;
template <> struct Chunk<float> {
  static constexpr int CE = 4;
  float f[4];
  __device__ __forceinline__ void load(const void* p) { uint4 v = *(const uint4*)p; f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w); }
  __device__ __forceinline__ void store(void* p) const { *(uint4*)p = make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])); }
};
template <> struct Chunk<bf16_t> {
  static constexpr int CE = 8;
  float f[8];
  __device__ __forceinline__ void load(const void* p) {
    uint4 v = *(const uint4*)p;
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[2 * i] = bf2f((uint16_t)(w[i] & 0xffffu)); f[2 * i + 1] = bf2f((uint16_t)(w[i] >> 16)); }
  }
  __device__ __forceinline__ void store(void* p) const {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)f2bf(f[2 * i]) | ((uint32_t)f2bf(f[2 * i + 1]) << 16);
    *(uint4*)p = make_uint4(w[0], w[1], w[2], w[3]);
  }
};

// ------------------------------------------------------------------ ingest
// caller batch [B][C][HW] fp32 (per replica) -> [W*B][HW][Cpad] T, zero channel padding
template <typename T>
__global__ void ingest_kernel(IngestParams p) {
  constexpr int CE = Chunk<T>::CE;
  const int chunks = p.Cpad / CE;
  const long long total = (long long)p.W * p.B * p.HW * chunks;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (long long)p.W * p.B) p.labels[i] = p.y[i / p.B][i % p.B];
  if (i >= total) return;
  // pixel index varies fastest across threads when the image has a spatial extent
  // (coalesced fp32 reads); chunk index fastest for flat inputs
  int n, hw, ch;
  if (p.HW > 1) {
    hw = (int)(i % p.HW);
    long long r = i / p.HW;
    ch = (int)(r % chunks);
    n = (int)(r / chunks);
  } else {
    hw = 0;
    ch = (int)(i % chunks);
    n = (int)(i / chunks);
  }
  const int s = n / p.B, b = n - s * p.B;
  const float* src = p.x[s] + (size_t)b * p.C * p.HW;
  Chunk<T> c;
#pragma unroll
  for (int e = 0; e < CE; ++e) {
    const int ci = ch * CE + e;
    c.f[e] = ci < p.C ? src[(size_t)ci * p.HW + hw] : 0.f;
  }
  c.store((char*)p.dst + (((size_t)n * p.HW + hw) * p.Cpad + (size_t)ch * CE) * sizeof(T));
}

// ------------------------------------------------------------------ pooling
template <typename T>
__global__ void maxpool_fwd_kernel(const char* x, char* y, int N, int H, int W, int C) {
  constexpr int CE = Chunk<T>::CE;
  const int chunks = C / CE, Ho = H / 2, Wo = W / 2;
  const long long total = (long long)N * Ho * Wo * chunks;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int ch = (int)(i % chunks);
  long long r = i / chunks;
  const int ow = (int)(r % Wo); r /= Wo;
  const int oh = (int)(r % Ho);
  const int n = (int)(r / Ho);
  Chunk<T> best, c;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const size_t off = ((((size_t)n * H + 2 * oh + (q >> 1)) * W + 2 * ow + (q & 1)) * C + (size_t)ch * CE) * sizeof(T);
    if (q == 0) best.load(x + off);
    else {
      c.load(x + off);
#pragma unroll
      for (int e = 0; e < CE; ++e) best.f[e] = c.f[e] > best.f[e] ? c.f[e] : best.f[e];
    }
  }
  best.store(y + ((((size_t)n * Ho + oh) * Wo + ow) * C + (size_t)ch * CE) * sizeof(T));
}

// gradient to the first maximum of each window (row-major order, strict comparisons);
// optionally times the ReLU derivative of the pre-pool tensor
template <typename T>
__global__ void maxpool_bwd_kernel(const char* dy, const char* x, char* dx, int N, int H, int W, int C, int relu_mask) {
  constexpr int CE = Chunk<T>::CE;
  const int chunks = C / CE, Ho = H / 2, Wo = W / 2;
  const long long total = (long long)N * Ho * Wo * chunks;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int ch = (int)(i % chunks);
  long long r = i / chunks;
  const int ow = (int)(r % Wo); r /= Wo;
  const int oh = (int)(r % Ho);
  const int n = (int)(r / Ho);
  Chunk<T> c[4], g;
  size_t off[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    off[q] = ((((size_t)n * H + 2 * oh + (q >> 1)) * W + 2 * ow + (q & 1)) * C + (size_t)ch * CE) * sizeof(T);
    c[q].load(x + off[q]);
  }
  g.load(dy + ((((size_t)n * Ho + oh) * Wo + ow) * C + (size_t)ch * CE) * sizeof(T));
  Chunk<T> o[4];
#pragma unroll
  for (int e = 0; e < CE; ++e) {
    int arg = 0;
    float best = c[0].f[e];
#pragma unroll
    for (int q = 1; q < 4; ++q)
      if (c[q].f[e] > best) { best = c[q].f[e]; arg = q; }
    const float gv = (relu_mask && !(best > 0.f)) ? 0.f : g.f[e];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q].f[e] = (q == arg) ? gv : 0.f;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q].store(dx + off[q]);
}

// Global average pool. A workgroup is (16-byte channel chunks of a pixel, row-lanes, images): the row-lanes of an image take
// every blockDim.y-th pixel and their partial sums are folded through LDS in a fixed order (blockIdx.y: chunks beyond the
// workgroup's). fp32 sums keep the order of the pixels, so there a lane walks all of them (ROWS false).
// Bound by latency while images are few, then by HBM. us, one thread per chunk that walks all pixels / one workgroup per
// image / here: bf16 8 x 8 x 64, 194 images 11 / 3.9 / 4.0; 2 x 2 x 16, 8192 images 2.9 / 40 / 2.7 (an image's 128
// row-lanes had four pixels); fp32 8 x 8 x 64, 194 images 8.8 / 8.2 / 8.1, 8192 images 22 / 77 / 22 (16 of 256 lanes were in use).
template <typename T, bool ROWS>
__global__ __launch_bounds__(256) void gap_fwd_kernel(const char* x, char* y, int N, int HW, int C) {
  constexpr int CE = Chunk<T>::CE;
  const int per = blockDim.x, rows = ROWS ? blockDim.y : 1, r = ROWS ? threadIdx.y : 0;
  const int ch = blockIdx.y * per + threadIdx.x, n = blockIdx.x * blockDim.z + threadIdx.z;
  const bool ok = n < N && ch < C / CE;
  Chunk<T> c;
  float acc[CE];
#pragma unroll
  for (int e = 0; e < CE; ++e) acc[e] = 0.f;
  if (ok) {
#pragma unroll ROWS ? 4 : 16
    for (int q = r; q < HW; q += rows) {
      c.load(x + (((size_t)n * HW + q) * C + (size_t)ch * CE) * sizeof(T));
#pragma unroll
      for (int e = 0; e < CE; ++e) acc[e] += c.f[e];
    }
  }
  if constexpr (ROWS) {
    __shared__ float red[256 * CE];
    const int at = (threadIdx.z * rows + r) * per + threadIdx.x;
#pragma unroll
    for (int e = 0; e < CE; ++e) red[e * 256 + at] = acc[e];
    __syncthreads();
    if (r != 0) return;
    for (int j = 1; j < rows; ++j)
#pragma unroll
      for (int e = 0; e < CE; ++e) acc[e] += red[e * 256 + at + j * per];
  }
  if (!ok) return;
  const float inv = 1.f / (float)HW;
#pragma unroll
  for (int e = 0; e < CE; ++e) c.f[e] = acc[e] * inv;
  c.store(y + ((size_t)n * C + (size_t)ch * CE) * sizeof(T));
}

template <typename T>
__global__ void gap_bwd_kernel(const char* dy, const char* x, char* dx, int N, int HW, int C, int relu_mask) {
  constexpr int CE = Chunk<T>::CE;
  const int chunks = C / CE;
  const long long total = (long long)N * HW * chunks;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int ch = (int)(i % chunks);
  const long long r = i / chunks;
  const int n = (int)(r / HW);
  Chunk<T> g, c;
  g.load(dy + ((size_t)n * C + (size_t)ch * CE) * sizeof(T));
  const size_t off = ((size_t)r * C + (size_t)ch * CE) * sizeof(T);
  const float inv = 1.f / (float)HW;
  if (relu_mask) c.load(x + off);
#pragma unroll
  for (int e = 0; e < CE; ++e) {
    float v = g.f[e] * inv;
    if (relu_mask && !(c.f[e] > 0.f)) v = 0.f;
    g.f[e] = v;
  }
  g.store(dx + off);
}

// ------------------------------------------------------------------ softmax cross-entropy
// One workgroup per data-group, a thread per sample row, a fixed-order tree for the loss sum. Bound by latency: one to a few rows per thread
// at the turn of the backward pass. Rows of at most 16 classes are read at once and kept (MAXC = 16; class by class, three times over, the
// kernel took 5.7 us at 10 classes and 194 samples, here 3.9); wider ones class by class (MAXC = 0). Sums in the order of the classes.
template <typename T, int MAXC>
__global__ __launch_bounds__(256) void softmax_ce_kernel(const float* logits, const int32_t* labels, char* dlogits,
                                                         float* loss, int B, int classes, int ldl, int ldg) {
  __shared__ float red[256];
  const int s = blockIdx.x;
  float lsum = 0.f;
  const float invB = 1.f / (float)B;
  for (int b = threadIdx.x; b < B; b += 256) {
    const size_t row = (size_t)s * B + b;
    const float* z = logits + row * ldl;
    const int y = labels[row];
    float zc[MAXC > 0 ? MAXC : 1];
    float mx, se = 0.f, zy;
    if (MAXC > 0) {
#pragma unroll
      for (int c = 0; c < MAXC; c += 4) {  // (a row's stride is a multiple of four floats; chunks past it repeat the last one)
        const float4 v = *(const float4*)(z + min(c, ldl - 4));
        zc[c] = v.x; zc[c + 1] = v.y; zc[c + 2] = v.z; zc[c + 3] = v.w;
      }
      mx = zy = zc[0];
#pragma unroll
      for (int c = 1; c < MAXC; ++c) {
        mx = c < classes && zc[c] > mx ? zc[c] : mx;
        zy = c == y ? zc[c] : zy;
      }
#pragma unroll
      for (int c = 0; c < MAXC; ++c) {
        const float e = __expf(zc[c] - mx);
        se = c < classes ? se + e : se;
      }
    } else {
      mx = z[0];
      for (int c = 1; c < classes; ++c) mx = z[c] > mx ? z[c] : mx;
      for (int c = 0; c < classes; ++c) se += __expf(z[c] - mx);
      zy = z[y];
    }
    const float lse = __logf(se);
    lsum += -(zy - mx - lse);
    auto gradient = [&](int c, float zv) { return c < classes ? (__expf(zv - mx - lse) - (c == y ? 1.f : 0.f)) * invB : 0.f; };
    if (dlogits) {
      char* out = dlogits + row * ldg * sizeof(T);
      if (MAXC > 0) {  // the stride of a gradient row is at most MAXC
#pragma unroll
        for (int c0 = 0; c0 < MAXC; c0 += Chunk<T>::CE) {
          Chunk<T> g;
#pragma unroll
          for (int e = 0; e < Chunk<T>::CE; ++e) g.f[e] = gradient(c0 + e, zc[(c0 + e) % (MAXC > 0 ? MAXC : 1)]);
          if (c0 < ldg) g.store(out + c0 * sizeof(T));
        }
      } else {
        for (int c0 = 0; c0 < ldg; c0 += Chunk<T>::CE) {
          Chunk<T> g;
#pragma unroll
          for (int e = 0; e < Chunk<T>::CE; ++e) g.f[e] = c0 + e < classes ? gradient(c0 + e, z[c0 + e]) : 0.f;
          g.store(out + c0 * sizeof(T));
        }
      }
    }
  }
  if (loss) {
    red[threadIdx.x] = lsum;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[s] = red[0] * invB;
  }
}

// ------------------------------------------------------------------ update
// One workgroup owns a tile of E weights of one tap, E / KC output channels x KC input channels (update_width: whole cache lines of a
// partial row where the layer is that wide), or E biases, and all of their nsplit partial rows (map entry: descriptor, tile). A row of the tile is read by E / 4 lanes, 16 bytes each, so the 256
// threads read R = 1024 / E rows at a time, eight such reads in flight per thread; row-lane r sums the splits r, r + R, ...
// The new weights leave three times: fp32 master, compute-precision copy, and, transposed through LDS, the snapshot
// [cin][tap][cout] that the backward pass of a later iteration multiplies by. (With the snapshot in a launch of its own, which read
// the master again, the pair took 125 us of a ResNet-18 step, modules one after another, here 75; 135 / 85 of ResNet-56, 20 / 16 of ResNet-20
// in one module; the three-layer perceptron, bound by its launches, went from 0.79 to 0.70 ms per 8 steps.)
// HBM-bound when enough reads are in flight: 4 bytes per partial value. E falls with the split count (update_elems).
// Order of the sum (bit-reproducible for a given split count): eight interleaved running sums, a fixed tree over
// them, a tree over the row-lanes of a wave, a fixed tree over the four waves through LDS.
// g = sum/W; v = mu*v + g; w -= lr*v (or lr*g).
__device__ __forceinline__ void add4(float4& a, const float4& b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; }

template <typename T, int E>
__device__ __forceinline__ void update_tile(const UpdateDesc& d, int tile_index, int slot, float invW, float lr, float mu, float4* red, float* tile) {
  constexpr int LPR = E / 4;      // lanes per row
  constexpr int R = 256 / LPR;    // row-lanes of the workgroup
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r0 = threadIdx.x / LPR, l = threadIdx.x % LPR;
  const int KC = update_width(d.Cinpad), KK = E / KC, cshift = __builtin_ctz(KC) - 2, kshift = __builtin_ctz(KK) - 1;
  const int kblocks = (d.Cout + KK - 1) / KK, cblocks = (d.Cinpad + KC - 1) / KC;
  const bool weights = tile_index < d.RS * cblocks * kblocks;
  int kb = 0, cb = 0, tap = 0;
  long long base;
  bool live;
  if (weights) {
    const int q = tile_index / kblocks;
    kb = tile_index - q * kblocks;
    tap = q / cblocks;
    cb = q - tap * cblocks;
    const int k = kb * KK + (l >> cshift), c = cb * KC + (l & ((1 << cshift) - 1)) * 4;
    live = k < d.Cout && c < d.Cinpad;
    base = ((long long)k * d.RS + tap) * d.Cinpad + c;
  } else {
    base = (long long)d.Cout * d.RS * d.Cinpad + (long long)(tile_index - d.RS * cblocks * kblocks) * E + l * 4;
    live = base < d.n;
  }
  float4 a[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live) {  // rows are pstride = n rounded up to 4 floats long: the vector read stays inside the row
    const float* src = d.partial + base;
    for (int j = r0; j < d.nsplit; j += 8 * R) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int jj = j + R * u;
        if (jj < d.nsplit) add4(a[u], *(const float4*)(src + (size_t)jj * d.pstride));
      }
    }
  }
#pragma unroll
  for (int w = 4; w > 0; w >>= 1)
#pragma unroll
    for (int u = 0; u < w; ++u) add4(a[u], a[u + w]);
#pragma unroll
  for (int o = 32; o >= LPR; o >>= 1)
    add4(a[0], make_float4(__shfl_xor(a[0].x, o, 64), __shfl_xor(a[0].y, o, 64), __shfl_xor(a[0].z, o, 64), __shfl_xor(a[0].w, o, 64)));
  if (E < 1024) {
    if (wave > 0 && lane < LPR) red[(wave - 1) * 64 + lane] = a[0];
    __syncthreads();
  }
  if (E == 1024 || (wave == 0 && lane < LPR)) {
    if (E < 1024) {
      const float4 r1 = red[lane], r2 = red[64 + lane], r3 = red[128 + lane];
      a[0].x = (a[0].x + r1.x) + (r2.x + r3.x); a[0].y = (a[0].y + r1.y) + (r2.y + r3.y);
      a[0].z = (a[0].z + r1.z) + (r2.z + r3.z); a[0].w = (a[0].w + r1.w) + (r2.w + r3.w);
    }
    float g[4] = {a[0].x * invW, a[0].y * invW, a[0].z * invW, a[0].w * invW};
    float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live && base + 4 <= d.n) {
      w = *(const float4*)(d.master + base);
      if (d.momentum) {
        float4 v = *(const float4*)(d.momentum + base);
        v.x = mu * v.x + g[0]; v.y = mu * v.y + g[1]; v.z = mu * v.z + g[2]; v.w = mu * v.w + g[3];
        *(float4*)(d.momentum + base) = v;
        g[0] = v.x; g[1] = v.y; g[2] = v.z; g[3] = v.w;
      }
      w.x -= lr * g[0]; w.y -= lr * g[1]; w.z -= lr * g[2]; w.w -= lr * g[3];
      *(float4*)(d.master + base) = w;
      if (d.work) {
        if (sizeof(T) == 2) {
          uint2 o;
          o.x = (uint32_t)f2bf(w.x) | ((uint32_t)f2bf(w.y) << 16);
          o.y = (uint32_t)f2bf(w.z) | ((uint32_t)f2bf(w.w) << 16);
          *(uint2*)((char*)d.work + base * 2) = o;
        } else {
          *(float4*)((char*)d.work + base * 4) = w;
        }
      }
    } else if (live) {  // the last biases of a layer
      for (long long i = base; i < d.n; ++i) {
        float wi = d.master[i];
        float gg = g[i - base];
        if (d.momentum) { const float v = mu * d.momentum[i] + gg; d.momentum[i] = v; gg = v; }
        wi -= lr * gg;
        d.master[i] = wi;
        if (d.work) {
          if (sizeof(T) == 2) ((uint16_t*)d.work)[i] = f2bf(wi);
          else ((float*)d.work)[i] = wi;
        }
      }
    }
    if (weights && d.stash) {  // zeros for the output channels past the last
      float* at = tile + (l & ((1 << cshift) - 1)) * 4 * (KK + 1) + (l >> cshift);
      at[0] = w.x; at[KK + 1] = w.y; at[2 * (KK + 1)] = w.z; at[3 * (KK + 1)] = w.w;
    }
  }
  if (!weights || !d.stash) return;  // the whole workgroup
  __syncthreads();
  // two output channels of one input channel per thread and turn
#pragma unroll
  for (int i = 0; i < (E / 2 + 255) / 256; ++i) {
    const int o = i * 256 + threadIdx.x;
    if (E < 512 && o >= E / 2) break;
    const int cl = o >> kshift, kl = (o & ((1 << kshift) - 1)) * 2;
    const int c = cb * KC + cl, k = kb * KK + kl;
    if (c >= d.Cin || k >= d.Coutpad) continue;
    const float v0 = tile[cl * (KK + 1) + kl], v1 = tile[cl * (KK + 1) + kl + 1];
    const size_t at = (size_t)slot * d.stash_slot_elems + ((size_t)c * d.RS + tap) * d.Coutpad + k;
    if (sizeof(T) == 2) *(uint32_t*)((uint16_t*)d.stash + at) = (uint32_t)f2bf(v0) | ((uint32_t)f2bf(v1) << 16);
    else *(float2*)((float*)d.stash + at) = make_float2(v0, v1);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void update_kernel(const UpdateDesc* descs, const int* tile_map, int slot, float invW, float lr, float mu) {
  __shared__ float4 red[3 * 64];
  __shared__ float tile[32 * 33];
  const UpdateDesc d = descs[tile_map[2 * blockIdx.x]];
  const int t = tile_map[2 * blockIdx.x + 1];
  switch (update_elems(sizeof(T) == 4 ? DT_F32 : DT_BF16, d.nsplit)) {
    case 64: update_tile<T, 64>(d, t, slot, invW, lr, mu, red, tile); break;
    case 256: update_tile<T, 256>(d, t, slot, invW, lr, mu, red, tile); break;
    default: update_tile<T, 1024>(d, t, slot, invW, lr, mu, red, tile); break;
  }
}

// work <- master (precision change only)
template <typename T>
__global__ __launch_bounds__(256) void recast_kernel(const UpdateDesc* descs, const int* block_map) {
  const UpdateDesc d = descs[block_map[2 * blockIdx.x]];
  const long long base = (long long)block_map[2 * blockIdx.x + 1] * 1024 + threadIdx.x * 4;
  if (!d.work) return;
  for (long long i = base; i < d.n && i < base + 4; ++i) {
    if (sizeof(T) == 2) ((uint16_t*)d.work)[i] = f2bf(d.master[i]);
    else ((float*)d.work)[i] = d.master[i];
  }
}

// Update (a)/(b) of Section 3.3 with a general mixing matrix P, for all W data-groups at once:
//   g_r = sum of data-group r's q splits (fixed order), v_r = mu*v_r + g_r, u_r = w_r - lr*v_r (or lr*g_r),
//   w_s = sum_r P[s][r] * u_r (r ascending, fp32), written to the fp32 master and the compute-precision copy.
// descs / range_map: data-group 0's entries (its `partial` points at split 0 of all W*q splits); data-group
// r's master / momentum / work lie r*rep_stride elements further.
// A workgroup owns E elements in all W copies, so the update is in place. Its four waves take the data-groups
// r = wave, wave + 4, ...: a partial row of the range is read by E / 4 lanes, the wave's 256 / E row-lanes take every
// (256 / E)-th split with eight reads in flight each, and u_r goes to LDS; after one barrier all threads share the W * E
// mixed values. HBM-bound; E falls with the split count for the reason given at update_kernel. (One thread per four
// elements that walked all W * q rows itself took 78 us per module of the ResNet-18 shapes with W = 4, this 50; an
// eight-module ResNet-56 on a ring of eight groups went from 2.38 to 1.85 ms per iteration.)
// Every layer's arrays are allocated in whole multiples of 64 elements and split rows in multiples of 4, so the
// four-wide accesses of the last thread of a layer stay inside that layer's padding.
template <typename T, int E>
__device__ __forceinline__ void gossip_range(const UpdateDesc& d, long long first, const float* P, int W, long long rep_stride,
                                             float lr, float mu, float4* u) {
  constexpr int LPR = E / 4, RL = 64 / LPR;  // lanes per row, row-lanes of a wave
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = d.nsplit;  // splits per data-group of this layer
  const int rl = lane / LPR, l = lane % LPR;
  const long long base = first + l * 4;
  for (int r = wave; r < W; r += 4) {
    float4 a[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (base < d.n) {
      const float* src = d.partial + (size_t)r * q * d.pstride + base;
      for (int j = rl; j < q; j += 8 * RL) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int jj = j + RL * k;
          if (jj < q) add4(a[k], *(const float4*)(src + (size_t)jj * d.pstride));
        }
      }
    }
#pragma unroll
    for (int w = 4; w > 0; w >>= 1)
#pragma unroll
      for (int k = 0; k < w; ++k) add4(a[k], a[k + w]);
#pragma unroll
    for (int o = 32; o >= LPR; o >>= 1)
      add4(a[0], make_float4(__shfl_xor(a[0].x, o, 64), __shfl_xor(a[0].y, o, 64), __shfl_xor(a[0].z, o, 64), __shfl_xor(a[0].w, o, 64)));
    if (rl != 0 || base >= d.n) continue;
    float4 g = a[0];
    if (d.momentum) {
      float4* vp = (float4*)(d.momentum + (long long)r * rep_stride + base);
      float4 v = *vp;
      v.x = mu * v.x + g.x; v.y = mu * v.y + g.y; v.z = mu * v.z + g.z; v.w = mu * v.w + g.w;
      *vp = v;
      g = v;
    }
    const float4 w = *(const float4*)(d.master + (long long)r * rep_stride + base);
    u[r * LPR + l] = make_float4(w.x - lr * g.x, w.y - lr * g.y, w.z - lr * g.z, w.w - lr * g.w);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < W * LPR; i += 256) {
    const int s = i / LPR, ll = i % LPR;
    const long long b = first + ll * 4;
    if (b >= d.n) continue;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r = 0; r < W; ++r) {
      const float c = P[s * W + r];
      const float4 t = u[r * LPR + ll];
      a.x = fmaf(c, t.x, a.x); a.y = fmaf(c, t.y, a.y); a.z = fmaf(c, t.z, a.z); a.w = fmaf(c, t.w, a.w);
    }
    *(float4*)(d.master + (long long)s * rep_stride + b) = a;
    if (d.work) {
      if (sizeof(T) == 2) {
        uint2 o;
        o.x = (uint32_t)f2bf(a.x) | ((uint32_t)f2bf(a.y) << 16);
        o.y = (uint32_t)f2bf(a.z) | ((uint32_t)f2bf(a.w) << 16);
        *(uint2*)((char*)d.work + ((long long)s * rep_stride + b) * 2) = o;
      } else {
        *(float4*)((char*)d.work + ((long long)s * rep_stride + b) * 4) = a;
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void gossip_update_kernel(const UpdateDesc* descs, const int* range_map, const float* P,
                                                            int W, long long rep_stride, float lr, float mu) {
  extern __shared__ float4 u[];  // [W][E / 4], E <= 256
  const UpdateDesc d = descs[range_map[2 * blockIdx.x]];
  const long long first = (long long)range_map[2 * blockIdx.x + 1] * 32;
  switch (gossip_elems(d.nsplit)) {
    case 32: gossip_range<T, 32>(d, first, P, W, rep_stride, lr, mu, u); break;
    case 64: gossip_range<T, 64>(d, first, P, W, rep_stride, lr, mu, u); break;
    default: gossip_range<T, 256>(d, first, P, W, rep_stride, lr, mu, u); break;
  }
}

// Disagreement between data-groups (experiment section). Workgroup b owns 1024 elements of one
// layer (block_map entry b of data-group 0) and writes, for part 0 (weight) and 1 (bias) and every
// data-group s, sum_i (w_s[i] - mean_r w_r[i])^2 over its elements of that part, in fp64, to
// out[(2*b + part) * W + s]. The host adds the blocks of a tensor in order and takes the square
// root of the maximum.
__global__ __launch_bounds__(256) void consensus_kernel(const UpdateDesc* descs, const int* block_map, int W,
                                                        long long rep_stride, double* out) {
  const UpdateDesc d = descs[block_map[2 * blockIdx.x]];
  const long long blk0 = (long long)block_map[2 * blockIdx.x + 1] * 1024;
  const long long nw = d.n - d.Cout;
  double acc[2][32];
#pragma unroll
  for (int r = 0; r < 32; ++r) acc[0][r] = acc[1][r] = 0.0;
  for (int it = 0; it < 4; ++it) {
    const long long i = blk0 + it * 256 + threadIdx.x;
    if (i >= d.n) break;
    float w[32];
    double mean = 0.0;
#pragma unroll
    for (int r = 0; r < 32; ++r)
      if (r < W) { w[r] = d.master[(long long)r * rep_stride + i]; mean += (double)w[r]; }
    mean /= (double)W;
    const bool is_bias = i >= nw;
#pragma unroll
    for (int r = 0; r < 32; ++r)
      if (r < W) {
        const double e = (double)w[r] - mean;
        acc[0][r] += is_bias ? 0.0 : e * e;
        acc[1][r] += is_bias ? e * e : 0.0;
      }
  }
  __shared__ double red[256];
#pragma unroll
  for (int part = 0; part < 2; ++part)
#pragma unroll
    for (int r = 0; r < 32; ++r) {
      if (r >= W) continue;  // uniform
      red[threadIdx.x] = acc[part][r];
      __syncthreads();
      for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
      }
      if (threadIdx.x == 0) out[((size_t)2 * blockIdx.x + part) * W + r] = red[0];
      __syncthreads();
    }
}

// transposed snapshot: stash[slot][c][tap][kpad] <- master[k][tap][cpad], zero for k >= Cout.
// One workgroup moves a 64(k) x 64(c) tile of one tap through LDS so that both the reads
// (64 consecutive c) and the writes (64 consecutive k) are whole cache lines.
// block_map[2*blk+1] = tile index = (tap * cblocks + cb) * kblocks + kb.
template <typename T>
__global__ __launch_bounds__(256) void stash_kernel(const UpdateDesc* descs, const int* block_map, int slot) {
  const UpdateDesc d = descs[block_map[2 * blockIdx.x]];
  if (!d.stash) return;
  __shared__ float tile[64][65];
  const int kblocks = (d.Coutpad + 63) / 64, cblocks = (d.Cin + 63) / 64;
  int t = block_map[2 * blockIdx.x + 1];
  const int kb = t % kblocks; t /= kblocks;
  const int cb = t % cblocks;
  const int tap = t / cblocks;
  const int ty = threadIdx.x >> 6, tx = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int k = kb * 64 + ty * 16 + i, c = cb * 64 + tx;
    tile[ty * 16 + i][tx] = (k < d.Cout && c < d.Cinpad) ? d.master[((size_t)k * d.RS + tap) * d.Cinpad + c] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = cb * 64 + ty * 16 + i, k = kb * 64 + tx;
    if (c < d.Cin && k < d.Coutpad) {
      const size_t o = (size_t)slot * d.stash_slot_elems + ((size_t)c * d.RS + tap) * d.Coutpad + k;
      const float v = tile[tx][ty * 16 + i];
      if (sizeof(T) == 2) ((uint16_t*)d.stash)[o] = f2bf(v);
      else ((float*)d.stash)[o] = v;
    }
  }
}

__global__ void param_permute_kernel(const float* canon, float* internal, int Cout, int Cin, int RS, int Cinpad, int to_internal) {
  const long long total = (long long)Cout * RS * Cinpad + Cout;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const long long nw = (long long)Cout * RS * Cinpad;
  const long long nwc = (long long)Cout * Cin * RS;
  if (i >= nw) {  // bias
    const long long k = i - nw;
    if (to_internal) internal[i] = canon[nwc + k];
    else ((float*)canon)[nwc + k] = internal[i];
    return;
  }
  const int c = (int)(i % Cinpad);
  const long long r = i / Cinpad;
  const int tap = (int)(r % RS);
  const int k = (int)(r / RS);
  if (c >= Cin) { if (to_internal) internal[i] = 0.f; return; }
  const size_t ci = ((size_t)k * Cin + c) * RS + tap;
  if (to_internal) internal[i] = canon[ci];
  else ((float*)canon)[ci] = internal[i];
}

__global__ void fill_zero_kernel(uint4* p, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

inline unsigned blocks_for(long long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

#define DDS_DISPATCH(dt, KERNEL, ...)                  \
  do {                                                 \
    if ((dt) == DT_F32) KERNEL<float> __VA_ARGS__;     \
    else KERNEL<bf16_t> __VA_ARGS__;                   \
  } while (0)

void launch_ingest(int dt, const IngestParams& p, hipStream_t s) {
  const long long total = (long long)p.W * p.B * p.HW * (p.Cpad / dtype_ce(dt));
  const long long n = total > (long long)p.W * p.B ? total : (long long)p.W * p.B;
  DDS_DISPATCH(dt, ingest_kernel, <<<blocks_for(n, 256), 256, 0, s>>>(p));
}

void launch_maxpool_fwd(int dt, const void* x, void* y, int N, int H, int W, int C, hipStream_t s) {
  const long long total = (long long)N * (H / 2) * (W / 2) * (C / dtype_ce(dt));
  DDS_DISPATCH(dt, maxpool_fwd_kernel, <<<blocks_for(total, 256), 256, 0, s>>>((const char*)x, (char*)y, N, H, W, C));
}

void launch_maxpool_bwd(int dt, const void* dy, const void* x, void* dx, int N, int H, int W, int C, int relu_mask,
                        hipStream_t s) {
  const long long total = (long long)N * (H / 2) * (W / 2) * (C / dtype_ce(dt));
  DDS_DISPATCH(dt, maxpool_bwd_kernel,
               <<<blocks_for(total, 256), 256, 0, s>>>((const char*)dy, (const char*)x, (char*)dx, N, H, W, C, relu_mask));
}

void launch_gap_fwd(int dt, const void* x, void* y, int N, int HW, int C, hipStream_t s) {
  const int chunks = C / dtype_ce(dt);
  if (dt == DT_F32) {  // one image a workgroup up to 1023 images, then as many as fill a wave
    const int per = chunks < 256 ? chunks : 256, most = per < 64 ? 64 / per : 1, want = N / 512;
    const int imgs = want < 1 ? 1 : want < most ? want : most;
    gap_fwd_kernel<float, false><<<dim3(blocks_for(N, imgs), blocks_for(chunks, per)), dim3(per, 1, imgs), 0, s>>>((const char*)x, (char*)y, N, HW, C);
    return;
  }
  // a row-lane for every pixel as long as the launch has less than 2^18 lanes: each one more is one more term to fold
  const int per = chunks < 256 ? chunks : 256;
  const long long want = (1ll << 18) / ((long long)N * chunks);
  int rows = 256 / per < HW ? 256 / per : HW;
  if (rows > want) rows = want < 1 ? 1 : (int)want;
  const int imgs = 256 / (per * rows);
  gap_fwd_kernel<bf16_t, true><<<dim3(blocks_for(N, imgs), blocks_for(chunks, per)), dim3(per, rows, imgs), 0, s>>>((const char*)x, (char*)y, N, HW, C);
}

void launch_gap_bwd(int dt, const void* dy, const void* x, void* dx, int N, int HW, int C, int relu_mask, hipStream_t s) {
  const long long total = (long long)N * HW * (C / dtype_ce(dt));
  DDS_DISPATCH(dt, gap_bwd_kernel,
               <<<blocks_for(total, 256), 256, 0, s>>>((const char*)dy, (const char*)x, (char*)dx, N, HW, C, relu_mask));
}

void launch_softmax_ce(int dt, const float* logits, const int32_t* labels, void* dlogits, float* loss, int W, int B,
                       int classes, int ldl, int ldg, hipStream_t s) {
  const bool few = classes <= 16 && ldl >= 4 && ldl % 4 == 0 && ldg <= 16;
  if (dt == DT_F32) {
    if (few) softmax_ce_kernel<float, 16><<<W, 256, 0, s>>>(logits, labels, (char*)dlogits, loss, B, classes, ldl, ldg);
    else softmax_ce_kernel<float, 0><<<W, 256, 0, s>>>(logits, labels, (char*)dlogits, loss, B, classes, ldl, ldg);
  } else {
    if (few) softmax_ce_kernel<bf16_t, 16><<<W, 256, 0, s>>>(logits, labels, (char*)dlogits, loss, B, classes, ldl, ldg);
    else softmax_ce_kernel<bf16_t, 0><<<W, 256, 0, s>>>(logits, labels, (char*)dlogits, loss, B, classes, ldl, ldg);
  }
}

void launch_update(int dt, const UpdateDesc* descs, const int* tile_map, int total_tiles, int slot, int W, float lr, float mu, hipStream_t s) {
  if (total_tiles <= 0) return;
  DDS_DISPATCH(dt, update_kernel, <<<total_tiles, 256, 0, s>>>(descs, tile_map, slot, 1.f / (float)W, lr, mu));
}

void launch_recast(int dt, const UpdateDesc* descs, const int* block_map, int total_blocks, hipStream_t s) {
  if (total_blocks <= 0) return;
  DDS_DISPATCH(dt, recast_kernel, <<<total_blocks, 256, 0, s>>>(descs, block_map));
}

void launch_stash(int dt, const UpdateDesc* descs, const int* block_map, int total_blocks, int slot, hipStream_t s) {
  if (total_blocks <= 0) return;
  DDS_DISPATCH(dt, stash_kernel, <<<total_blocks, 256, 0, s>>>(descs, block_map, slot));
}

void launch_gossip_update(int dt, const UpdateDesc* descs, const int* range_map, int total_ranges, const float* P, int W,
                          long long rep_stride, float lr, float mu, hipStream_t s) {
  if (total_ranges <= 0) return;
  DDS_DISPATCH(dt, gossip_update_kernel,
               <<<total_ranges, 256, (size_t)W * 1024, s>>>(descs, range_map, P, W, rep_stride, lr, mu));
}

void launch_consensus(const UpdateDesc* descs, const int* block_map, int total_blocks, int W, long long rep_stride,
                      double* out, hipStream_t s) {
  if (total_blocks <= 0) return;
  consensus_kernel<<<total_blocks, 256, 0, s>>>(descs, block_map, W, rep_stride, out);
}

void launch_param_permute(const float* canon, float* internal, int Cout, int Cin, int RS, int Cinpad, int to_internal,
                          hipStream_t s) {
  const long long total = (long long)Cout * RS * Cinpad + Cout;
  param_permute_kernel<<<blocks_for(total, 256), 256, 0, s>>>(canon, internal, Cout, Cin, RS, Cinpad, to_internal);
}

void launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  fill_zero_kernel<<<(unsigned)blocks, 256, 0, s>>>((uint4*)p, n16);
}

}  // namespace dds
