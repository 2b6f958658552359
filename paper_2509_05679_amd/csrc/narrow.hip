// Kernels for the narrow layers (16 channels: the first stage of the ResNet-20 / ResNet-56 shapes), bf16.
//
// At 16 channels a 3x3 convolution does 4.6 kFLOP per pixel against 64-96 bytes of traffic: it is bound by
// memory, not by the matrix unit, and a tile sized for wide layers (64 or more output columns, operands staged
// in LDS) spends its time on padding. These kernels use v_mfma_f32_16x16x32_bf16 with the 16 output channels as
// the rows and 16 consecutive pixels as the columns of one accumulator tile, and keep everything else out of
// the way:
//   forward / dgrad: all nine taps of the weights (4.6 KB) live in registers as the A operand; the B operand of
//   a tap is read straight from global memory, 16 bytes per lane (eight channels of one pixel, shifted by the
//   tap) -- neighbouring taps re-read the same cache lines from the vector cache, so no LDS and no barrier;
//   weight gradient (also of the 8- and 32-channel layers): see wgrad_slim_kernel below.
#include "device_once.h"
#include "kernels.h"
#include "lds_copy.h"

namespace dds {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ f32x4_t mfma16(const uint4& a, const uint4& b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// 3x3, stride 1, pad 1, 16 input channels (channel stride 16), at most 16 output channels (stride 16).
// One wave owns GROUPS runs of 16 consecutive pixels of the flattened (image, row, column) index; the image width
// is a multiple of 16, so a run lies inside one image row. Lane l = 16 g + j holds, as B operand of MFMA t,
// channels 8 (g & 1) .. +8 of pixel j shifted by tap 2 t + (g >> 1), and as A operand the same k-slice of weight
// row j; the accumulator gives it output channels 4 g .. 4 g + 3 of pixel j: one 8-byte store, and the four lane
// groups together write the 512 contiguous bytes of the run.
// DGRAD: x is the output gradient, w the transposed snapshot [cin][tap][cout], tap (r, s) gathers at
// (h + 1 - r, w + 1 - s); the epilogue options are the ones of ConvParams.
template <bool DGRAD, int GROUPS>
__global__ __launch_bounds__(256) void conv16_direct_kernel(ConvParams p) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * 256 + threadIdx.x) >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int half = g & 1;
  const int ngroups = p.M >> 4;
  const int grp0 = wave * GROUPS;
  if (grp0 >= ngroups) return;
  const int HW = p.H * p.W;

  const char* wbase = (const char*)p.w;
  const float* bias = p.bias;
  if (p.nrep > 1) {  // a run never leaves its image, a workgroup may: weights are picked per wave
    const int img = (grp0 << 4) / HW;
    const int r = min(img / (p.Nimg / p.nrep), p.nrep - 1);
    wbase += (size_t)r * p.w_rep;
    if (bias) bias += (size_t)r * p.bias_rep;
  }
  // weights: MFMA t, lane (j, g): row j, tap 2 t + (g >> 1), channels 8 half .. +8; zero past Nout and past tap 8
  uint4 wa[5];
  int dr[5], ds[5];
  bool tap_ok[5];
#pragma unroll
  for (int t = 0; t < 5; ++t) {
    const int tap = 2 * t + (g >> 1);
    tap_ok[t] = tap < 9;
    const int tt = tap_ok[t] ? tap : 0;
    const int r = tt / 3, s = tt - 3 * r;
    dr[t] = DGRAD ? 1 - r : r - 1;
    ds[t] = DGRAD ? 1 - s : s - 1;
    const bool ok = tap_ok[t] && j < p.Nout;
    const uint4 v = *(const uint4*)(wbase + ((size_t)((ok ? j : 0) * 9 + tt) * 16 + half * 8) * 2);
    wa[t] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
  }
  float ab[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int n = 4 * g + e;
    ab[e] = (bias != nullptr && n < p.Nout) ? p.alpha * bias[n] : 0.f;
  }
  const float lower = p.relu ? 0.f : -__builtin_inff();

#pragma unroll
  for (int u = 0; u < GROUPS; ++u) {
    const int grp = grp0 + u;
    if (grp >= ngroups) break;  // wave-uniform
    const int pix = (grp << 4) + j;
    const int img = pix / HW, rem = pix - img * HW;
    const int h = rem / p.W, w = rem - h * p.W;
    const char* ximg = (const char*)p.x + (size_t)img * HW * 32 + half * 16;
    uint4 xb[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      const int hh = h + dr[t], ww = w + ds[t];
      const bool ok = tap_ok[t] && (unsigned)hh < (unsigned)p.H && (unsigned)ww < (unsigned)p.W;
      const uint4 v = *(const uint4*)(ximg + (size_t)(ok ? hh * p.W + ww : rem) * 32);  // unconditional, clamped
      xb[t] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
    }
    // epilogue operands of this lane's four channels (8 bytes each), also unconditional
    const size_t o = (size_t)pix * 16 + 4 * g;
    uint2 rs = make_uint2(0u, 0u), mk = make_uint2(0u, 0u);
    uint32_t keep = 0xfu;
    if (p.res) rs = *(const uint2*)((const uint16_t*)p.res + o);
    if (p.maskbits) keep = ((uint32_t)((const uint16_t*)p.maskbits)[pix] >> (4 * g)) & 0xfu;
    else if (p.mask) {
      mk = *(const uint2*)((const uint16_t*)p.mask + o);
      keep = ((int)(mk.x << 16) >= 0x10000 ? 1u : 0u) | ((int)mk.x >= 0x10000 ? 2u : 0u) |
             ((int)(mk.y << 16) >= 0x10000 ? 4u : 0u) | ((int)mk.y >= 0x10000 ? 8u : 0u);
    }
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 5; ++t) acc = mfma16(wa[t], xb[t], acc);
    const float r4[4] = {__uint_as_float(rs.x << 16), __uint_as_float(rs.x & 0xffff0000u),
                         __uint_as_float(rs.y << 16), __uint_as_float(rs.y & 0xffff0000u)};
    float v[4];
    uint32_t signs = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float t = fmaf(p.alpha, acc[e], ab[e]) + r4[e];
      t = __builtin_amdgcn_fmed3f(t, lower, __builtin_inff());
      v[e] = ((keep >> e) & 1u) ? t : 0.f;
    }
    uint2 out;
    out.x = pack_bf16_rne(v[0], v[1]);
    out.y = pack_bf16_rne(v[2], v[3]);
    *(uint2*)((uint16_t*)p.y + o) = out;
    if (p.bits_out) {
      // the sign of the stored (rounded) value, as every other producer defines the plane
      signs = ((int)(out.x << 16) >= 0x10000 ? 1u : 0u) | ((int)out.x >= 0x10000 ? 2u : 0u) |
              ((int)(out.y << 16) >= 0x10000 ? 4u : 0u) | ((int)out.y >= 0x10000 ? 8u : 0u);
      uint32_t word = signs << (4 * g);
      word |= (uint32_t)__shfl_xor((int)word, 16, 64);
      word |= (uint32_t)__shfl_xor((int)word, 32, 64);
      if (g == 0) ((uint16_t*)p.bits_out)[pix] = (uint16_t)word;
    }
  }
}


// ------------------------------------------------------------------ weight gradient, rows of at most 32 input channels
// dW[k][tap][c] = sum over pixels p of dY[p][k] * X[p + tap][c] for 3x3 stride-1 pad-1 layers of 8, 16 or 32 input
// and at most 32 (8 or 16 input: 64) output channels. All of dW is 32 NM x 32 NT (n = tap * Cx + c; the layout of a partial row),
// which one wave holds in its accumulators: the four waves of a workgroup share the pixels, not the channels, and add their
// sums in LDS when the workgroup has walked its split. Pixels of a data-group are numbered as in wgrad_flat_body (a
// row pitch of W + 1, an extra row above every image; zeros at the extra positions), so that any image size will do, a tile is
// `tile` consecutive positions and the nine taps are constant distances. Tiles travel global -> LDS in two slots as plain
// [position][channels] rows; ds_read_b64_tr_b16 hands a lane four positions of one channel, and because every lane supplies the
// address of its own four channels, one fragment of 32 columns may hold 1, 2 or 4 taps. Rows and columns past the real ones
// multiply whatever lies there and are never stored. (An infinite activation makes NaN of taps that meet it from an extra
// position; the centre tap of the same filter is then infinite or NaN whatever the kernel.)
// Bound by memory (64 to 144 bytes of a pixel against 4.6 to 18 kFLOP) and by one barrier per tile. A launch takes several
// layers: workgroup -> (layer, split). Alone, 1024 images: 16 -> 16 channels at 32 x 32 27.8 -> 19.1 us (512 workgroups, 3.5 TB/s;
// a kernel that staged its tiles through registers before), 32 -> 32 at 16 x 16 27.9 -> 18.3 us and the stem with 16 outputs 95 -> 14.4
// us (64 x 64 blocks of wgrad_dma_body, 3/4 and 31/32 padding before), with 64 outputs and 512 images 50 -> 21.6 us. Tiles of
// 256 positions (54 KB limit below) against 512: 19.1 / 22.5 us for the 16-channel layers.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
#define DDS_LDS_AS __attribute__((address_space(3)))
__device__ __forceinline__ uint2 lds_tr16_b64(uint32_t lds_byte_address) {
  s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t DDS_LDS_AS*)(size_t)lds_byte_address);
  return __builtin_bit_cast(uint2, v);
}
template <int MT> struct SlimAcc { typedef f32x16_t type; };
template <> struct SlimAcc<16> { typedef f32x4_t type; };
__device__ __forceinline__ f32x4_t slim_mfma(const uint4& a, const uint4& b, f32x4_t c) { return mfma16(a, b, c); }
__device__ __forceinline__ f32x16_t slim_mfma(const uint4& a, const uint4& b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

struct SlimLayer {
  const void* dy;
  const void* x;
  float* partial;
  long long Pl;
  Divisor dQ, dH;        // by Q and by H + 1
  int first;             // first workgroup of this layer
  int q, rep_tiles;      // splits and tiles per data-group
  int H, W, Q, imgs_rep; // Q: position pitch of an image row, W + 1
  int tile;              // positions per tile, a multiple of 256
  int ylog;              // a row of dY is 16 << ylog bytes
  int xfills;            // 1 KiB fills of a tile's X patch
  int Mout;
  float alpha;
};
struct SlimGroup {
  const void* zeros;
  int n;
  SlimLayer layer[kWgradGroupMax];
};

// XB: bytes of an X row (16, 32, 64), NM: 32-row blocks of output channels; 0: one block of 16 rows, in 16 x 16 tiles of dW
// (a 32 x 32 tile would multiply half padding)
template <int XB, int NM>
__global__ __launch_bounds__(256, 2) void wgrad_slim_kernel(SlimGroup grp) {
  constexpr int MT = NM == 0 ? 16 : 32;     // rows and columns of a tile of dW
  constexpr int KS = 512 / MT;              // positions per MFMA
  constexpr int NA = MT * MT / 64;          // accumulators of a lane and tile
  constexpr int MB = NM == 0 ? 1 : NM;
  constexpr int Cx = XB / 2, NK = 9 * Cx, NT = (NK + MT - 1) / MT;
  constexpr int XLOG = XB == 16 ? 0 : XB == 32 ? 1 : 2;
  typedef typename SlimAcc<MT>::type acc_t;
  extern __shared__ __align__(16) char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int li = 0;
  while (li + 1 < grp.n && (int)blockIdx.x >= grp.layer[li + 1].first) ++li;
  const SlimLayer& p = grp.layer[li];
  const int z = blockIdx.x - p.first;
  // split z = (data-group, j): the data-group's tiles are dealt to its q splits as evenly as whole tiles allow
  const int zr = z / p.q, zj = z - zr * p.q;
  const int tile0 = (int)(((long long)zj * p.rep_tiles) / p.q);
  const int ntiles = (int)(((long long)(zj + 1) * p.rep_tiles) / p.q) - tile0;
  const int ylog = p.ylog, T = p.tile, Q = p.Q, H1 = p.H + 1, W = p.W, imgs = p.imgs_rep, xfills = p.xfills;
  const int ybytes = T << (ylog + 4);       // dY part of a slot
  const int slot_bytes = ybytes + xfills * 1024;
  const int yfills = ybytes >> 10;
  const Divisor dQ = p.dQ, dH = p.dH;
  const char* zeros = (const char*)grp.zeros;
  const size_t pix0 = (size_t)zr * imgs * p.H * W;  // first pixel of the data-group
  const char* dy = (const char*)p.dy + (pix0 << (ylog + 4));
  const char* x = (const char*)p.x + (pix0 << (XLOG + 4));

  // position in the data-group -> pixel of the data-group, -1 on the extra rows and columns: with L = u / Q and
  // image i = L / (H + 1), the positions before u hold L extra columns and i + 1 extra rows of W
  auto pixel = [&](int u) {
    const uint32_t uu = (uint32_t)max(u, 0);
    const uint32_t line = __umulhi(uu, dQ.mul) >> dQ.shift, im = __umulhi(line, dH.mul) >> dH.shift;
    const int w = (int)(uu - __umul24(line, Q)), h1 = (int)(line - __umul24(im, H1));
    const int pix = (int)(uu - line) - (int)__umul24(im + 1, W);
    return u >= 0 && w < W && h1 > 0 && (int)im < imgs ? pix : -1;
  };
  auto fill_tile = [&](int t, int slot) {
    if (t >= ntiles) return;
    const int u0 = (tile0 + t) * T;
    const uint32_t base = lds0 + slot * slot_bytes;
    for (int f = wave; f < yfills; f += 4) {
      const int piece = f * 64 + lane;
      const int pix = pixel(u0 + (piece >> ylog));
      const char* src = dy + ((((size_t)(uint32_t)pix << ylog) + (piece & ((1 << ylog) - 1))) << 4);
      dma16(pix >= 0 ? src : zeros, base + f * 1024);
    }
    for (int f = wave; f < xfills; f += 4) {
      const int piece = f * 64 + lane;
      const int pix = pixel(u0 - Q - 1 + (piece >> XLOG));
      const char* src = x + ((((size_t)(uint32_t)pix << XLOG) + (piece & ((1 << XLOG) - 1))) << 4);
      dma16(pix >= 0 ? src : zeros, base + ybytes + f * 1024);
    }
  };
  fill_tile(0, 0);

  // fragment addressing: a 16-lane group reads four positions of 16 channels at a time, lane -> (position, four channels)
  const int lq = lane & 15, rsub = lq >> 2, seg = lq & 3;
  const int cgrp = NM == 0 ? 0 : (lane >> 4) & 1, kgrp = NM == 0 ? lane >> 4 : lane >> 5;  // 16-channel half, eight positions of a step
  const int row0 = wave * (T >> 2) + 8 * kgrp + rsub;  // the waves take a quarter of a tile each
  const uint32_t a_lane = ((uint32_t)row0 << (ylog + 4)) + cgrp * 32 + seg * 8;
  uint32_t b_lane[NT];
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int n = MT * b + 16 * cgrp + 4 * seg;
    const int tap = min(n / Cx, 8), c = n % Cx;
    b_lane[b] = (row0 + (tap / 3) * Q + tap % 3) * XB + c * 2 + ybytes;
  }
  acc_t acc[MB][NT], accb[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int e = 0; e < NA; ++e) {
      accb[m][e] = 0.f;
#pragma unroll
      for (int b = 0; b < NT; ++b) acc[m][b][e] = 0.f;
    }
  const uint4 ones = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
  const uint32_t y4 = 4u << (ylog + 4), yks = (uint32_t)KS << (ylog + 4);

  for (int t = 0; t < ntiles; ++t) {
    wait_vm<0>();
    wg_barrier();
    fill_tile(t + 1, (t + 1) & 1);
    const uint32_t base = lds0 + (t & 1) * slot_bytes;
    uint32_t ya = base + a_lane, xb[NT];
#pragma unroll
    for (int b = 0; b < NT; ++b) xb[b] = base + b_lane[b];
    for (int i = 0; i < T >> 8; ++i) {  // 64 positions of this wave
#pragma unroll
      for (int ks = 0; ks < 64 / KS; ++ks) {
        uint4 a[MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const uint2 a0 = lds_tr16_b64(ya + m * 64), a1 = lds_tr16_b64(ya + y4 + m * 64);
          a[m] = make_uint4(a0.x, a0.y, a1.x, a1.y);
        }
        ya += yks;
#pragma unroll
        for (int b = 0; b < NT; ++b) {
          const uint2 b0 = lds_tr16_b64(xb[b] + ks * KS * XB), b1 = lds_tr16_b64(xb[b] + (ks * KS + 4) * XB);
          const uint4 bf = make_uint4(b0.x, b0.y, b1.x, b1.y);
#pragma unroll
          for (int m = 0; m < MB; ++m) acc[m][b] = slim_mfma(a[m], bf, acc[m][b]);
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) accb[m] = slim_mfma(a[m], ones, accb[m]);  // bias gradient: column sums of dY
      }
#pragma unroll
      for (int b = 0; b < NT; ++b) xb[b] += 64 * XB;
    }
  }
  wait_vm<0>();

  // The four waves' sums meet in LDS, 48 KiB at a time, and leave as whole rows of a tile.
  float* out = p.partial + (size_t)z * p.Pl;
  float* red = (float*)smem;
  constexpr int NBLK = MB * NT, BATCH = 3072 / (MT * MT), TSZ = MT * MT;
  const int rgrp = NM == 0 ? lane >> 4 : lane >> 5;
#pragma unroll
  for (int b0 = 0; b0 < NBLK; b0 += BATCH) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      if (b0 + i >= NBLK) continue;
#pragma unroll
      for (int e = 0; e < NA; ++e)
        red[(wave * BATCH + i) * TSZ + (8 * (e >> 2) + 4 * rgrp + (e & 3)) * MT + (lane & (MT - 1))] = acc[(b0 + i) / NT][(b0 + i) % NT][e];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < BATCH * TSZ / 1024; ++j) {
      const int o = j * 1024 + tid * 4, blk = b0 + o / TSZ, r = o % TSZ;
      const int m = blk / NT * MT + r / MT, n = blk % NT * MT + r % MT;
      const float4 s0 = *(const float4*)(red + o), s1 = *(const float4*)(red + 3072 + o);
      const float4 s2 = *(const float4*)(red + 6144 + o), s3 = *(const float4*)(red + 9216 + o);
      if (blk < NBLK && m < p.Mout && n < NK)
        *(float4*)(out + (size_t)m * NK + n) = make_float4(p.alpha * ((s0.x + s1.x) + (s2.x + s3.x)), p.alpha * ((s0.y + s1.y) + (s2.y + s3.y)),
                                                           p.alpha * ((s0.z + s1.z) + (s2.z + s3.z)), p.alpha * ((s0.w + s1.w) + (s2.w + s3.w)));
    }
  }
  __syncthreads();
  if ((lane & (MT - 1)) == 0) {
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int e = 0; e < NA; ++e) red[wave * 64 + m * MT + 8 * (e >> 2) + 4 * rgrp + (e & 3)] = accb[m][e];
  }
  __syncthreads();
  if (tid < MT * MB && tid < p.Mout) out[(size_t)p.Mout * NK + tid] = p.alpha * ((red[tid] + red[64 + tid]) + (red[128 + tid] + red[192 + tid]));
}

// The layer's part of a launch but for its pointers and its place in it; false: not a layer of this kernel.
bool slim_layer(const WgradParams& p, int W, SlimLayer& l) {
  if (p.R != 3 || p.S != 3 || p.stride != 1 || p.pad != 1 || p.H != p.Ho || p.W != p.Wo || W < 1 || p.Nimg % W != 0) return false;
  if (p.Cx != 8 && p.Cx != 16 && p.Cx != 32) return false;
  if (p.Mout > p.ldy || p.zeros == nullptr || p.NK != 9 * p.Cx) return false;
  l.ylog = p.ldy == 8 ? 0 : p.ldy == 16 ? 1 : p.ldy == 32 ? 2 : p.ldy == 64 && p.Cx < 32 ? 3 : -1;
  if (l.ylog < 0) return false;
  l.H = p.H; l.W = p.W; l.Q = p.W + 1;
  l.imgs_rep = p.Nimg / W;
  const long long positions = (long long)l.imgs_rep * (p.H + 1) * l.Q;
  // positions are 32-bit numbers, rows of positions and sides 24-bit ones
  if (positions + 1024 + 4 * l.Q >= (1ll << 31) || (long long)l.imgs_rep * (p.H + 1) + 2048 >= (1 << 24) || p.H >= (1 << 23) || p.W >= (1 << 23)) return false;
  const int xb = p.Cx * 2;
  for (l.tile = 512;; l.tile = 256) {  // three workgroups of two slots each share a CU
    l.xfills = (int)(((long long)(l.tile + 2 * l.Q + 2) * xb + 1023) / 1024);
    const long long smem = 2ll * ((l.tile << (l.ylog + 4)) + 1024ll * l.xfills);
    if (smem <= 54000) break;
    if (l.tile == 256) {
      if (smem > 160 * 1024) return false;  // rows of at most about 1900 (8 channels) to 380 (32) pixels
      break;
    }
  }
  l.rep_tiles = (int)((positions + l.tile - 1) / l.tile);
  l.dQ = make_divisor(l.Q);
  l.dH = make_divisor(p.H + 1);
  l.Mout = p.Mout;
  l.alpha = p.alpha;
  return true;
}

// wgrad_slim_kernel's NM
inline int slim_blocks(const WgradParams& p) { return p.ldy <= 16 && p.Cx <= 16 ? 0 : p.ldy <= 32 ? 1 : 2; }

template <int XB, int NM>
void launch_slim_inst(const SlimGroup& g, int wgs, int smem, hipStream_t s) {
  static DeviceOnce lds;
  allow_whole_lds(lds, (const void*)wgrad_slim_kernel<XB, NM>);
  wgrad_slim_kernel<XB, NM><<<wgs, 256, smem, s>>>(g);
}

}  // namespace

// True if the launch was taken: bf16, 3x3 stride 1 pad 1, 16-channel input and output rows, image width a multiple of 16.
bool launch_conv_narrow(const ConvParams& p, hipStream_t s) {
  if (p.R != 3 || p.S != 3 || p.stride != 1 || p.pad != 1 || p.H != p.Ho || p.W != p.Wo) return false;
  if (p.Cx != 16 || p.ldy != 16 || p.Nout > 16 || p.out_f32 || p.x2 != nullptr) return false;
  if (p.W % 16 != 0 || p.M % 16 != 0 || p.M != p.Nimg * p.H * p.W) return false;
  // a wave's runs (64 pixels) must not straddle two data-groups
  if (p.nrep > 1 && (p.Nimg % p.nrep != 0 || (p.H * p.W) % 64 != 0)) return false;
  constexpr int GROUPS = 4;
  const int ngroups = p.M / 16;
  const int waves = (ngroups + GROUPS - 1) / GROUPS;
  const int blocks = (waves + 3) / 4;
  if (p.dgrad) conv16_direct_kernel<true, GROUPS><<<blocks, 256, 0, s>>>(p);
  else conv16_direct_kernel<false, GROUPS><<<blocks, 256, 0, s>>>(p);
  return true;
}

int wgrad_slim_tiles(const WgradParams& shape, int nrep, int* variant) {
  SlimLayer l{};
  if (!slim_layer(shape, nrep, l)) return 0;
  *variant = shape.Cx + slim_blocks(shape);
  return l.rep_tiles;
}

bool launch_wgrad_slim(const WgradParams* p, int n, hipStream_t s) {
  if (n < 1 || n > kWgradGroupMax) return false;
  SlimGroup g{};
  g.zeros = p[0].zeros;
  int wgs = 0, smem = 3 * 16384;  // the closing reduction
  for (int i = 0; i < n; ++i) {
    SlimLayer& l = g.layer[i];
    if (p[i].nrep < 1 || p[i].nsplit % p[i].nrep != 0 || !slim_layer(p[i], p[i].nrep, l)) return false;
    if (p[i].Cx != p[0].Cx || slim_blocks(p[i]) != slim_blocks(p[0])) return false;
    l.q = p[i].nsplit / p[i].nrep;
    if (l.q < 1 || l.q > l.rep_tiles) return false;  // no empty split
    l.dy = p[i].dy; l.x = p[i].x; l.partial = p[i].partial; l.Pl = p[i].Pl;
    l.first = wgs;
    wgs += p[i].nsplit;
    const int need = 2 * ((l.tile << (l.ylog + 4)) + 1024 * l.xfills);
    smem = smem > need ? smem : need;
  }
  g.n = n;
#define DDS_SLIM_CASE(CX, NM) \
  case CX * 4 + NM: launch_slim_inst<CX * 2, NM>(g, wgs, smem, s); break;
  switch (p[0].Cx * 4 + slim_blocks(p[0])) {
    DDS_SLIM_CASE(8, 0) DDS_SLIM_CASE(8, 1) DDS_SLIM_CASE(8, 2)
    DDS_SLIM_CASE(16, 0) DDS_SLIM_CASE(16, 1) DDS_SLIM_CASE(16, 2)
    DDS_SLIM_CASE(32, 1)
    default: return false;
  }
#undef DDS_SLIM_CASE
  return true;
}

}  // namespace dds
