// Kernels for the narrow layers (16 channels: the first stage of the ResNet-20 / ResNet-56 shapes), bf16.
//
// At 16 channels a 3x3 convolution does 4.6 kFLOP per pixel against 64-96 bytes of traffic: it is bound by
// memory, not by the matrix unit, and a tile sized for wide layers (64 or more output columns, operands staged
// in LDS) spends its time on padding. These kernels use v_mfma_f32_16x16x32_bf16 with the 16 output channels as
// the rows and 16 consecutive pixels as the columns of one accumulator tile, and keep everything else out of
// the way:
//   forward / dgrad (and the forward pass of a stem): all nine taps of the weights (4.6 KB) live in registers as the A operand; the B
//   operand of a tap is 16 bytes per lane (eight channels of one pixel, shifted by the tap) of a patch in LDS;
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

// 1 in each half of a packed bf16 pair >= 0 that is not zero (one instruction: min as unsigned 16-bit numbers)
__device__ __forceinline__ uint32_t nonzero2(uint32_t pair) {
  typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, pair), (u16x2_t){1, 1}));
}

// 3x3, stride 1, pad 1, CIN = 8 or 16 input channels (their stride), at most 16 NB output channels (stride 16 NB).
// A workgroup owns 64 GROUPS consecutive pixels of the flattened (image, row, column) index; in it the nine taps of a pixel
// are the pixels at distance -W-1 .. W+1, so its patch is 64 GROUPS + 2W + 2 consecutive pixels, copied global -> LDS as they lie; of wider
// images it is three runs of 64 GROUPS + 2 pixels, W apart (`pitch` is the distance of two kernel rows in LDS: W or a run's length).
// A wave owns GROUPS runs of 16 pixels. An MFMA multiplies 32 / CIN taps: lane l = 16 g + j holds, as B operand, eight channels of
// pixel j shifted by its tap (16 channels: tap 2 t + (g >> 1), channels 8 (g & 1) .. +8; 8 channels: tap 4 t + g), and as A operand
// the same k-slice of a weight row of each of the NB blocks; rows are dealt to the blocks so that the accumulators give it the 4 NB
// output channels from 4 NB g on of pixel j: 8, 16 or 32 consecutive bytes, and a wave whole lines. Taps outside the image (and past the ninth) read zeros that lie behind the patch: one
// select per tap, of an address that is the same in every run up to the instruction's offset.
// ROWS16: the image width is a multiple of 16, so a run lies inside one image row whose place is a scalar.
// DGRAD: x is the output gradient, w the transposed snapshot [cin][tap][cout], tap (r, s) gathers at
// (h + 1 - r, w + 1 - s); the epilogue options are the ones of ConvParams.
// Bound by memory, then by what every tile costs beside it. 16 -> 16 channels at 32 x 32, 1024 images, alone: operands read straight
// from global memory 24.8 us forward (with a residual 28.5) and 24.3 us backward, of which the five operand reads of a run, at 24
// cycles of the vector cache each, are 13; here 20.1 (23.2) and 20.6 us (69 to 103 MB). Stem to 16 channels (a gather through registers in 256 x 32
// tiles before) 40.4 -> 16.4 us, to 64 channels, 512 images, 49.6 -> 32.1 us. 16 -> 16 channels, rows of 512 / 1024 / 2000 pixels, 2^20 of
// them: one run 36 / 52 / 75 us forward, 33 / 46 / 72 us backward, three runs 29 / 26 / 24 and 25 / 23 / 22 us, operands from global memory
// 29 and 25 us at every width.
template <int CIN, int NB, bool DGRAD, bool ROWS16, int GROUPS>
__global__ __launch_bounds__(256) void conv_direct_kernel(ConvParams p, int fills, int pitch, Divisor dW, Divisor dH) {
  constexpr int PB = CIN * 2, PLOG = CIN == 16 ? 1 : 0, TPM = 32 / CIN, NM = (9 + TPM - 1) / TPM, OB = 32 * NB;  // OB: bytes of an output pixel
  extern __shared__ __align__(16) char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int lane = threadIdx.x & 63;
  const int j = lane & 15, g = lane >> 4;
  const int half = CIN == 16 ? g & 1 : 0, tapl = CIN == 16 ? g >> 1 : g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.x * (64 * GROUPS), row0 = wave * (16 * GROUPS), pix0 = m0 + row0;

  // the patch; pixels before the tensor's first or after its last repeat that pixel (no tap inside an image reads them)
  auto copy = [&](int f, int pix) {
    const int piece = f * 64 + lane;
    pix = min(max(pix + (piece >> PLOG), 0), p.M - 1);
    dma16((const char*)p.x + ((((size_t)(uint32_t)pix << PLOG) + (piece & ((1 << PLOG) - 1))) << 4), lds0 + f * 1024);
  };
  const int jump = p.W - pitch;
  if (jump == 0) {
    for (int f = wave; f < fills; f += 4) copy(f, m0 - p.W - 1);
  } else {
    for (int f = wave; f < fills; f += 4) {
      const int row = (f * 64 + lane) >> PLOG;
      copy(f, m0 - p.W - 1 + (row >= pitch ? jump : 0) + (row >= 2 * pitch ? jump : 0));
    }
  }
  const uint32_t zeros = fills * 1024;
  if (threadIdx.x < GROUPS * PB) *(uint4*)(smem + zeros + threadIdx.x * 16) = make_uint4(0u, 0u, 0u, 0u);

  const char* wbase = (const char*)p.w;
  const float* bias = p.bias;
  if (p.nrep > 1) {  // the pixels of a wave belong to one data-group, those of a workgroup may not
    const int r = min(pix0 / (p.M / p.nrep), p.nrep - 1);
    wbase += (size_t)r * p.w_rep;
    if (bias) bias += (size_t)r * p.bias_rep;
  }
  // weights: MFMA t, block b, lane (j, g): row j of the block, this lane's tap and channels; zero past Nout and past tap 8
  uint4 wa[NB][NM];
  int dr[NM], ds[NM];
  uint32_t toff[NM];    // LDS address at the wave's first run
  uint32_t leaves = 0;  // nibble t: tap t of this lane leaves the image at its top row, bottom row, first or last run
#pragma unroll
  for (int t = 0; t < NM; ++t) {
    const int tap = TPM * t + tapl, tt = tap < 9 ? tap : 0;
    const int r = tt / 3, s = tt - 3 * r;
    dr[t] = DGRAD ? 1 - r : r - 1;
    ds[t] = DGRAD ? 1 - s : s - 1;
    toff[t] = tap < 9 ? (uint32_t)((pitch + 1 + row0 + j + dr[t] * pitch + ds[t]) * PB + half * 16) : zeros;
    leaves |= ((dr[t] < 0 ? 1u : 0u) | (dr[t] > 0 ? 2u : 0u) | (ds[t] < 0 && j == 0 ? 4u : 0u) | (ds[t] > 0 && j == 15 ? 8u : 0u)) << (4 * t);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = 4 * NB * (j >> 2) + 4 * b + (j & 3);
      const bool ok = tap < 9 && n < p.Nout;
      const uint4 v = *(const uint4*)(wbase + ((size_t)((ok ? n : 0) * 9 + tt) * CIN + half * 8) * 2);
      wa[b][t] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  // epilogue operands of this lane's channels; a run past the last pixel reads the last one's
  const uint32_t lane_out = (uint32_t)(j * OB + 8 * NB * g);
  uint2 rs[GROUPS][NB], mk[GROUPS][NB];
  uint32_t keep[GROUPS];
  auto pixel_at = [&](int u) { return (size_t)(ROWS16 ? min(pix0 + 16 * u, p.M - 16) : min(pix0 + 16 * u + j, p.M - 1)); };
  const uint32_t lane_in = ROWS16 ? lane_out : (uint32_t)(8 * NB * g);
  auto load_channels = [&](const void* src, int u, uint2 (&v)[NB]) {
    const char* at = (const char*)src + pixel_at(u) * OB + lane_in;
    if (NB == 1) {
      v[0] = *(const uint2*)at;
    } else {
#pragma unroll
      for (int b = 0; b + 1 < NB; b += 2) {
        const uint4 q = *(const uint4*)(at + 8 * b);
        v[b] = make_uint2(q.x, q.y);
        v[b + 1] = make_uint2(q.z, q.w);
      }
    }
  };
  if (p.res) {
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) load_channels(p.res, u, rs[u]);
  }
  if (p.maskbits) {  // NB == 1 (dgrad)
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) keep[u] = *(const uint16_t*)((const char*)p.maskbits + pixel_at(u) * 2 + (ROWS16 ? 2 * j : 0));
  } else if (p.mask) {
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) load_channels(p.mask, u, mk[u]);
  }
  float ab[NB][4];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) ab[b][e] = 0.f;
  if (bias) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = 4 * NB * g + 4 * b + e;
        const float v = p.alpha * bias[min(n, p.Nout - 1)];
        ab[b][e] = n < p.Nout ? v : 0.f;
      }
  }
  const float lower = p.relu ? 0.f : -__builtin_inff();
  wait_vm<0>();
  __syncthreads();

#pragma unroll
  for (int u = 0; u < GROUPS; ++u) {
    const int run = pix0 + 16 * u;
    if (run >= p.M) break;  // wave-uniform
    const bool in = ROWS16 || run + j < p.M;
    uint4 xb[NM];
    {
      const int pix = ROWS16 ? run : run + j;
      const uint32_t line = __umulhi((uint32_t)pix, dW.mul) >> dW.shift;
      const int h = (int)(line - (__umulhi(line, dH.mul) >> dH.shift) * (uint32_t)p.H), w = pix - (int)line * p.W;
      const uint32_t edges = (h == 0 ? 0x11111u : 0u) | (h == p.H - 1 ? 0x22222u : 0u) | (w == 0 ? 0x44444u : 0u) |
                             (w + 16 == p.W ? 0x88888u : 0u);
      const uint32_t out = leaves & edges;
#pragma unroll
      for (int t = 0; t < NM; ++t) {
        const bool leave = ROWS16 ? (out & (0xfu << (4 * t))) != 0 : (unsigned)(h + dr[t]) >= (unsigned)p.H || (unsigned)(w + ds[t]) >= (unsigned)p.W;
        xb[t] = *(const uint4*)(smem + (leave ? zeros : toff[t]) + 16 * u * PB);
      }
    }
    uint32_t out[2 * NB], signs = 0;  // signs: this lane's 4 NB stored, rounded values that are > 0
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NM; ++t) acc = mfma16(wa[b][t], xb[t], acc);
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaf(p.alpha, acc[e], ab[b][e]);
      if (p.res) {
        v[0] += __uint_as_float(rs[u][b].x << 16); v[1] += __uint_as_float(rs[u][b].x & 0xffff0000u);
        v[2] += __uint_as_float(rs[u][b].y << 16); v[3] += __uint_as_float(rs[u][b].y & 0xffff0000u);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_fmed3f(v[e], lower, __builtin_inff());  // one instruction; NaN -> lower
      if (p.maskbits) {
#pragma unroll
        for (int e = 0; e < 4; ++e)  // bit -> 0 / all ones, then and
          v[e] = __uint_as_float(__float_as_uint(v[e]) & (uint32_t)__builtin_amdgcn_sbfe((int)(keep[u] >> (4 * g)), e, 1));
      } else if (p.mask) {
        if ((int)(mk[u][b].x << 16) < 0x10000) v[0] = 0.f;
        if ((int)mk[u][b].x < 0x10000) v[1] = 0.f;
        if ((int)(mk[u][b].y << 16) < 0x10000) v[2] = 0.f;
        if ((int)mk[u][b].y < 0x10000) v[3] = 0.f;
      }
      out[2 * b] = pack_bf16_rne(v[0], v[1]);
      out[2 * b + 1] = pack_bf16_rne(v[2], v[3]);
      if (p.bits_out) {  // (behind a ReLU: no value is negative)
        const uint32_t t = nonzero2(out[2 * b]) | nonzero2(out[2 * b + 1]) << 2;  // channels 0, 2 in bits 0, 2; 1, 3 in bits 16, 18
        signs |= ((t | t >> 15) & 0xfu) << (4 * b);
      }
    }
    char* y = (char*)p.y + (size_t)run * OB + lane_out;
    if (in) {
      if (NB == 1) *(uint2*)y = make_uint2(out[0], out[1]);
#pragma unroll
      for (int b = 0; b + 1 < NB; b += 2) *(uint4*)(y + 8 * b) = make_uint4(out[2 * b], out[2 * b + 1], out[(2 * b + 2) % (2 * NB)], out[(2 * b + 3) % (2 * NB)]);
    }
    if (p.bits_out) {
      char* bits = (char*)p.bits_out + (size_t)run * (2 * NB);
      if (NB == 1) {  // two lanes hold a byte
        const uint32_t byte = signs | (uint32_t)__shfl_xor((int)signs, 16, 64) << 4;
        if (!(g & 1) && in) *(uint8_t*)(bits + (uint32_t)(2 * j + (g >> 1))) = (uint8_t)byte;
      } else if (NB == 2) {
        if (in) *(uint8_t*)(bits + (uint32_t)(4 * j + g)) = (uint8_t)signs;
      } else {
        if (in) *(uint16_t*)(bits + (uint32_t)(8 * j + 2 * g)) = (uint16_t)signs;
      }
    }
  }
}

// ------------------------------------------------------------------ weight gradient, rows of at most 32 input channels
// dW[k][tap][c] = sum over pixels p of dY[p][k] * X[p + tap][c] for 3x3 stride-1 pad-1 layers of 8, 16 or 32 input
// and at most 32 (8 or 16 input: 64) output channels. All of dW is 32 NM x 32 NT (n = tap * Cx + c; the layout of a partial row),
// which one wave holds in its accumulators: the four waves of a workgroup share the pixels, not the channels, and add their
// sums in LDS when the workgroup has walked its split. A tile is `tile` consecutive pixels of a data-group; their dY rows are
// copied as they lie. X is numbered as in wgrad_flat_body (a row pitch of W + 1, an extra row above every image; zeros at
// the extra positions), so that any image size will do and the nine taps are constant distances from a pixel's position.
// Tiles travel global -> LDS in two slots as plain [pixel or position][channels] rows; ds_read_b64_tr_b16 hands a lane four of
// them of one channel, and because every lane supplies the address of its own row and four channels, the rows may be any
// pixels' positions, and one fragment of 32 columns may hold 1, 2 or 4 taps. Rows and columns past the real ones
// multiply whatever lies there and are never stored. No product pairs a pixel with a tap that does not see it: an
// infinite or NaN activation meets zeros of dY only where that gradient itself is zero.
// Bound by memory (64 to 144 bytes of a pixel against 4.6 to 18 kFLOP) and by one barrier per tile. A launch takes several
// layers: workgroup -> (layer, split). Alone, 1024 images: 16 -> 16 channels at 32 x 32 27.8 -> 19.1 us (512 workgroups, 3.5 TB/s;
// a kernel that staged its tiles through registers before), 32 -> 32 at 16 x 16 27.9 -> 18.3 us and the stem with 16 outputs 95 -> 14.4
// us (64 x 64 blocks of wgrad_dma_body, 3/4 and 31/32 padding before), with 64 outputs and 512 images 50 -> 21.6 us. Tiles of
// 256 (54 KB limit below) against 512: 19.1 / 22.5 us for the 16-channel layers. (dY numbered by positions too, with zeros at the
// extra ones, saves the division of a row address and makes NaN of border taps that an infinite activation does not reach; 16 -> 16 channels
// at 32 x 32 with their stem 34.4 us so and 32.0 here.)
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
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
  Divisor dQ, dH1;       // by Q and by H + 1 (positions)
  Divisor dW, dH;        // by W and by H (pixels): make_divisor1
  int first;             // first workgroup of this layer
  int q, rep_tiles;      // splits and tiles per data-group
  int H, W, Q, imgs_rep; // Q: position pitch of an image row, W + 1
  int tile;              // pixels per tile, a multiple of 256
  int ylog;              // a row of dY is 16 << ylog bytes
  int xfills;            // 1 KiB fills of a tile's X patch at most
  int slots;             // tiles in LDS
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
  constexpr int KS = 512 / MT;              // pixels per MFMA
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
  const bool two = p.slots == 2;
  const int ybytes = T << (ylog + 4);       // dY part of a slot
  const int slot_bytes = ybytes + xfills * 1024;
  const int yfills = ybytes >> 10;
  const Divisor dQ = p.dQ, dH1 = p.dH1, dW = p.dW, dH = p.dH;
  const char* zeros = (const char*)grp.zeros;
  const int pixels = imgs * p.H * W;        // of a data-group
  const size_t pix0 = (size_t)zr * pixels;  // its first
  const char* dy = (const char*)p.dy + (pix0 << (ylog + 4));
  const char* x = (const char*)p.x + (pix0 << (XLOG + 4));

  // position in the data-group -> pixel of the data-group, -1 on the extra rows and columns: with L = u / Q and
  // image i = L / (H + 1), the positions before u hold L extra columns and i + 1 extra rows of W
  auto pixel = [&](int u) {
    const uint32_t uu = (uint32_t)max(u, 0);
    const uint32_t line = __umulhi(uu, dQ.mul) >> dQ.shift, im = __umulhi(line, dH1.mul) >> dH1.shift;
    const int w = (int)(uu - __umul24(line, Q)), h1 = (int)(line - __umul24(im, H1));
    const int pix = (int)(uu - line) - (int)__umul24(im + 1, W);
    return u >= 0 && w < W && h1 > 0 && (int)im < imgs ? pix : -1;
  };
  // pixel of the data-group -> its position, less the Q of the first image's extra row (pixels past the last one count on into
  // further images, whose positions hold zeros)
  auto position = [&](uint32_t n) {
    const uint32_t line = divide(n, dW), im = divide(line, dH);
    return n + line + __umul24(im, Q);
  };
  auto fill_tile = [&](int t, int slot) {
    if (t >= ntiles) return;
    const int n0 = (tile0 + t) * T;
    const uint32_t base = lds0 + slot * slot_bytes;
    for (int f = wave; f < yfills; f += 4) {
      const int piece = f * 64 + lane;
      const int pix = n0 + (piece >> ylog);
      const char* src = dy + ((((size_t)(uint32_t)pix << ylog) + (piece & ((1 << ylog) - 1))) << 4);
      dma16(pix < pixels ? src : zeros, base + f * 1024);
    }
    const int u0 = (int)position(n0);  // position of the patch: u0 + Q less Q + 1
    const int fills = (int)((position(n0 + T - 1) - u0 + 2 * Q + 3) * XB + 1023) >> 10;
    for (int f = wave; f < fills; f += 4) {
      const int piece = f * 64 + lane;
      const int pix = pixel(u0 - 1 + (piece >> XLOG));
      const char* src = x + ((((size_t)(uint32_t)pix << XLOG) + (piece & ((1 << XLOG) - 1))) << 4);
      dma16(pix >= 0 ? src : zeros, base + ybytes + f * 1024);
    }
  };
  fill_tile(0, 0);

  // fragment addressing: a 16-lane group reads four pixels of 16 channels at a time, lane -> (pixel, four channels)
  const int lq = lane & 15, rsub = lq >> 2, seg = lq & 3;
  const int cgrp = NM == 0 ? 0 : (lane >> 4) & 1, kgrp = NM == 0 ? lane >> 4 : lane >> 5;  // 16-channel half, eight pixels of a step
  const int row0 = wave * (T >> 2) + 8 * kgrp + rsub;  // the waves take a quarter of a tile each
  const uint32_t a_lane = ((uint32_t)row0 << (ylog + 4)) + cgrp * 32 + seg * 8;
  uint32_t b_lane[NT];
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int n = MT * b + 16 * cgrp + 4 * seg;
    const int tap = min(n / Cx, 8), c = n % Cx;
    b_lane[b] = ((tap / 3) * Q + tap % 3) * XB + c * 2 + ybytes;
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
    if (two) fill_tile(t + 1, (t + 1) & 1);
    const uint32_t base = lds0 + (two ? t & 1 : 0) * slot_bytes;
    const uint32_t n0 = (tile0 + t) * T, x0 = base - position(n0) * XB;  // x0 + position * XB: LDS row of the top left tap
    uint32_t ya = base + a_lane;
    for (int i = 0; i < T >> 8; ++i) {  // 64 pixels of this wave
#pragma unroll
      for (int ks = 0; ks < 64 / KS; ++ks) {
        uint4 a[MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const uint2 a0 = lds_tr16_b64(ya + m * 64), a1 = lds_tr16_b64(ya + y4 + m * 64);
          a[m] = make_uint4(a0.x, a0.y, a1.x, a1.y);
        }
        ya += yks;
        const uint32_t n = n0 + row0 + 64 * i + KS * ks;
        const uint32_t xa = x0 + position(n) * XB, xc = x0 + position(n + 4) * XB;
#pragma unroll
        for (int b = 0; b < NT; ++b) {
          const uint2 b0 = lds_tr16_b64(xa + b_lane[b]), b1 = lds_tr16_b64(xc + b_lane[b]);
          const uint4 bf = make_uint4(b0.x, b0.y, b1.x, b1.y);
#pragma unroll
          for (int m = 0; m < MB; ++m) acc[m][b] = slim_mfma(a[m], bf, acc[m][b]);
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) accb[m] = slim_mfma(a[m], ones, accb[m]);  // bias gradient: column sums of dY
      }
    }
    if (!two) {
      wg_barrier();
      fill_tile(t + 1, 0);
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
  const long long positions = (long long)l.imgs_rep * (p.H + 1) * l.Q, pixels = (long long)l.imgs_rep * p.H * p.W;
  // positions are 32-bit numbers (a tile's last pixels may lie in images past the last), rows of positions and sides 24-bit ones
  if (positions + 4096 + 4ll * l.Q >= (1ll << 31) || (long long)l.imgs_rep * (p.H + 1) + 2048 >= (1 << 24) || p.H >= (1 << 23) || p.W >= (1 << 23)) return false;
  const int xb = p.Cx * 2;
  // what a tile's pixels cross of boundaries `every` pixels apart; tiles begin at multiples of their size
  auto crossed = [](long long tile, long long every) {
    return every % tile == 0 ? 0 : tile % every == 0 ? tile / every - 1 : (tile - 2) / every + 1;
  };
  l.slots = 2;
  for (l.tile = 512;; l.tile = 256) {  // three workgroups of two slots each share a CU
    const long long rows = crossed(l.tile, p.W), images = crossed(l.tile, (long long)p.H * p.W);
    l.xfills = (int)(((l.tile + rows + (images + 2) * l.Q + 2) * xb + 1023) / 1024);
    const long long slot = (l.tile << (l.ylog + 4)) + 1024ll * l.xfills;
    if (2 * slot <= 54000) break;
    if (l.tile == 256) {
      // One tile at a time, copy and products in turn: rows of more than 1021 (16 channels in and out) or 380 (32) pixels, 680 or 253 where tiles run from one
      // image into the next. 378 pixels of 32 channels 97 us with the stem, with two slots 86, wgrad_gemm_kernel 490.
      if (2 * slot > 160 * 1024) l.slots = 1;
      if (slot > 160 * 1024) return false;
      break;
    }
  }
  l.rep_tiles = (int)((pixels + l.tile - 1) / l.tile);
  l.dQ = make_divisor(l.Q);
  l.dH1 = make_divisor(p.H + 1);
  l.dW = make_divisor1(p.W);
  l.dH = make_divisor1(p.H);
  l.Mout = p.Mout;
  l.alpha = p.alpha;
  return true;
}

// wgrad_slim_kernel's NM
inline int slim_blocks(const WgradParams& p) { return p.ldy <= 16 && p.Cx <= 16 ? 0 : p.ldy <= 32 ? 1 : 2; }

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

template <int XB, int NM>
void launch_slim_inst(const SlimGroup& g, int wgs, int smem, hipStream_t s) {
  static DeviceOnce lds;
  allow_whole_lds(lds, (const void*)wgrad_slim_kernel<XB, NM>);
  wgrad_slim_kernel<XB, NM><<<wgs, 256, smem, s>>>(g);
}

}  // namespace

template <int CIN, int NB, bool DGRAD, bool ROWS16>
void launch_direct_inst(const ConvParams& p, hipStream_t s) {
  constexpr int GROUPS = NB == 4 ? 2 : 4, PB = CIN * 2;
  const int pitch = min(p.W, 64 * GROUPS + 2), fills = cdiv((64 * GROUPS + 2 + 2 * pitch) * PB, 1024);
  conv_direct_kernel<CIN, NB, DGRAD, ROWS16, GROUPS><<<cdiv(p.M, 64 * GROUPS), 256, fills * 1024 + GROUPS * PB * 16, s>>>(p, fills, pitch, make_divisor(p.W), make_divisor(p.H));
}
template <int CIN, int NB, bool DGRAD>
void launch_direct(const ConvParams& p, hipStream_t s) {
  if (p.W % 16 == 0) launch_direct_inst<CIN, NB, DGRAD, true>(p, s);
  else launch_direct_inst<CIN, NB, DGRAD, false>(p, s);
}

// True if the launch was taken: bf16, 3x3 stride 1 pad 1, from rows of 16 channels to rows of 16 in either direction and,
// forward, from rows of 8 (the stem) to rows of 16, 32 or 64.
bool launch_conv_narrow(const ConvParams& p, hipStream_t s) {
  if (p.R != 3 || p.S != 3 || p.stride != 1 || p.pad != 1 || p.H != p.Ho || p.W != p.Wo) return false;
  if (p.out_f32 || p.x2 != nullptr || p.Nout > p.ldy || p.M != p.Nimg * p.H * p.W) return false;
  if (p.H < 2 || p.W < 2) return false;  // make_divisor
  // a wave's runs must not straddle two data-groups
  if (p.nrep > 1 && (p.Nimg % p.nrep != 0 || (p.Nimg / p.nrep * (long long)p.H * p.W) % 64 != 0)) return false;
  if (p.Cx == 16 && p.ldy == 16) {
    if (p.dgrad) launch_direct<16, 1, true>(p, s);
    else launch_direct<16, 1, false>(p, s);
    return true;
  }
  if (p.Cx != 8 || p.dgrad) return false;
  if (p.ldy == 16) launch_direct<8, 1, false>(p, s);
  else if (p.ldy == 32) launch_direct<8, 2, false>(p, s);
  else if (p.ldy == 64) launch_direct<8, 4, false>(p, s);
  else return false;
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
    const int need = l.slots * ((l.tile << (l.ylog + 4)) + 1024 * l.xfills);
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
