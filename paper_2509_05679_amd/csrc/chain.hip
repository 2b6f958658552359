// Runs of consecutive 3x3 stride-1 layers of equal width (16 to 128 channels), bf16, in one launch: forward or input gradient.
//
// An image of these layers fits in LDS (32 KB at 32 x 32 x 16, 16 x 16 x 32 takes 16 KB, 8 x 8 x 64 takes 8 KB), and nothing but the
// weights ties one image to another: a workgroup reads whole images once, takes them through every layer of the run and only
// writes each layer's output (what the other pass and the weight gradients read). A launch per layer costs 5 to 8 us whatever
// its work, reads every tensor again and leaves its first copies and its last stores without anything beside them.
#include "device_once.h"
#include "kernels.h"
#include "lds_copy.h"
#include "norm_fold.h"

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

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 lds_read16(uint32_t at) {
  const u32x4_t v = *(const u32x4_t DDS_LDS_AS*)(size_t)at;
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 lds_read8(uint32_t at) {
  const u32x2_t v = *(const u32x2_t DDS_LDS_AS*)(size_t)at;
  return make_uint2(v.x, v.y);
}
__device__ __forceinline__ void lds_write16(uint32_t at, uint32_t a, uint32_t b, uint32_t c, uint32_t d) { *(u32x4_t DDS_LDS_AS*)(size_t)at = (u32x4_t){a, b, c, d}; }
__device__ __forceinline__ void lds_write8(uint32_t at, uint32_t a, uint32_t b) { *(u32x2_t DDS_LDS_AS*)(size_t)at = (u32x2_t){a, b}; }

// 1 in each half of a packed bf16 pair >= 0 that is not zero: min(., 1) (which the compiler would turn into comparisons and selects)
__device__ __forceinline__ uint32_t nonzero2(uint32_t pair) {
  uint32_t r;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(pair), "s"(0x00010001u));
  return r;
}
// halves of a packed pair times 0 or 1 each
__device__ __forceinline__ uint32_t keep2(uint32_t pair, uint32_t ones) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2_t, pair) * __builtin_bit_cast(u16x2_t, ones));
}

constexpr int kWaves = 8;
constexpr int sign_slots(int C) { return C == 16 ? 3 : 2; }

struct ChainGeom {
  int imgs;            // images of a workgroup
  uint32_t plane;      // bytes of LDS of 16 channels of one layer's images, by positions
  uint32_t buf_bytes;  // of all channels, whole 1 KiB fills
  uint32_t sign_bytes; // input gradient: of the images' signs, whole fills
  uint32_t fold_at;    // NORM: where the normalisation's factors are made, behind everything else
  Divisor dP;          // by the plane's 16-byte pieces
  Divisor dQ, dH1;     // by W + 1 and H + 1 (positions)
  Divisor dW, dH;      // by W and H (pixels)
};

// How a workgroup of eight waves is laid out. A wave owns runs of 16 pixels (columns of v_mfma_f32_16x16x32_bf16) and NBW of the C / 16
// blocks of output channels (its rows); a step multiplies 32 input channels, two taps' worth of them at 16 channels.
template <int C>
struct Shape {
  static constexpr int PB = 2 * C, CPP = PB / 16, NBLK = C / 16;  // CPP: 16-byte pieces of a pixel
  static constexpr int WN = C == 64 ? 2 : 1, WM = kWaves / WN;    // waves over the output channels and over the pixels
  static constexpr int NBW = NBLK / WN;
  static constexpr int SPP = C / 32 * 3;                          // C > 16: steps of a tap row, whose weights are refilled together
};

// Images lie in LDS by positions: a row pitch of Q = W + 1 whose first column, and one row above every image and below the last, is
// padding and stays zero, so that the nine taps are constant distances from a pixel's position and no tap needs a test. Each 16
// channels have a plane of their own (32 bytes a position: of the sixteen lanes that one cycle of a 16-byte read serves, quads of even or odd
// bit parity, no two meet in a bank, wherever the run starts, and a tap's column is a constant in the instruction). Two
// buffers, one of them the layer's input, the other its output; the output buffer still holds the input of the layer before, which is
// what a residual layer adds: each lane reads the four or eight channels that it is about to overwrite. Outputs leave for memory at
// the start of the next layer, 16 bytes a lane as they lie, and their signs with them.
// Weights: at 16 channels in registers (20 of them). Else in LDS as operand fragments (1 KB each, read as they lie); a tap row's are replaced by
// the next layer's as soon as all waves have multiplied it, so they arrive under the rest of the layer.
// The bias is what the accumulators start from. (Input gradients have neither bias nor ReLU.)
// Bound by LDS reads, matrix unit and the epilogue's vector instructions about equally, which a single workgroup on a CU walks one after the other;
// for many images by the stores. us per layer of a run of 14 against a launch each (and 7 to 9 us a launch on top): 16 channels at 32 x 32, 194
// images 2.6 against 7.2 to 8, 1024 images 7.4 forward and 9.0 backward (33 MB written, 4.5 TB/s) against 22; 32 at 16 x 16 1.9 against 5.6 and 5.5 against 14;
// 64 at 8 x 8 2.8 and 2.4 against 5.8, 5.1 against 12. (With operands read where they are used, each product waited for its LDS read: 3.9 us at 16
// channels and 194 images; with one set of weights in registers and signs read by the epilogue, backward 10.2 us at 1024.)
// NORM: a single layer whose input is made here, by a normalisation: the image arrives as the convolution before left it (forward; what the normalisation adds
// in the second buffer) or as the gradient behind the normalisation (input gradient; its own input in the second buffer), is streamed in place
// and to memory, and multiplied. Saves a launch and a read of the tensor in either direction. Bound by memory for many images: 16 channels at 32 x 32, 776
// images, forward 24.5 us for 75 to 100 MB (streaming and convolution apart: 15.3 + 17.8), input gradient 28.2 us for 100 to 125 MB (14.1 + 16.6); 32
// channels at 16 x 16 17.1 (11.4 + 12.5) and 20.0 (8.6 + 12.5), where a workgroup's phases follow one another. Normalised
// ResNet-20 in two modules, us per 8 steps: 4 groups of 194 10030 / 9694, of 16 4436 / 3805, one of 194 4949 / 4574, 4 of 200 recomputing 13436 / 12335.
template <int C, int RUNS, bool DGRAD, bool NORM>
__global__ __launch_bounds__(64 * kWaves, C == 16 || (C == 32 && RUNS <= 4) ? 4 : 2) void conv_chain_kernel(ChainParams p, ChainGeom g, BnParams norm) {
  typedef Shape<C> S;
  constexpr int PB = S::PB, CPP = S::CPP, NBLK = S::NBLK, NBW = S::NBW, WM = S::WM;
  extern __shared__ __align__(16) char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WN, wn = wave % S::WN;
  const int HW = p.H * p.W, Q = p.W + 1;
  const int img0 = blockIdx.x * g.imgs, imgs = min(g.imgs, p.Nimg - img0);
  const int pixels = imgs * HW;
  const size_t pix0 = (size_t)img0 * HW;  // the workgroup's images are consecutive pixels of every tensor
  const int wrep = p.nrep > 1 ? img0 / (p.Nimg / p.nrep) : 0;  // the launcher made sure that they share a data-group
  const size_t wrep_off = (size_t)wrep * p.w_rep;
  const int plane = (int)g.plane, row = Q * 32;  // row: distance of two image rows
  const uint32_t wbuf = 2 * g.buf_bytes;

  // Row r of a block of weights holds output channel chan_of(block, r), so that a lane ends with 4 (C == 16) or 8 consecutive ones
  auto chan_of = [](int b, int r) { return C == 16 ? r : 32 * (b >> 1) + 8 * (r >> 2) + 4 * (b & 1) + (r & 3); };
  // tap whose operand is the pixel a rows below and b columns right of the neighbourhood's top left corner
  auto tap_of = [](int a, int b) { return DGRAD ? 8 - 3 * a - b : 3 * a + b; };
  // C == 16: steps 0-2 hold (0, step) and (1, step), step 3 (2, 0) and (2, 1), step 4 (2, 2); lane (j, q) has 16 bytes of row j at position q / 2
  uint4 wreg[C == 16 ? 5 : 1], next_wreg[C == 16 ? 5 : 1];
  auto load_weights = [&](const void* w, uint4 (&a)[C == 16 ? 5 : 1]) {
    if (C == 16) {
#pragma unroll
      for (int t = 0; t < 5; ++t) {
        const int tap = t < 3 ? tap_of(q >> 1, t) : tap_of(2, t == 3 ? q >> 1 : 2);
        a[t] = *(const uint4*)((const char*)w + wrep_off + (uint32_t)((j * 9 + tap) * PB + (q & 1) * 16));
        if (t == 4 && q >= 2) a[t] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  };
  constexpr int PER = S::SPP * NBLK;  // fragments of a tap row
  constexpr int FP = (PER + kWaves - 1) / kWaves;  // copies of a tap row by each wave (past the end: the last fragment again)
  auto fill_weights = [&](const void* w, int a) {
#pragma unroll
    for (int i = 0; i < FP; ++i) {
      const int f = min(wave + kWaves * i, PER - 1);
      const int step = f / NBLK, n = chan_of(f % NBLK, j);
      const int b = C == 32 ? step : step >> 1, k = C == 32 ? q * 16 : (step & 1) * 64 + q * 16;
      dma16((const char*)w + wrep_off + (uint32_t)((n * 9 + tap_of(a, b)) * PB + k), lds0 + wbuf + (a * PER + f) * 1024);
    }
  };
  // input images by positions; the padding comes from the block of zeros
  auto fill_images = [&](const void* src, uint32_t dst) {
    const char* base = (const char*)src + pix0 * PB;
    for (int f = wave; f < (int)(g.buf_bytes >> 10); f += kWaves) {
      const uint32_t piece = f * 64 + lane, pl = divide(piece, g.dP), in_plane = piece - pl * (uint32_t)(plane >> 4);
      const uint32_t u = in_plane >> 1, line = divide(u, g.dQ), im = divide(line, g.dH1);
      const int w = (int)(u - line * Q) - 1, h = (int)(line - im * (p.H + 1)) - 1;
      const bool in = w >= 0 && h >= 0 && (int)im < imgs && pl < NBLK;
      const char* at = base + (uint32_t)((im * HW + h * p.W + w) * PB + pl * 32 + (in_plane & 1) * 16);
      dma16(in ? at : (const char*)p.zeros, lds0 + dst + f * 1024);
    }
  };
  ChainLayer L = p.layer[0];
  SplitFold<DGRAD, 64 * kWaves, C> fold;
  const int nrep0 = NORM ? img0 / (p.Nimg / norm.W) : 0;  // data-group of the normalisation
  if (NORM) fold.request(norm, nrep0);
  fill_images(NORM && DGRAD ? norm.dy : NORM ? norm.x : p.x, 0);
  load_weights(L.w, wreg);
  if (C != 16) {
#pragma unroll
    for (int a = 0; a < 3; ++a) fill_weights(L.w, a);
  }
  const void* second = NORM ? DGRAD ? norm.x : norm.res : p.res;  // what the second buffer holds at first
  if (second) {
    fill_images(second, g.buf_bytes);
  } else if (!NORM) {
    for (uint32_t a = tid * 16; a < g.buf_bytes; a += 1024 * kWaves) lds_write16(lds0 + g.buf_bytes + a, 0u, 0u, 0u, 0u);
  }

  // pixel of the workgroup -> its position's LDS address in the first plane of the first buffer
  auto position = [&](uint32_t n) {
    const uint32_t line = divide(n, g.dW), im = divide(line, g.dH);
    return (int)(lds0 + ((line + im + 1) * Q + (n - line * p.W) + 1) * 32);  // im images above, one padding row each
  };
  // Sums of these with a layer's offsets are formed where they are used: the compiler would keep every one of them in a register.
  auto opaque = [](int v) { asm volatile("" : "+v"(v)); return v; };
  // LDS address, in the layer's input buffer, of this lane's part of the operand at the top left corner of its pixel's neighbourhood, for every
  // run (runs past the last pixel read it again); own: distance to the lane's output channels of that pixel
  int at[RUNS];
#pragma unroll
  for (int u = 0; u < RUNS; ++u)
    at[u] = position((uint32_t)min((wm + WM * u) * 16 + j, pixels - 1)) - row - 32 + (q & 1) * 16 + (q >> 1) * (C == 16 ? row : plane);
  const int own = row + 32 + (C == 16 ? q * 8 - (q & 1) * 16 - (q >> 1) * row : 2 * wn * plane);
  // the 16-byte pieces of an output that this thread stores (past the end: the last one again)
  constexpr int NS = (RUNS * WM * 16 * CPP + 64 * kWaves - 1) / (64 * kWaves);
  int piece[NS], piece_at[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    piece[k] = min(tid + 64 * kWaves * k, pixels * CPP - 1);
    const int c = piece[k] % CPP;
    piece_at[k] = position((uint32_t)piece[k] / CPP) + (c & 1) * 16 + (c >> 1) * plane;
  }
  auto store_out = [&](int buf, char* y, char* bits) {
    uint32_t s[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const uint4 v = lds_read16(opaque(piece_at[k]) + buf);
      *(uint4*)(y + ((uint32_t)opaque(piece[k]) << 4)) = v;
      if (!DGRAD) s[k] = nonzero2(v.x) | nonzero2(v.y) << 2 | nonzero2(v.z) << 4 | nonzero2(v.w) << 6;  // behind a ReLU: nothing is negative
    }
    if (!DGRAD && bits) {  // pair e's low half belongs to bit 2 e, its high half (bit 16) to bit 2 e + 1
#pragma unroll
      for (int k = 0; k < NS; ++k) *(uint8_t*)(bits + (uint32_t)opaque(piece[k])) = (uint8_t)(s[k] | s[k] >> 15);
    }
  };
  // What else a layer reads from memory is asked for a layer ahead: its bias (forward), or the signs of its outputs (input gradient), bytes
  // as they lie, copied to slots behind the weights (16 channels, whose layers are the shortest: two layers ahead).
  constexpr int SG = DGRAD ? 1 : 0;
  const size_t sign0 = pix0 * (C / 8);  // first byte of this workgroup's images in a sign plane, copied from the 16-byte line that holds it
  const uint32_t signs = wbuf + (C == 16 ? 0 : 3 * PER * 1024);
  auto load_bias = [&](const ChainLayer& l, f32x4_t (&b)[NBW]) {
    const float* at = l.bias ? l.bias + (size_t)wrep * p.bias_rep : (const float*)p.zeros;
#pragma unroll
    for (int i = 0; i < NBW; ++i) b[i] = *(const f32x4_t*)(at + chan_of(wn * NBW + i, 4 * q));
  };
  auto fill_signs = [&](const ChainLayer& l, int slot) {  // one copy by each wave (past the end: the last one again)
    const char* from = l.maskbits ? (const char*)l.maskbits : (const char*)p.zeros;
    const size_t last = l.maskbits ? ((size_t)p.Nimg * HW * (C / 8) - 1) & ~(size_t)15 : 0;  // (blocks of the arena are whole lines)
    const int f = min(wave, (int)(g.sign_bytes >> 10) - 1);
    const size_t off = (sign0 & ~(size_t)15) + (size_t)(f * 64 + lane) * 16;
    dma16(from + (off < last ? off : last), lds0 + signs + slot * g.sign_bytes + f * 1024);
  };
  constexpr int SLOTS = sign_slots(C);
  const uint32_t sign_at = lds0 + signs + (uint32_t)(sign0 & 15) + (C == 16 ? 0 : 4 * wn + q);
  f32x4_t start[NBW] = {}, next_start[NBW] = {};
  if (!DGRAD) load_bias(L, start);
  if (DGRAD) fill_signs(L, 0);
  if (DGRAD && C == 16 && !NORM && p.n > 1) fill_signs(p.layer[1], 1);
  float* cf = (float*)(smem + g.fold_at + 8 * fold.kDoubles);
  if (NORM) fold.finish(norm, nrep0, img0 % (p.Nimg / norm.W) == 0, (double*)(smem + g.fold_at), cf);
  wait_vm<0>();
  wg_barrier();
  if (NORM) {  // what is normalised -> the layer's input, in place and to memory (the expressions are those of bn_fwd_apply_kernel and bn_bwd_apply_kernel)
    const int c0 = tid % CPP * 8;
    float k[DGRAD ? 5 : 2][8];
#pragma unroll
    for (int i = 0; i < (DGRAD ? 5 : 2); ++i) {
      const float4 lo = *(const float4*)(cf + i * C + c0), hi = *(const float4*)(cf + i * C + c0 + 4);
      k[i][0] = lo.x; k[i][1] = lo.y; k[i][2] = lo.z; k[i][3] = lo.w; k[i][4] = hi.x; k[i][5] = hi.y; k[i][6] = hi.z; k[i][7] = hi.w;
    }
    char* out = (char*)(DGRAD ? norm.dx : norm.y) + pix0 * PB;
    char* out_bits = !DGRAD && norm.bits_out ? (char*)norm.bits_out + pix0 * (C / 8) : nullptr;
    auto halves = [](const uint4& v, float (&f)[8]) {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = __uint_as_float(e & 1 ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16);
    };
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      if (tid + 64 * kWaves * i >= pixels * CPP) break;
      const int mine = opaque(piece_at[i]);
      float f[8], h[8] = {};
      halves(lds_read16(mine), f);
      if (second) halves(lds_read16(mine + (int)g.buf_bytes), h);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (DGRAD) {
          const float xh = (h[e] - k[0][e]) * k[DGRAD ? 1 : 0][e];
          f[e] = k[DGRAD ? 2 : 0][e] * f[e] - k[DGRAD ? 3 : 0][e] - xh * k[DGRAD ? 4 : 0][e];
        } else {
          float v = fmaf(f[e], k[0][e], k[1][e]);
          if (second) v += h[e];
          if (norm.relu) v = v > 0.f ? v : 0.f;
          f[e] = v;
        }
      }
      const uint4 o = make_uint4(pack_bf16_rne(f[0], f[1]), pack_bf16_rne(f[2], f[3]), pack_bf16_rne(f[4], f[5]), pack_bf16_rne(f[6], f[7]));
      lds_write16(mine, o.x, o.y, o.z, o.w);
      *(uint4*)(out + ((uint32_t)opaque(piece[i]) << 4)) = o;
      if (out_bits) {
        const uint32_t t = nonzero2(o.x) | nonzero2(o.y) << 2 | nonzero2(o.z) << 4 | nonzero2(o.w) << 6;
        *(uint8_t*)(out_bits + (uint32_t)opaque(piece[i])) = (uint8_t)(t | t >> 15);
      }
    }
    wg_barrier();
    if (DGRAD && p.res) fill_images(p.res, g.buf_bytes);
  }

  // A wave's loads, copies and stores retire in the order of their issue; copies are waited for by the number of younger operations, so
  // that neither the stores nor the copies of later pieces are.
  char *prev_y = nullptr, *prev_bits = nullptr;
  for (int l = 0; l < (NORM ? 1 : p.n); ++l) {
    const int src = l & 1 ? (int)g.buf_bytes : 0, dst = (int)g.buf_bytes - src;
    const bool more = !NORM && l + 1 < p.n;
    const ChainLayer next = NORM ? L : p.layer[more ? l + 1 : l];
    if (!DGRAD && !NORM) load_bias(next, next_start);  // (the last layer: its own again)
    if (!NORM) load_weights(next.w, next_wreg);
    if (!NORM && l > 0) store_out(src, prev_y, prev_bits);
    if (DGRAD && C == 16 && !NORM && l + 2 < p.n) fill_signs(p.layer[l + 2], (l + 2) % SLOTS);

    // Operands of one item (a step and G of the runs) are requested while the item before is multiplied; left to itself the compiler
    // reads each one just ahead of its product and waits for it.
    f32x4_t acc[RUNS][NBW];
    constexpr int G = RUNS == 1 ? 1 : RUNS > 4 && C == 16 ? 2 : RUNS < 4 ? RUNS : 4, NG = (RUNS + G - 1) / G;
    uint4 x[2][G];
    if (C == 16) {
      const int last = 2 * row + (q >> 1) * (32 - row);  // steps 3 and 4: the neighbourhood's last row
      auto request = [&](int i, uint4 (&v)[G]) {
        const int t = i / NG;
#pragma unroll
        for (int k = 0; k < G; ++k) {
          const int u = i % NG * G + k;
          if (u >= RUNS) continue;
          v[k] = lds_read16(t < 3 ? at[u] + 32 * t : t == 3 ? at[u] + last : q >= 2 ? (int)lds0 : at[u] + last + 64);  // (no tap: position 0, which is padding)
        }
      };
      request(0, x[0]);
#pragma unroll
      for (int i = 0; i < 5 * NG; ++i) {
        if (i + 1 < 5 * NG) request(i + 1, x[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < G; ++k) {
          const int u = i % NG * G + k;
          if (u < RUNS) acc[u][0] = mfma16(wreg[i / NG], x[i & 1][k], i < NG ? start[0] : acc[u][0]);
        }
      }
    } else {
      const uint32_t wfrag = lds0 + wbuf + wn * NBW * 1024 + lane * 16;
      constexpr int KS = C == 16 ? 1 : C / 32, ITEMS = 3 * KS * NG;  // of a tap row: columns b, within them k-steps, within them groups of runs
      uint4 w[2][NBW];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        auto request = [&](int i, uint4 (&v)[G]) {
          const int st = i / NG, b = st / KS, ks = st % KS;
          if (i % NG == 0)
#pragma unroll
            for (int n = 0; n < NBW; ++n) w[st & 1][n] = lds_read16(wfrag + (a * PER + st * NBLK + n) * 1024);
#pragma unroll
          for (int k = 0; k < G; ++k) {
            const int u = i % NG * G + k;
            if (u < RUNS) v[k] = lds_read16(at[u] + ks * 2 * plane + 32 * b);
          }
        };
        request(0, x[0]);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          if (i + 1 < ITEMS) request(i + 1, x[(i + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < G; ++k) {
            const int u = i % NG * G + k;
            if (u >= RUNS) continue;
#pragma unroll
            for (int n = 0; n < NBW; ++n) acc[u][n] = mfma16(w[i / NG & 1][n], x[i & 1][k], a == 0 && i < NG ? start[n] : acc[u][n]);
          }
        }
#pragma unroll
        for (int u = 0; u < RUNS; ++u) at[u] = opaque(at[u] + (a < 2 ? row : -2 * row));
        // This row's weights have been read by everyone, and the next row's, copied during the layer before, are there (behind the last row:
        // this layer's signs). Younger than they: the copies behind them, this layer's stores, the next layer's weights so far.
        constexpr int OPS = NS, OPSB = DGRAD ? NS : 2 * NS;  // without and with the signs of the layer before (the bias is not counted on)
        const bool with_bits = !DGRAD && prev_bits;
        if (NORM) continue;
        if (a == 0) {
          if (with_bits) wait_vm<FP + SG + OPSB>();
          else wait_vm<FP + SG + OPS>();
        } else if (a == 1) {
          if (!more) wait_vm<SG + OPS>();
          else if (with_bits) wait_vm<SG + OPSB + FP>();
          else wait_vm<SG + OPS + FP>();
        } else if (DGRAD) {
          if (more) wait_vm<OPS + 2 * FP>();
          else wait_vm<OPS>();
        }
        wg_barrier();
        if (more) fill_weights(next.w, a);
        if (DGRAD && a == 2 && more) fill_signs(next, (l + 1) & 1);
      }
    }

    if (NORM && L.add) {  // what the layer adds, asked for ahead of the products
      wait_vm<0>();
      wg_barrier();
    }
    // epilogue, a few runs at a time: what they add, arithmetic, stores
    const int to_own = own + dst - src, to_next = dst - src;
    constexpr int NV = 4 * NBW, GRP = C == 16 ? 4 : 2;
    const float lower = !DGRAD && L.relu ? 0.f : -__builtin_inff();
    const uint32_t all = DGRAD && !L.maskbits ? 0xffffu : 0u;
#pragma unroll
    for (int u0 = 0; u0 < RUNS; u0 += GRP) {
      float v[GRP][NV];
      if (L.add) {
        uint32_t r[GRP][NV / 2];
#pragma unroll
        for (int i = 0; i < GRP && u0 + i < RUNS; ++i) {
          const uint32_t mine = at[u0 + i] + to_own;
          if (C == 16) { const uint2 t = lds_read8(mine); r[i][0] = t.x; r[i][1] = t.y; }
          else { const uint4 t = lds_read16(mine); r[i][0] = t.x; r[i][1] = t.y; r[i][NV / 2 - 2] = t.z; r[i][NV / 2 - 1] = t.w; }
        }
#pragma unroll
        for (int i = 0; i < GRP && u0 + i < RUNS; ++i)
#pragma unroll
          for (int e = 0; e < NV; ++e)
            v[i][e] = fmaf(L.alpha, acc[u0 + i][e >> 2][e & 3], __uint_as_float(e & 1 ? r[i][e >> 1] & 0xffff0000u : r[i][e >> 1] << 16));
      } else {
#pragma unroll
        for (int i = 0; i < GRP && u0 + i < RUNS; ++i)
#pragma unroll
          for (int e = 0; e < NV; ++e) v[i][e] = L.alpha * acc[u0 + i][e >> 2][e & 3];
      }
      uint32_t keep[GRP];
      if (DGRAD) {
        const int n0 = opaque(wm * 16 + j);
#pragma unroll
        for (int i = 0; i < GRP && u0 + i < RUNS; ++i) {
          const uint32_t from = sign_at + l % SLOTS * g.sign_bytes + min(n0 + WM * 16 * (u0 + i), pixels - 1) * (C / 8);
          if (C == 16) keep[i] = *(const uint16_t DDS_LDS_AS*)(size_t)from;
          else keep[i] = *(const uint8_t DDS_LDS_AS*)(size_t)from;
        }
      }
#pragma unroll
      for (int i = 0; i < GRP && u0 + i < RUNS; ++i) {
        const int u = u0 + i;
        if (!DGRAD)
#pragma unroll
          for (int e = 0; e < NV; ++e) v[i][e] = __builtin_amdgcn_fmed3f(v[i][e], lower, __builtin_inff());  // one instruction; NaN -> lower
        uint32_t o[NV / 2];
#pragma unroll
        for (int e = 0; e < NV / 2; ++e) o[e] = pack_bf16_rne(v[i][2 * e], v[i][2 * e + 1]);
        if (DGRAD) {  // bits 2 e and 2 e + 1 of the signs -> 0 / 1 in either half of a pair
          const uint32_t k = (C == 16 ? keep[i] >> (4 * q) : keep[i]) | all, k2 = k | k << 15;
#pragma unroll
          for (int e = 0; e < NV / 2; ++e) o[e] = keep2(o[e], (k2 >> (2 * e)) & 0x00010001u);
        }
        const uint32_t mine = at[u] + to_own;
        const int n = (wm + WM * u) * 16;
        if (n + 16 <= pixels || n + j < pixels) {
          if (C == 16) lds_write8(mine, o[0], o[1]);
          else lds_write16(mine, o[0], o[1], o[NV / 2 - 2], o[NV / 2 - 1]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < RUNS; ++u) at[u] = opaque(at[u] + to_next);
    prev_y = (char*)L.y + pix0 * PB;
    prev_bits = L.bits_out ? (char*)L.bits_out + pix0 * (C / 8) : nullptr;
    L = next;
#pragma unroll
    for (int b = 0; b < NBW; ++b) start[b] = next_start[b];
    if (C == 16) {
#pragma unroll
      for (int t = 0; t < 5; ++t) wreg[t] = next_wreg[t];
    }
    // the next layer's first tap row, or (16 channels) its signs: older than this layer's stores and the signs after them
    if (NORM) {}
    else if (more && C != 16) wait_vm<2 * FP + SG>();
    else if (DGRAD && l + 2 < p.n) wait_vm<NS + 1>();
    else if (DGRAD && more) wait_vm<NS>();
    wg_barrier();
  }
  store_out(NORM || (p.n & 1) ? (int)g.buf_bytes : 0, prev_y, prev_bits);
}

// Wider layers, whose image fits in LDS once: 64 channels at up to 1024 pixels, 128 at up to 256. The outputs of a layer wait in the accumulators
// until every wave has read its last operand, then take the input's place. A wave owns 64 output channels of RUNS runs of 16 pixels; a stage is half
// of a tap's input channels (18 a layer, 32 MFMAs of a wave at full size). Its weights travel in a ring of four slots, four stages ahead;
// the fragments of the next stage are read into registers during this one, so that between a stage's barrier and its first product lies
// nothing. What a residual layer adds is read from memory again, where this lane (or the launch before) wrote it. Lanes whose run ends past the
// last pixel repeat it: they compute and write the same values.
// us a layer and pass, a launch a layer / here: 64 channels at 32 x 32, 256 images 28 / 24, 512 images 52 / 45; 128 channels at 16 x 16, 256 images
// 32 / 19, 512 images 45 / 38, of which the matrix unit is busy for 8 an image. The rest goes to 18 barriers and an epilogue that waits for its
// residual and signs and for room among the stores. Stores spread over the next layer's stages, with the residual asked for in the last ones, took
// registers that 64 channels do not have (32 us at 256 images) and gave nothing at 128 channels.
struct WideGeom {
  int imgs;
  uint32_t plane, buf_bytes;
  Divisor dP, dQ, dH1, dW, dH;
};

template <int C, int RUNS, bool DGRAD>
__global__ __launch_bounds__(64 * kWaves, 2) void conv_wide_chain_kernel(ChainParams p, WideGeom g) {
  constexpr int PB = 2 * C, NBLK = C / 16, WN = C / 64, WM = kWaves / WN;
  constexpr int KPS = C / 64;                       // 32-channel steps of a stage
  constexpr int SLOT = KPS * NBLK * 1024;           // fragments of a stage
  constexpr int FILLS = C == 64 ? 1 : 2;            // copies of a wave: every other stage (C == 64), or two a stage
  constexpr int YOUNGER = C == 64 ? 1 : 2 * FILLS;  // copies of a wave behind the ones that a stage waits for
  extern __shared__ __align__(16) char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(DDS_LDS_AS char*)smem;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int HW = p.H * p.W, Q = p.W + 1;
  const int img0 = blockIdx.x * g.imgs, imgs = min(g.imgs, p.Nimg - img0);
  const int pixels = imgs * HW;
  const size_t pix0 = (size_t)img0 * HW;  // the workgroup's images are consecutive pixels of every tensor
  const int wrep = p.nrep > 1 ? img0 / (p.Nimg / p.nrep) : 0;
  const size_t wrep_off = (size_t)wrep * p.w_rep;
  const int plane = (int)g.plane, row = Q * 32;
  const uint32_t ring = lds0 + g.buf_bytes;

  auto opaque = [](int v) { asm volatile("" : "+v"(v)); return v; };
  auto chan_of = [](int b, int r) { return 32 * (b >> 1) + 8 * (r >> 2) + 4 * (b & 1) + (r & 3); };  // as in conv_chain_kernel
  const int wblock = chan_of(C == 64 ? wave & 3 : wave, 0) * 9 * PB;
  auto fill_stage = [&](const void* w, int t, int slot) {  // stage t of a layer
    const int tap = DGRAD ? 8 - (t >> 1) : t >> 1;
    const int l = opaque(lane);  // (formed here: kept, it would go to scratch memory, and a read of that waits for every copy)
    const uint32_t wlane = (uint32_t)(chan_of(0, l & 15) * 9 * PB + (l >> 4) * 16);
    const uint64_t from = (uint64_t)w + wrep_off + (uint32_t)(wblock + tap * PB + (t & 1) * C);  // (uniform, which the compiler loses track of)
    const char* base = (const char*)((uint64_t)__builtin_amdgcn_readfirstlane((int)(from >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)from));
    if (C == 64) {
      if (wave >> 2 == (t & 1)) dma16s(base, wlane, ring + slot * SLOT + (wave & 3) * 1024);
    } else {
#pragma unroll
      for (int k = 0; k < KPS; ++k) dma16s(base + k * 64, wlane, ring + slot * SLOT + (k * NBLK + wave) * 1024);
    }
  };
  {
    const char* base = (const char*)p.x + pix0 * PB;
    for (int f = wave; f < (int)(g.buf_bytes >> 10); f += kWaves) {
      const uint32_t piece = f * 64 + lane, pl = divide(piece, g.dP), in_plane = piece - pl * (uint32_t)(plane >> 4);
      const uint32_t u = in_plane >> 1, line = divide(u, g.dQ), im = divide(line, g.dH1);
      const int w = (int)(u - line * Q) - 1, h = (int)(line - im * (p.H + 1)) - 1;
      const bool in = w >= 0 && h >= 0 && (int)im < imgs && pl < NBLK;
      const char* at = base + (uint32_t)((im * HW + h * p.W + w) * PB + pl * 32 + (in_plane & 1) * 16);
      dma16(in ? at : (const char*)p.zeros, lds0 + f * 1024);
    }
  }
  ChainLayer L = p.layer[0];
#pragma unroll
  for (int t = 0; t < 4; ++t) fill_stage(L.w, t, t);

  int at[RUNS];  // as in conv_chain_kernel; the tap row moves it
#pragma unroll
  for (int u = 0; u < RUNS; ++u) {
    const uint32_t n = (uint32_t)min((wm + WM * u) * 16 + j, pixels - 1);
    const uint32_t line = divide(n, g.dW), im = divide(line, g.dH);
    at[u] = (int)(lds0 + ((line + im + 1) * Q + (n - line * p.W) + 1) * 32) - row - 32 + (q & 1) * 16 + (q >> 1) * plane;
  }
  const int own = row + 32 + wn * 4 * plane;
  auto load_bias = [&](const ChainLayer& l, f32x4_t (&b)[4]) {
    const float* from = l.bias ? l.bias + (size_t)wrep * p.bias_rep : (const float*)p.zeros;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = *(const f32x4_t*)(from + chan_of(wn * 4 + i, 4 * q));
  };
  f32x4_t start[4] = {};
  if (!DGRAD) load_bias(L, start);
  wait_vm<0>();
  wg_barrier();

  constexpr int G = RUNS < 2 ? 1 : 2, NG = (RUNS + G - 1) / G, ITEMS = KPS * NG;  // items of a stage: steps, within them groups of runs
  uint4 x[2][G], w[2][KPS][4];
  auto read_weights = [&](int slot, uint4 (&v)[KPS][4]) {
#pragma unroll
    for (int k = 0; k < KPS; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[k][i] = lds_read16(ring + slot * SLOT + (k * NBLK + wn * 4 + i) * 1024 + lane * 16);
  };
  read_weights(0, w[0]);
  int slot = 0;
  const void *before = p.res, *input = p.x;  // what the layer before read, what this one does
  for (int l = 0; l < p.n; ++l) {
    const bool more = l + 1 < p.n;
    const ChainLayer next = p.layer[more ? l + 1 : l];
    f32x4_t acc[RUNS][4];
    auto request = [&](int i, int item, uint4 (&v)[G]) {  // stage 6 a + i: tap column i / 2, half i % 2 of the channels
      const int ks = (i & 1) * KPS + item / NG;
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const int u = item % NG * G + k;
        if (u < RUNS) v[k] = lds_read16((ks == 0 ? at[u] : opaque(at[u]) + ks * 2 * plane) + 32 * (i >> 1));
      }
    };
    request(0, 0, x[0]);
#pragma unroll
    for (int u = 0; u < RUNS; ++u)
#pragma unroll
      for (int n = 0; n < 4; ++n) acc[u][n] = start[n];
#pragma unroll 1
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        // Everyone has read this stage's weights, and the next stage's are there: copied four stages ahead. (In order: behind them this wave's copies
        // of two more stages and, at a layer's first three, the stores of the layer before.)
        if (a == 0 && i < 3 && l > 0) wait_vm<YOUNGER + 2 * RUNS>();
        else if (i >= 3 && a == 2 && !more) wait_vm<0>();  // (nothing is copied any more)
        else wait_vm<YOUNGER>();
        wg_barrier();
        const int t = a * 6 + i + 4;
        if (t < 18) fill_stage(L.w, t, slot);
        else if (more) fill_stage(next.w, t - 18, slot);
        slot = (slot + 1) & 3;
        read_weights(slot, w[(i + 1) & 1]);
#pragma unroll
        for (int item = 0; item < ITEMS; ++item) {
          const int cur = i * ITEMS + item;
          if (item + 1 < ITEMS) request(i, item + 1, x[(cur + 1) & 1]);
          else if (i < 5) request(i + 1, 0, x[(cur + 1) & 1]);
          else {
#pragma unroll
            for (int u = 0; u < RUNS; ++u) at[u] = opaque(at[u] + row);
            if (a < 2) request(0, 0, x[(cur + 1) & 1]);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < G; ++k) {
            const int u = item % NG * G + k;
            if (u >= RUNS) continue;
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[u][n] = mfma16(w[i & 1][item / NG][n], x[cur & 1][k], acc[u][n]);
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < RUNS; ++u) at[u] = opaque(at[u] - 3 * row);

    // epilogue: a run at a time, what it needs from memory asked for a run ahead
    const float lower = !DGRAD && L.relu ? 0.f : -__builtin_inff();
    const char* res = (const char*)before + pix0 * PB;
    const char* mask = DGRAD ? (const char*)L.maskbits + pix0 * (C / 8) : nullptr;
    const int n0 = opaque(wm * 16 + j);
    auto pixel = [&](int u) { return min(opaque(n0) + WM * 16 * u, pixels - 1); };
    uint4 r[2][2];
    uint32_t keep[2][2];
    auto ask = [&](int u, int set) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        if (L.add) r[set][b] = *(const uint4*)(res + (uint32_t)(pixel(u) * PB + wn * 128 + b * 64 + q * 16));
        if (DGRAD) keep[set][b] = L.maskbits ? *(const uint8_t*)(mask + (uint32_t)(pixel(u) * (C / 8) + wn * 8 + b * 4 + q)) : 0xffu;
      }
    };
    ask(0, 0);
    wg_barrier();  // every wave has read its last operand
    char* y = (char*)L.y + pix0 * PB;
    char* bits = !DGRAD && L.bits_out ? (char*)L.bits_out + pix0 * (C / 8) : nullptr;
#pragma unroll
    for (int u = 0; u < RUNS; ++u) {
      const int set = u & 1;
      if (u + 1 < RUNS) ask(u + 1, set ^ 1);
      else if (!DGRAD) load_bias(next, start);  // (the last layer: its own again)
      {
        const int n = pixel(u);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = L.alpha * acc[u][2 * b + (e >> 2)][e & 3];
          if (L.add) {
            const uint32_t rr[4] = {r[set][b].x, r[set][b].y, r[set][b].z, r[set][b].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += __uint_as_float(e & 1 ? rr[e >> 1] & 0xffff0000u : rr[e >> 1] << 16);
          }
          if (!DGRAD)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __builtin_amdgcn_fmed3f(v[e], lower, __builtin_inff());  // one instruction; NaN -> lower
          uint32_t o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = pack_bf16_rne(v[2 * e], v[2 * e + 1]);
          if (DGRAD) {  // bits 2 e and 2 e + 1 of the signs -> 0 / 1 in either half of a pair
            const uint32_t k2 = keep[set][b] | keep[set][b] << 15;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = keep2(o[e], (k2 >> (2 * e)) & 0x00010001u);
          }
          lds_write16(at[u] + own + b * 2 * plane, o[0], o[1], o[2], o[3]);
          *(uint4*)(y + (uint32_t)(n * PB + wn * 128 + b * 64 + q * 16)) = make_uint4(o[0], o[1], o[2], o[3]);
          if (!DGRAD && bits) {  // pair e's low half belongs to bit 2 e, its high half (bit 16) to bit 2 e + 1; behind a ReLU nothing is negative
            const uint32_t t = nonzero2(o[0]) | nonzero2(o[1]) << 2 | nonzero2(o[2]) << 4 | nonzero2(o[3]) << 6;
            *(uint8_t*)(bits + (uint32_t)(n * (C / 8) + wn * 8 + b * 4 + q)) = (uint8_t)(t | t >> 15);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    before = input;
    input = L.y;
    L = next;
    wg_barrier();
  }
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

int plane_bytes(int H, int W, int imgs) { return ((imgs * (H + 1) + 1) * (W + 1) + 1) * 32; }
int buffer_bytes(int C, int H, int W, int imgs) { return cdiv(plane_bytes(H, W, imgs) * (C / 16), 1024) * 1024; }
int sign_bytes(int C, int H, int W, int imgs) {  // of the 16-byte lines that may hold them
  const int n = imgs * H * W * (C / 8);
  return cdiv(n % 16 ? n + 15 : n, 1024) * 1024;
}
int weight_bytes(int C) { return C == 16 ? 0 : 9 * C / 32 * (C / 16) * 1024; }
int lds_bytes(int C, int H, int W, int imgs) { return 2 * buffer_bytes(C, H, W, imgs) + weight_bytes(C) + sign_slots(C) * sign_bytes(C, H, W, imgs); }
// with a normalisation: one slot of signs, and where its factors are made (SplitFold::kDoubles and kBnCoefRows rows)
int norm_fold_at(int C, int H, int W, int imgs) { return 2 * buffer_bytes(C, H, W, imgs) + weight_bytes(C) + sign_bytes(C, H, W, imgs); }
int norm_lds_bytes(int C, int H, int W, int imgs) { return norm_fold_at(C, H, W, imgs) + 8 * 2 * kWaves * C + 4 * kBnCoefRows * C; }
int wave_rows(int C) { return C == 64 ? kWaves / 2 : kWaves; }
int most_runs(int C) { return C == 64 ? 4 : 8; }

template <int C, int RUNS, bool NORM>
void launch_inst(const ChainParams& p, const ChainGeom& g, const BnParams& n, int wgs, int smem, hipStream_t s) {
  static DeviceOnce lds[2];
  if (p.dgrad) {
    allow_whole_lds(lds[1], (const void*)conv_chain_kernel<C, RUNS, true, NORM>);
    conv_chain_kernel<C, RUNS, true, NORM><<<wgs, 64 * kWaves, smem, s>>>(p, g, n);
  } else {
    allow_whole_lds(lds[0], (const void*)conv_chain_kernel<C, RUNS, false, NORM>);
    conv_chain_kernel<C, RUNS, false, NORM><<<wgs, 64 * kWaves, smem, s>>>(p, g, n);
  }
}

int wide_lds_bytes(int C, int H, int W, int imgs) { return buffer_bytes(C, H, W, imgs) + 4 * (C / 64) * (C / 16) * 1024; }
template <int C, int RUNS>
void launch_wide_inst(const ChainParams& p, const WideGeom& g, int wgs, int smem, hipStream_t s) {
  static DeviceOnce lds[2];
  if (p.dgrad) {
    allow_whole_lds(lds[1], (const void*)conv_wide_chain_kernel<C, RUNS, true>);
    conv_wide_chain_kernel<C, RUNS, true><<<wgs, 64 * kWaves, smem, s>>>(p, g);
  } else {
    allow_whole_lds(lds[0], (const void*)conv_wide_chain_kernel<C, RUNS, false>);
    conv_wide_chain_kernel<C, RUNS, false><<<wgs, 64 * kWaves, smem, s>>>(p, g);
  }
}

}  // namespace

// Images of a workgroup: as few as fill the chip once; more share a copy of the weights.
static int images_of(int C, int H, int W, int Nimg, int nrep) {
  if ((C != 16 && C != 32 && C != 64) || H < 1 || W < 1 || Nimg < 1 || nrep < 1 || Nimg % nrep != 0) return 0;
  if ((long long)H * W > 4096) return 0;  // (far beyond what LDS holds; keeps the products below in range)
  auto fits = [&](int imgs) {
    return lds_bytes(C, H, W, imgs) <= 160 * 1024 && cdiv(cdiv(imgs * H * W, 16), wave_rows(C)) <= most_runs(C);
  };
  int imgs = 0;
  for (int i = 1; i <= 8 && fits(i) && (nrep == 1 || Nimg / nrep % i == 0); i *= 2) {
    imgs = i;
    if (cdiv(Nimg, i) <= 256) break;
  }
  return imgs;
}

// The same of the wide kernel.
static int wide_images_of(int C, int H, int W, int Nimg, int nrep) {
  if ((C != 64 && C != 128) || H < 1 || W < 1 || Nimg < 1 || nrep < 1 || Nimg % nrep != 0 || (long long)H * W > 4096) return 0;
  auto fits = [&](int imgs) {
    return wide_lds_bytes(C, H, W, imgs) <= 160 * 1024 && cdiv(cdiv(imgs * H * W, 16), kWaves * 64 / C) <= (C == 64 ? 8 : 4);
  };
  int imgs = 0;
  for (int i = 1; i <= 8 && fits(i) && (nrep == 1 || Nimg / nrep % i == 0); i *= 2) {
    imgs = i;
    if (cdiv(Nimg, i) <= 256) break;
  }
  return imgs;
}
static int wide_runs(int C, int H, int W, int imgs) { return cdiv(cdiv(imgs * H * W, 16), kWaves * 64 / C); }

// Fewest layers of a wide run worth a shared launch. An image keeps its CU for the whole run, so the images have to fill the chip once (192 of 256
// CUs and more) or twice (460 of 512). us per step of a net with two (four) such layers, a launch a layer / here: 64 channels at 32 x 32, 128 images 174
// / 192 (273 / 291), 194 images 243 / 223 (397 / 359), 256 images 296 / 280 (455 / 401), 384 images 376 / 406 (612 / 627), 460 images 436 / 443
// (719 / 679), 700 images 598 / 623 (974 / 1036); at 24 x 24, 256 images 214 / 182 (345 / 269), 384 images 287 / 295 (440 / 423), 512 images 348 /
// 331 (540 / 471); 128 channels at 16 x 16, 128 images 160 / 160 (249 / 244), 256 images 261 / 227 (388 / 312), 512 images 380 / 343 (647 / 562), 1024 images 652
// / 629 (1108 / 1050); at 12 x 12, 160 images 148 / 149 (228 / 218), 194 images 159 / 155 (256 / 238), 256 images 201 / 170 (325 / 253), 384 images 267 /
// 278 (395 / 399), 512 images 317 / 286 (513 / 439), 700 images 359 / 371 (599 / 601); at 8 x 8, 128 images 92 / 107 (127 / 150), 194 images 120 / 113 (184 /
// 159), 512 images 161 / 143 (253 / 205).
static int wide_least(int C, int H, int W, int Nimg, int nrep) {
  const int imgs = wide_images_of(C, H, W, Nimg, nrep);
  if (imgs == 0) return 0;
  const int wgs = cdiv(Nimg, imgs);
  if (wgs < 192 || (wgs > 256 && wgs < 460) || wgs > 512) return 0;
  return wgs > 256 && wide_runs(C, H, W, imgs) == 8 ? 4 : 2;
}

// us per step of a net with two (six) such layers in one module, a launch a layer / here, at the best of several runs: 16 channels at 32 x 32, 64
// images 75 / 76, 194 images 98 / 90, 776 images 200 / 194; 32 channels at 16 x 16, 64 images 74 / 67, 776 images 138 / 128; 64 channels at 8 x
// 8, 64 images 78 / 74, 776 images 124 / 112. Where one image takes more than half of a CU's LDS, two layers do not make up for a last
// round of few workgroups, and other modules' kernels find no room beside them: 64 channels at 14 x 14, 64 images 87 / 92 (137 / 132), 194 images 115 /
// 105 (214 / 159), 776 images 221 / 228 (458 / 413); 32 channels at 28 x 28, 8 images 69 / 75 (106 / 112), 194 images 114 / 110 (199 / 159), 776
// images 267 / 273 (527 / 504). Two such layers of 64 channels in either of two modules, 194 images of 14 x 14: 180 / 183.
int conv_chain_least(int C, int H, int W, int Nimg, int nrep) {
  const int imgs = images_of(C, H, W, Nimg, nrep);
  if (imgs == 0) return wide_least(C, H, W, Nimg, nrep);
  if (imgs > 1 || lds_bytes(C, H, W, 1) <= 80 * 1024) return 2;
  return Nimg < 64 && H * W > 640 ? 0 : 4;
}

static void launch_wide_chain(int C, const ChainParams& p, hipStream_t s) {
  WideGeom g;
  g.imgs = wide_images_of(C, p.H, p.W, p.Nimg, p.nrep > 1 ? p.nrep : 1);
  g.plane = plane_bytes(p.H, p.W, g.imgs);
  g.buf_bytes = buffer_bytes(C, p.H, p.W, g.imgs);
  g.dP = make_divisor1(g.plane / 16);
  g.dQ = make_divisor1(p.W + 1);
  g.dH1 = make_divisor1(p.H + 1);
  g.dW = make_divisor1(p.W);
  g.dH = make_divisor1(p.H);
  const int wgs = cdiv(p.Nimg, g.imgs), smem = wide_lds_bytes(C, p.H, p.W, g.imgs);
  const int runs = wide_runs(C, p.H, p.W, g.imgs);
#define DDS_WIDE_CASE(C, RUNS) \
  case (C) * 8 + (RUNS) - 1: launch_wide_inst<C, RUNS>(p, g, wgs, smem, s); break;
  switch (C * 8 + runs - 1) {
    DDS_WIDE_CASE(64, 2) DDS_WIDE_CASE(64, 3) DDS_WIDE_CASE(64, 4)
    DDS_WIDE_CASE(64, 5) DDS_WIDE_CASE(64, 6) DDS_WIDE_CASE(64, 7) DDS_WIDE_CASE(64, 8)
    DDS_WIDE_CASE(128, 1) DDS_WIDE_CASE(128, 2) DDS_WIDE_CASE(128, 3) DDS_WIDE_CASE(128, 4)
  }
#undef DDS_WIDE_CASE
}

template <bool NORM>
static void launch_narrow(int C, int imgs, const ChainParams& p, const BnParams& n, hipStream_t s) {
  ChainGeom g;
  g.imgs = imgs;
  g.buf_bytes = buffer_bytes(C, p.H, p.W, imgs);
  g.plane = plane_bytes(p.H, p.W, imgs);
  g.sign_bytes = sign_bytes(C, p.H, p.W, imgs);
  g.fold_at = norm_fold_at(C, p.H, p.W, imgs);
  g.dP = make_divisor1(g.plane / 16);
  g.dQ = make_divisor1(p.W + 1);
  g.dH1 = make_divisor1(p.H + 1);
  g.dW = make_divisor1(p.W);
  g.dH = make_divisor1(p.H);
  const int wgs = cdiv(p.Nimg, imgs), smem = NORM ? norm_lds_bytes(C, p.H, p.W, imgs) : lds_bytes(C, p.H, p.W, imgs);
  const int runs = cdiv(cdiv(imgs * p.H * p.W, 16), wave_rows(C));
#define DDS_CHAIN_CASE(C, RUNS) \
  case (C) * 8 + (RUNS) - 1: launch_inst<C, RUNS, NORM>(p, g, n, wgs, smem, s); break;
  switch (C * 8 + runs - 1) {
    DDS_CHAIN_CASE(16, 1) DDS_CHAIN_CASE(16, 2) DDS_CHAIN_CASE(16, 3) DDS_CHAIN_CASE(16, 4)
    DDS_CHAIN_CASE(16, 5) DDS_CHAIN_CASE(16, 6) DDS_CHAIN_CASE(16, 7) DDS_CHAIN_CASE(16, 8)
    DDS_CHAIN_CASE(32, 1) DDS_CHAIN_CASE(32, 2) DDS_CHAIN_CASE(32, 3) DDS_CHAIN_CASE(32, 4)
    DDS_CHAIN_CASE(32, 5) DDS_CHAIN_CASE(32, 6) DDS_CHAIN_CASE(32, 7) DDS_CHAIN_CASE(32, 8)
    DDS_CHAIN_CASE(64, 1) DDS_CHAIN_CASE(64, 2) DDS_CHAIN_CASE(64, 3) DDS_CHAIN_CASE(64, 4)
  }
#undef DDS_CHAIN_CASE
}

void launch_conv_chain(int C, const ChainParams& p, hipStream_t s) {
  const int imgs = images_of(C, p.H, p.W, p.Nimg, p.nrep > 1 ? p.nrep : 1);
  if (imgs == 0) launch_wide_chain(C, p, s);
  else launch_narrow<false>(C, imgs, p, BnParams{}, s);
}

// Images of a workgroup that normalises, all of one data-group; 0: a launch each. Where two workgroups share a CU, one's copies run beside the
// other's products. Larger ones have to be done in one round, and to fill it unless an image is small. us per step of a net of five normalised layers of 2
// groups of 97 (4 of 194), streamed apart / here: 16 channels at 32 x 32 243 / 219 (529 / 498), at 16 x 16 206 / 166 (260 / 231), 32 channels at 16 x 16
// 227 / 197 (355 / 329), 64 channels at 8 x 8 223 / 196 (304 / 306), at 4 x 4 215 / 179 (225 / 238: 388 workgroups; 4 groups of 256, 256 of them:
// 214 / 194). One workgroup a CU, 4 groups of 16, 64 and 194: 32 channels at 28 x 28 222 / 237, 357 / 318, 748 / 833; 64 channels at 14 x 14 226 / 230, 301 / 276, -.
static int norm_images_of(int C, int H, int W, int Nimg, int W_groups) {
  if ((C != 16 && C != 32 && C != 64) || H < 1 || W < 1 || Nimg < 1 || W_groups < 1 || Nimg % W_groups != 0 || (long long)H * W > 4096) return 0;
  auto runs = [&](int imgs) { return cdiv(cdiv(imgs * H * W, 16), wave_rows(C)); };
  auto fits = [&](int imgs, int room) { return norm_lds_bytes(C, H, W, imgs) <= room && runs(imgs) <= most_runs(C) && Nimg / W_groups % imgs == 0; };
  const bool two = fits(1, 80 * 1024);
  const int room = two ? 80 * 1024 : 160 * 1024, enough = two ? 512 : 256;
  if (!fits(1, room)) return 0;
  int imgs = 1;
  while (cdiv(Nimg, imgs) > enough && imgs < 8 && fits(2 * imgs, room)) imgs *= 2;
  const int wgs = cdiv(Nimg, imgs);
  if (!two && (wgs > 256 || (runs(1) > 2 && wgs < 192))) return 0;
  return imgs;
}
bool norm_conv_fits(int C, int H, int W, int Nimg, int W_groups) { return norm_images_of(C, H, W, Nimg, W_groups) > 0; }
void launch_norm_conv(int C, const ChainParams& p, const BnParams& n, hipStream_t s) {
  launch_narrow<true>(C, norm_images_of(C, p.H, p.W, p.Nimg, n.W), p, n, s);
}

}  // namespace dds
