// What the kernels that stream a batch normalisation share: the join of its splits' sums and the per-channel factors (norm.hip has the formulas).
#pragma once
#include "kernels.h"

namespace dds {
namespace {

// The sums a, b of channel c of data-group `rep` -> the factors of the streaming kernel, coef[row * stride]; `leave`: and what
// outlives it. Forward (sum x, sum x^2): mean, rstd (and the gamma in use) into `stats`; coef rows: scale, shift. Backward (sum g,
// sum g*xhat): dbeta, dgamma in fp32 into row `rep` of the parameter-gradient partials (dgamma[c] at c * gstride,
// dbeta[c] at C * gstride + c: the layout of a 1x1 "convolution" with one input channel, so that the update kernels
// treat gamma / beta like any other layer with one split per data-group); coef rows: mean, rstd, and k0, k1, k2 of
// dx = k0 * dy - k1 - xhat * k2. Channels past C (row padding) get zeros.
// What they need beside the sums is asked for (channel_inputs) before those are there.
struct ChannelInputs { float mean, rstd, gamma, beta; };
template <bool BWD>
__device__ __forceinline__ ChannelInputs channel_inputs(const BnParams& p, int rep, int c) {
  ChannelInputs in{};
  if (BWD) {
    const float* st = p.stats + (size_t)rep * 3 * p.ld + c;
    in.mean = st[0];
    in.rstd = st[p.ld];
    in.gamma = st[2 * p.ld];
  } else {
    const int k = c < p.C ? c : p.C - 1;
    in.gamma = p.gamma[(size_t)rep * p.rep_stride + (size_t)k * p.gstride];
    in.beta = p.beta[(size_t)rep * p.rep_stride + k];
  }
  return in;
}
template <bool BWD>
__device__ __forceinline__ void channel_factors(const BnParams& p, const ChannelInputs& in, int rep, int c, double a, double b, bool leave, float* coef, int stride) {
  const double m = (double)p.rows_per_rep;
  const bool real = c < p.C;
  if (BWD) {
    const float gr = in.gamma * in.rstd;
    if (real && leave) {
      float* row = p.partial + (size_t)rep * p.pstride;
      row[(size_t)c * p.gstride] = (float)b;
      row[(size_t)p.C * p.gstride + c] = (float)a;
    }
    // dx = gr * (alpha*dy - db/m - xhat*dg/m), db and dg already carry alpha
    coef[0] = real ? in.mean : 0.f;
    coef[stride] = real ? in.rstd : 0.f;
    coef[2 * stride] = real ? gr * p.alpha : 0.f;
    coef[3 * stride] = real ? gr * (float)(a / m) : 0.f;
    coef[4 * stride] = real ? gr * (float)(b / m) : 0.f;
  } else {
    const double mean = a / m;
    double var = b / m - mean * mean;
    var = var > 0.0 ? var : 0.0;
    const float meanf = (float)mean, rstd = (float)(1.0 / sqrt(var + (double)p.eps));
    const float g = real ? in.gamma : 0.f, beta = real ? in.beta : 0.f;
    if (leave) {
      float* st = p.stats + (size_t)rep * 3 * p.ld;
      st[c] = meanf;
      st[p.ld + c] = rstd;
      st[2 * p.ld + c] = g;
    }
    coef[0] = p.alpha * g * rstd;
    coef[stride] = p.alpha * (beta - meanf * g * rstd);
  }
}

// The per-channel factors from the splits' sums, by every workgroup of a streaming kernel, for rows of at most kBnFoldLd channels (bn_plan):
// THREADS / C' split lanes x C' channels, C' = ld rounded up to a power of two; a lane has at most kBnFoldSums / THREADS splits
// to add (eight of 256 threads). request() asks for everything that comes from memory, ahead of the first rows (loads return in order); finish()
// leaves the factors at cf[row * PITCH + c] in LDS, and the first workgroup of a data-group what outlives the kernel.
template <bool BWD, int THREADS, int PITCH = kBnFoldLd>  // PITCH: at least the row's channels
struct SplitFold {
  static constexpr int V = kBnFoldSums / THREADS, WAVES = THREADS / 64, kDoubles = 2 * WAVES * PITCH;
  int c, clog;
  double2 v[V];
  ChannelInputs in;
  __device__ __forceinline__ void request(const BnParams& p, int rep) {
    clog = p.ld > 32 ? 6 : p.ld > 16 ? 5 : p.ld > 8 ? 4 : 3;
    c = threadIdx.x & ((1 << clog) - 1);
    const int j = threadIdx.x >> clog, cc = min(c, p.ld - 1);
    const double* row = p.scratch + ((size_t)rep * p.nsums * p.ld + cc) * 2;
#pragma unroll
    for (int u = 0; u < V; ++u) v[u] = *(const double2*)(row + (size_t)min(j + u * (THREADS >> clog), p.nsums - 1) * p.ld * 2);
    in = channel_inputs<BWD>(p, rep, min((int)threadIdx.x, p.ld - 1));
  }
  __device__ __forceinline__ void finish(const BnParams& p, int rep, bool leave, double* red, float* cf) {  // red: kDoubles
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const bool ok = (int)(threadIdx.x >> clog) + u * (THREADS >> clog) < p.nsums;
      a += ok ? v[u].x : 0.0;
      b += ok ? v[u].y : 0.0;
    }
    for (int d = 1 << clog; d < 64; d <<= 1) {
      a += __shfl_xor(a, d, 64);
      b += __shfl_xor(b, d, 64);
    }
    if ((int)(threadIdx.x & 63) < 1 << clog) {
      red[(threadIdx.x >> 6) * PITCH + c] = a;
      red[(WAVES + (threadIdx.x >> 6)) * PITCH + c] = b;
    }
    __syncthreads();
    if ((int)threadIdx.x < p.ld) {
      a = b = 0.0;
      for (int j = 0; j < WAVES; ++j) { a += red[j * PITCH + threadIdx.x]; b += red[(WAVES + j) * PITCH + threadIdx.x]; }
      channel_factors<BWD>(p, in, rep, threadIdx.x, a, b, leave, cf + threadIdx.x, PITCH);
    }
    __syncthreads();
  }
};

}  // namespace
}  // namespace dds
