// Launch interface between the host engine and the HIP kernels (gfx950 only).
// Internal to the library: plain structs of device pointers and sizes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dds {

enum DType : int { DT_F32 = 0, DT_BF16 = 1 };

inline int dtype_size(int dt) { return dt == DT_F32 ? 4 : 2; }
// channels per 16-byte chunk; every tensor's channel stride is a multiple of this
inline int dtype_ce(int dt) { return dt == DT_F32 ? 4 : 8; }

// Implicit-GEMM convolution / linear, forward or input-gradient (dgrad) form.
//   y[m, n] = epilogue( sum_{tap, c} gather(x; m, tap)[c] * w[n, tap, c] )
// forward : m = (img, ho, wo), gathers x at (ho*stride - pad + r, wo*stride - pad + s)
// dgrad   : m = (img, h, w) of the conv input, x is the output gradient, gathers at
//           ((h + pad - r)/stride, (w + pad - s)/stride) when divisible, w is the
//           transposed weight snapshot [cin][tap][cout_padded]
// epilogue: v = alpha * (acc + bias[n]); v += res[m, n]; relu; v = mask[m, n] > 0 ? v : 0
// Size of the block of zeros every launch may read padding from: at least one pixel row
// (all channels of one pixel) of any tensor the asynchronous kernels accept.
constexpr int kZeroBytes = 16384;

struct ConvParams {
  const void* x;
  const void* w;
  void* y;
  const float* bias;  // fp32 [Nout] or null
  const void* res;    // same layout as y (dtype T) or null
  const void* mask;   // same layout as y (dtype T) or null
  // Sign planes of ReLU outputs: [pixel][ldy / 8] bytes, bit c % 8 of byte c / 8 set iff channel c
  // of the stored tensor is > 0 (needs ldy % 8 == 0). bits_out: written with y by a forward launch
  // with relu. maskbits: what a dgrad launch multiplies by instead of reading `mask` (the full tensor).
  void* bits_out;
  const void* maskbits;
  // dgrad of a stride-2 layer only: gradient of a 1x1 stride-2 pad-0 shortcut that shares this
  // layer's input, folded in as extra reduction steps. x2: [Nimg][H][W][Cx2] (same pixel grid as x),
  // w2: [Nout][Cx2]; output pixel (oh, ow) with oh, ow even receives sum_k x2[oh/2, ow/2, k] * w2[n][k].
  const void* x2;
  const void* w2;
  int Cx2;
  const void* zeros;  // kZeroBytes zero bytes (source of padding rows for LDS fills)
  int Nimg, H, W, Cx; // gathered tensor: NHWC, channel stride Cx (= GEMM-K per tap)
  int Ho, Wo;         // pixel grid of y; M = Nimg*Ho*Wo
  int M;
  int Nout;           // valid rows of w
  int ldy;            // channel stride of y / res / mask
  int R, S, stride, pad;
  int Ktot;           // R*S*Cx
  float alpha;
  int relu;
  int out_f32;        // y is fp32 regardless of T (logits)
  int dgrad;
  // Data-groups with weights of their own (general mixing matrix): the Nimg images are nrep equal
  // groups of consecutive images and group r multiplies by w + r*w_rep bytes, adds bias + r*bias_rep
  // floats and (folded shortcut) uses w2 + r*w2_rep bytes. nrep <= 1: one weight set for all images.
  int nrep;
  long long w_rep, w2_rep, bias_rep;
};

// A run of 3x3 stride-1 pad-1 layers of C channels in and out, bf16 (chain.hip): layer i + 1 reads what layer i writes. Epilogue of a layer:
// v = alpha * (acc + bias[n]); v += what the layer before read (layer 0: res), if add; relu; v = maskbits ? v : 0. Weights as in ConvParams.
constexpr int kChainMax = 16;
struct ChainLayer {
  const void* w;
  const float* bias;     // or null
  void* y;
  void* bits_out;        // sign plane of y or null
  const void* maskbits;  // sign plane or null
  float alpha;
  int relu, add;
};
struct ChainParams {
  const void* x;    // input of layer 0
  const void* res;  // what layer 0 adds, or null
  const void* zeros;
  int Nimg, H, W, n, dgrad;
  int nrep;         // data-groups with weights of their own, as in ConvParams
  long long w_rep, bias_rep;
  ChainLayer layer[kChainMax];
};

// Weight-gradient GEMM with split reduction:
//   partial[z][m*NK + n] = alpha * sum_{p in split z} dy[p, m] * gather(x; p, n)
//   partial[z][Mout*NK + m] = alpha * sum_p dy[p, m]                (bias gradient)
// m = output channel, n = (tap, c), p = output pixel (img, ho, wo).
struct WgradParams {
  const void* dy;   // [P][ldy]
  const void* x;    // [Nimg][H][W][Cx]
  float* partial;   // [nsplit][Pl]
  const void* zeros; // kZeroBytes zero bytes
  int Nimg, H, W, Cx, Ho, Wo;
  int Mout;         // real output channels
  int ldy;
  int R, S, stride, pad;
  int NK;           // R*S*Cx
  int P;            // Nimg*Ho*Wo
  int pix_per_split; // wgrad_gemm_kernel: pixels per split (P / nsplit, splits are equal)
  int nsplit;
  int nrep;          // data-groups: equal runs of consecutive images; nsplit is a multiple of it and no split
                     // holds pixels of two data-groups (the asynchronous kernels deal each group's tiles to its
                     // nsplit / nrep splits as evenly as whole tiles allow). 1: only the sum over all images is asked for
  long long Pl;     // floats between consecutive splits (>= Mout*NK + Mout)
  float alpha;
};

// Training-mode batch normalisation of a [W * rows_per_rep][ld] tensor, statistics per data-group.
//   forward : y = relu?( alpha * (gamma * (x - mean) * rstd + beta) + res ), stats <- mean, rstd, gamma
//   backward: dgamma / dbeta partial rows (one per (data-group, split)), dx from dy, x and the saved stats
constexpr int kBnCoefRows = 5;
struct BnPlan {
  int nsums, nsplit;
  long long rows_per_sum, rows_per_split;
  bool fold;
};
BnPlan bn_plan(int W, long long rows_per_rep, int ld, int es);
constexpr int kBnFoldLd = 64, kBnFoldSums = 2048;

struct BnParams {
  const void* x;      // input of the normalisation (the convolution output), dtype T
  void* y;            // forward output, dtype T
  const void* res;    // added after the normalisation (same layout as y) or null
  void* bits_out;     // sign plane of y ([row][ld / 8] bytes) or null
  const void* dy;     // backward: gradient with respect to y (already masked by y > 0 where relu)
  void* dx;           // backward: gradient with respect to x
  const float* gamma; // fp32 master: gamma[c * gstride]
  const float* beta;  // beta[c]
  long long rep_stride;  // floats between the parameters of consecutive data-groups (0: shared)
  int gstride;
  float* stats;       // [W][3][ld]: mean, rstd, gamma of this mini-batch
  double* scratch;    // [W][nsums][ld][2] per-split sums (forward: x, x^2; backward: g, g * xhat)
  float* coef;        // [W][kBnCoefRows][ld] per-channel factors of the streaming kernel that follows
  float* partial;     // backward: [W][pstride] parameter-gradient rows, one per data-group
  long long pstride;
  int W, C, ld;
  int nsums, nsplit;  // row splits of a data-group: of the kernels that sum, of those that stream
  long long rows_per_rep, rows_per_sum, rows_per_split;
  bool fold;          // the streaming kernels join the splits' sums themselves
  bool streamed_later;  // only the sums are launched: the streaming rides in the convolution that follows (launch_norm_conv)
  float eps, alpha;
  int relu;
};

struct IngestParams {
  const float* x[32];
  const int32_t* y[32];
  void* dst;        // [W*B][H][W][Cpad] dtype T
  int32_t* labels;  // [W*B]
  int W, B, C, HW, Cpad;
};

// One entry per parameter tensor block of a module (weights followed by bias).
struct UpdateDesc {
  float* master;        // [n] fp32, internal layout
  float* momentum;      // [n] or null
  const float* partial; // [nsplit][n]
  void* work;           // compute-precision copy [n] or null (fp32 path uses master)
  void* stash;          // transposed snapshots [slot][Cin][RS][Coutpad] or null
  long long stash_slot_elems;
  long long n;          // Cout*RS*Cinpad + Cout
  long long pstride;    // floats between consecutive splits of `partial` (n rounded up to 4)
  int nsplit;
  int Cout, RS, Cinpad, Cin, Coutpad;
};

// Returns the class of dds_profile_read: 1 = the kernels made for 3x3 stride-1 layers (conv3x3_dma, conv_direct), 0 = those that
// take any layer (conv_gather, conv_gemm, linear) and the forward pass of a stem (conv_direct, 8 channels).
int launch_conv(int dt, const ConvParams& p, hipStream_t s);
// plain products of few rows (linear.hip); false: not taken, nothing launched
bool launch_linear(int dt, const ConvParams& p, hipStream_t s);
// bf16 3x3 stride-1 layers with 16-channel rows, stems (narrow.hip); false: not taken, nothing launched
bool launch_conv_narrow(const ConvParams& p, hipStream_t s);
// Fewest layers that are faster in one launch than in one each; 0: no number is, or the kernel does not take them.
int conv_chain_least(int C, int H, int W, int Nimg, int nrep);
void launch_conv_chain(int C, const ChainParams& p, hipStream_t s);
// A batch normalisation whose sums are there (n.fold) and a single such layer that reads what it makes, in one launch; forward: n.x, n.res -> n.y
// -> layer; input gradient: n.dy, n.x -> n.dx -> layer (p.res: what the layer adds). norm_conv_fits: is there such a kernel
bool norm_conv_fits(int C, int H, int W, int Nimg, int W_groups);
void launch_norm_conv(int C, const ChainParams& p, const BnParams& n, hipStream_t s);
// n layers of one key (wgrad_work), or one of any kind. Returns 1 if wgrad_tiles or wgrad_slim took them, whose 3x3 and stride-2
// layers have a class of their own, 0 if wgrad_gemm or wgrad_f32 did; -1, nothing launched, if their splits fit none of them.
int launch_wgrad(int dt, const WgradParams* p, int n, hipStream_t s);
// Layers of one key, if it is not 0, may share a launch; a split of theirs is at least one of `tiles` tiles of a data-group,
// and each is walked by `blocks` workgroups. shape: every field that describes the layer (Nimg, H, W, Cx, Ho, Wo, Mout, ldy,
// R, S, stride, pad, NK, P, nrep, zeros non-null); nsplit, pix_per_split and the other pointers are ignored.
struct WgradWork { int key, blocks, tiles; };
WgradWork wgrad_work(int dt, const WgradParams& shape);
// Layers that one weight-gradient launch can take at most.
constexpr int kWgradGroupMax = 16;
// bf16 3x3 stride-1 layers of 8, 16 or 32 input channels (narrow.hip): tiles of one of nrep data-groups (0: not such a layer)
// with the kernel's variant, and the launch for n layers of one variant (false: not taken, nothing launched)
int wgrad_slim_tiles(const WgradParams& shape, int nrep, int* variant);
bool launch_wgrad_slim(const WgradParams* p, int n, hipStream_t s);
// Chooses the split counts of the pixel reductions of layers that share a launch (n > 1: one key): multiples of nrep, so that no
// split mixes two data-groups. one_module: no other module's launches share the chip.
void wgrad_choose_splits(int dt, const WgradParams* shapes, int n, bool one_module, int* nsplit);

void launch_ingest(int dt, const IngestParams& p, hipStream_t s);
void launch_maxpool_fwd(int dt, const void* x, void* y, int N, int H, int W, int C, hipStream_t s);
void launch_maxpool_bwd(int dt, const void* dy, const void* x, void* dx, int N, int H, int W, int C,
                        int relu_mask, hipStream_t s);
void launch_gap_fwd(int dt, const void* x, void* y, int N, int HW, int C, hipStream_t s);
void launch_gap_bwd(int dt, const void* dy, const void* x, void* dx, int N, int HW, int C, int relu_mask,
                    hipStream_t s);
// logits fp32 [W*B][ldl]; dlogits dtype T [W*B][ldg] (may be null); loss [W] (may be null)
void launch_softmax_ce(int dt, const float* logits, const int32_t* labels, void* dlogits, float* loss,
                       int W, int B, int classes, int ldl, int ldg, hipStream_t s);
// Elements of a parameter block that one workgroup of the update kernel owns: the fewer, the more splits have to be
// summed for each, so that a launch always has thousands of partial rows in flight (see update_kernel).
// fp32 nets keep one size and with it one order of the sum for every split count (on the exact-mean path: gossip_elems).
__host__ __device__ inline int update_elems(int dt, int nsplit) {
  return dt == DT_F32 ? 256 : nsplit <= 8 ? 1024 : nsplit <= 64 ? 256 : 64;
}
// Input channels of a tile of the update kernel, a power of two (8 to 32; a tile has at least two output channels).
__host__ __device__ inline int update_width(int Cinpad) { return Cinpad <= 8 ? 8 : Cinpad <= 16 ? 16 : 32; }
// Workgroups of the update kernel for one layer.
inline int update_tiles(int dt, int nsplit, int Cout, int RS, int Cinpad) {
  const int e = update_elems(dt, nsplit), kc = update_width(Cinpad), kk = e / kc;
  return RS * ((Cout + kk - 1) / kk) * ((Cinpad + kc - 1) / kc) + (Cout + e - 1) / e;
}
// update: g = (1/W) sum over splits, momentum, SGD on the fp32 master, recast into `work`, transposed into snapshot `slot`.
// tile_map: device array of (descriptor, tile) pairs, one per workgroup.
void launch_update(int dt, const UpdateDesc* descs_dev, const int* tile_map_dev, int total_tiles, int slot, int W,
                   float lr, float mu, hipStream_t s);
// The other kernels' block_map: device array of (descriptor, block) pairs, one per 1024 elements.
// General mixing matrix (W weight copies, rep_stride elements apart; a descriptor's nsplit = splits per data-group):
// u_r = w_r - lr*direction_r from data-group r's own splits, then w_s = sum_r P[s][r] u_r into master
// and `work`. descs / range_map: the entries of data-group 0, one per workgroup of gossip_elems(nsplit) elements.
// P: device, W x W row-major.
// (In fp32 as well, so that there the order of a sum depends on the split count.)
__host__ __device__ inline int gossip_elems(int nsplit) { return nsplit >= 32 ? 32 : nsplit >= 8 ? 64 : 256; }
void launch_gossip_update(int dt, const UpdateDesc* descs_dev, const int* range_map_dev, int total_ranges,
                          const float* P_dev, int W, long long rep_stride, float lr, float mu, hipStream_t s);
// Squared distances to the data-group mean: out[(2*b + part) * W + s] for workgroup b of the
// update block map of data-group 0 (1024 elements of one layer each); part 0 = weight, 1 = bias; fp64.
void launch_consensus(const UpdateDesc* descs_dev, const int* block_map_dev, int total_blocks, int W,
                      long long rep_stride, double* out_dev, hipStream_t s);
// work <- master
void launch_recast(int dt, const UpdateDesc* descs_dev, const int* block_map_dev, int total_blocks,
                   hipStream_t s);
// stash[slot] <- transpose(master); block_map enumerates blocks of Cin*RS*Coutpad elements
void launch_stash(int dt, const UpdateDesc* descs_dev, const int* block_map_dev, int total_blocks, int slot,
                  hipStream_t s);
// three kernels each: per-split sums, their fold per data-group and channel, the streaming pass
void launch_bn_forward(int dt, const BnParams& p, hipStream_t s);
void launch_bn_backward(int dt, const BnParams& p, hipStream_t s);
// canonical [Cout][Cin][R][S] (+bias) <-> internal [Cout][RS][Cinpad] (+bias)
void launch_param_permute(const float* canon, float* internal, int Cout, int Cin, int RS, int Cinpad,
                          int to_internal, hipStream_t s);
void launch_fill_zero(void* p, size_t bytes, hipStream_t s);

}  // namespace dds
