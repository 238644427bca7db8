// Launch interface of the learned-start kernels: 3x3 convolutions and their
// gradients (conv.hip); the complex MSE head, Adam, the network input map built
// from measured intensities, and whole-object restriction / prolongation (cnn.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cnn {

// Activations of the hidden layers are channels-last, [B][H][W][32]; the network's
// input, output and output gradient are planes, [B][c][H][W].

// Compute copies of the weights.  Square (32 -> 32) layers: fwd, FWD_VECS float2 each
// (the products' operands in lane order, see prep_kernel), and frag, FRAG_VECS vectors of bf16 parts each
// for backward-data; the first layer keeps its order (first[32][cin][9]); the head becomes
// head[32][9][2] and, transposed and flipped, head_t[32][2][9].  With bf16 the
// copies hold the weights rounded to bf16.  *wbad: set where a square layer's weight is not finite (zero before the launch).
constexpr int FWD_VECS = 4 * 9 * 2 * 64, FRAG_VECS = 18 * 3 * 64;
struct PrepArgs {
  const float* p;               // parameter vector
  int64_t off_sq[3], off_first, off_head;   // offsets of the layers' weights
  int cin;
  bool bf16;
  float2* fwd;                  // [3][FWD_VECS]
  uint4* frag;                  // [3][FRAG_VECS]
  float *first, *head, *head_t;
  int* wbad;
};
hipError_t launch_prep(const PrepArgs& a, hipStream_t s);

// Square layer, forward: out = relu(conv3x3(in) + bias) with zero padding 1 (H, W: the
// output's size; up: in has half of it and is read through nearest 2x upsampling).
hipError_t launch_conv32(bool up, const float* in, const float2* w, const float* bias, float* out, int batch, int H,
                         int W, hipStream_t s);
// Square layer, backward-data of in (H x W): zero where omask <= 0; up: the sum of each
// 2 x 2 block, out and omask of half the size.  w: the layer's weights as stored.
hipError_t launch_conv32_backward(bool up, bool bf16, const float* in, const uint4* frag, const float* w, float* out,
                                  const float* omask, const int* wbad, int batch, int H, int W, hipStream_t s);
// First layer (planes in; + bias, ReLU), head (planes out; + bias) and the head's
// backward-data (planes in; zero where omask <= 0).
hipError_t launch_conv_first(int ci, const float* in, const float* w, const float* bias, float* out, int batch, int H,
                             int W, hipStream_t s);
hipError_t launch_conv_head(const float* in, const float* w, const float* bias, float* out, int batch, int H, int W,
                            hipStream_t s);
hipError_t launch_conv_head_backward(const float* dy, const float* w, float* out, const float* omask, int batch,
                                     int H, int W, hipStream_t s);

// Weight and bias gradients of a layer (w[co][ci][9], then b[co]) from its input and its
// output gradient, through at most WGRAD_MAX_WORKGROUPS rows of partial sums in `part`.
constexpr int WGRAD_MAX_WORKGROUPS = 512;
constexpr int SQ_ROW = 9 * 32 * 32 + 32;   // floats per row of a square layer
constexpr int thin_row(int cn, bool head) { return (9 * cn + 31) / 32 * 1024 + (head ? 0 : 32); }
hipError_t launch_wgrad32(bool up, const float* in, const float* dout, float* part, float* grad, int batch, int H,
                          int W, hipStream_t s);
hipError_t launch_wgrad_first(int ci, const float* in, const float* dout, float* part, float* grad, int batch, int H,
                              int W, hipStream_t s);
hipError_t launch_wgrad_head(const float* in, const float* dy, float* part, float* grad, int batch, int H, int W,
                             hipStream_t s);

// Masked complex MSE of exp(y0 + i y1) against target; dy gets the gradient.
// y, dy: [B][2][HW]; target: [B][HW] complex; mask: [HW].  Per-block FP64 loss
// partials go to part (n_blocks returned by cmse_blocks).  With rot non-null
// each sample's prediction is first rotated by its best global phase
// (rot[b] = ip / |ip|, ip = sum mask conj(pred) t, partials in ip_part
// [B][cmse_ip_blocks(hw)]).  A mask that is not finite and >= 0 (out->bad) or all zero
// (out->msum = 0) leaves dy alone.
struct CmseHead {
  double msum;   // the mask's sum, 0 where it is refused
  int bad;
};
struct CmseResult {
  double loss, msum;
  int bad;
};
int cmse_blocks(int batch, int hw);
int cmse_ip_blocks(int hw);
// out: memory the host reads after the stream is synchronised
hipError_t launch_cmse(const float* y, const float2* target, const float* mask, float2* rot, double2* ip_part,
                       float* dy, double* part, int batch, int hw, CmseHead* head, CmseResult* out, hipStream_t s);

// Adam with bias corrections c1 = 1/(1-b1^t), c2 = 1/(1-b2^t); reset: moments to zero.  Both
// clear *wbad (see PrepArgs) for the weight preparation that follows.
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, int* wbad, hipStream_t s);
hipError_t launch_adam_reset(float* m, float* v, int64_t n, int* wbad, hipStream_t s);

// Network input map.  a2[i] = |Q_i|^2, out = ||Q||_2.
hipError_t launch_probe_norm(const double2* q, int m, double* out, double* a2, hipStream_t s);
// stats[k] = (mean sqrt(d_k) / ||Q||_2, row and column frequency centres of mass of d_k, 0) from
// sqrt(d) in the kernel order of plan (m, rb); the sums do not depend on rb.
hipError_t launch_position_stats(const float* sqrtd, int n_pos, int m, int rb, const double* qnorm, double4* stats,
                                 hipStream_t s);
// fine[ch][r][c] = sum_k |Q(p-o_k)|^2 stats[k][ch] / sum_k |Q(p-o_k)|^2 over the positions
// in the pixel's tile list (0 where uncovered), ch < 3.
hipError_t launch_map_fine(const double4* stats, const double* a2, int m, const int* tile_ptr, const int4* tile_ent,
                           int tiles_x, int tiles_y, int tile_w, int tile_h, int nr, int nc, double* fine,
                           hipStream_t s);
// out[ch][i][j] = mean of fine[ch] over the fr x fc block (i, j).
hipError_t launch_pool(const double* fine, int nr, int nc, int fr, int fc, float* out, hipStream_t s);
// out = the S x S phase whose gradient is (sy * gy, sx * gx) in the least-squares
// (periodic, spectral) sense, mean 0; S <= 64.  scratch: S * S values.
constexpr int PHASE_MAX_SIDE = 64;
hipError_t launch_integrate_phase(const float* gy, const float* gx, int S, double sy, double sx, double2* scratch,
                                  float* out, hipStream_t s);

// z[r][c] = coarse[r / f][c / f]; format 0 complex64, 1 complex128, 2 planes
// (log-amplitude, phase) float [2][sr][sc].
hipError_t launch_prolong_object(const void* coarse, int format, int sr, int sc, int f, float2* z, int nr, int nc,
                                 hipStream_t s);
// out[i][j] = mean of z over the f x f block (i, j) (complex64 in and out).
hipError_t launch_restrict_object(const float2* z, int nr, int nc, int f, float2* out, hipStream_t s);

}  // namespace cnn
