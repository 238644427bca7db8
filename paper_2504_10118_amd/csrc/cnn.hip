// Learned-start kernels for gfx950 apart from the convolutions: the complex MSE
// head, Adam, the network input map computed from the measured intensities,
// and whole-object restriction / prolongation (2x2 average pooling and 2x2
// replication applied repeatedly, i.e. f x f block means and copies).
//
// All reductions run in a fixed order, so every result is bitwise
// reproducible run to run.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "cnn.h"

namespace cnn {

namespace {

// ---------------------------------------------------------------------------
// Complex MSE head
// ---------------------------------------------------------------------------
constexpr int CMSE_THREADS = 256;

__device__ __forceinline__ float2 pred_of(const float* __restrict__ y, size_t b, int p, int hw) {
  const float la = y[(b * 2) * hw + p], ph = y[(b * 2 + 1) * hw + p];
  float sn, cs;
  sincosf(ph, &sn, &cs);
  const float amp = expf(la);
  return make_float2(amp * cs, amp * sn);
}

// per-block partial sums of mask * conj(pred) * t for each sample: part[b][blockIdx.x]
__global__ __launch_bounds__(CMSE_THREADS) void cmse_ip_kernel(const float* __restrict__ y,
                                                               const float2* __restrict__ tgt,
                                                               const float* __restrict__ mask,
                                                               double2* __restrict__ part, int hw) {
  __shared__ double rr[CMSE_THREADS], ri[CMSE_THREADS];
  const int b = blockIdx.y;
  const int p = blockIdx.x * CMSE_THREADS + threadIdx.x;
  double a = 0.0, c = 0.0;
  if (p < hw) {
    const float2 pr = pred_of(y, b, p, hw);
    const float2 t = tgt[(size_t)b * hw + p];
    const double mk = mask[p];
    a = mk * ((double)pr.x * t.x + (double)pr.y * t.y);
    c = mk * ((double)pr.x * t.y - (double)pr.y * t.x);
  }
  rr[threadIdx.x] = a;
  ri[threadIdx.x] = c;
  __syncthreads();
  for (int s = CMSE_THREADS / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      rr[threadIdx.x] += rr[threadIdx.x + s];
      ri[threadIdx.x] += ri[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(size_t)b * gridDim.x + blockIdx.x] = make_double2(rr[0], ri[0]);
}

// Workgroup 0: the mask's sum, and whether all its values are finite and >= 0 (a mask
// that is not, or whose sum is 0, gives head->msum = 0).  Workgroup b + 1: rot[b] = ip / |ip|
// (1 where ip = 0), ip = sum of the sample's partials in order.
__global__ __launch_bounds__(256) void cmse_head_kernel(const float* __restrict__ mask, int hw,
                                                        const double2* __restrict__ part, int nblk,
                                                        float2* __restrict__ rot, CmseHead* __restrict__ head) {
  __shared__ double rr[256], ri[256];
  double a = 0.0, c = 0.0;
  if (blockIdx.x == 0) {
#pragma unroll 8
    for (int i = threadIdx.x; i < hw; i += 256) {
      const float v = mask[i];
      a += (double)v;
      c += (v >= 0.0f && v <= 3.402823466e38f) ? 0.0 : 1.0;
    }
  } else {
    const size_t b = blockIdx.x - 1;
    for (int i = threadIdx.x; i < nblk; i += 256) {
      a += part[b * nblk + i].x;
      c += part[b * nblk + i].y;
    }
  }
  rr[threadIdx.x] = a;
  ri[threadIdx.x] = c;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      rr[threadIdx.x] += rr[threadIdx.x + s];
      ri[threadIdx.x] += ri[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x) return;
  if (blockIdx.x == 0) {
    head->bad = ri[0] > 0.0 ? 1 : 0;
    head->msum = (ri[0] > 0.0 || !(rr[0] > 0.0)) ? 0.0 : rr[0];
  } else {
    const double n = sqrt(rr[0] * rr[0] + ri[0] * ri[0]);
    rot[blockIdx.x - 1] = n > 0.0 ? make_float2((float)(rr[0] / n), (float)(ri[0] / n)) : make_float2(1.0f, 0.0f);
  }
}

// dy is left as it was where the mask is refused (head->msum = 0)
__global__ __launch_bounds__(CMSE_THREADS) void cmse_kernel(const float* __restrict__ y,
                                                            const float2* __restrict__ tgt,
                                                            const float* __restrict__ mask,
                                                            const float2* __restrict__ rot, float* __restrict__ dy,
                                                            double* __restrict__ part, int batch, int hw,
                                                            const CmseHead* __restrict__ head) {
  __shared__ double red[CMSE_THREADS];
  const size_t i = (size_t)blockIdx.x * CMSE_THREADS + threadIdx.x;
  const double msum = head->msum;
  const float inv_norm = (float)(1.0 / ((double)batch * msum));
  double l = 0.0;
  if (i < (size_t)batch * hw && msum > 0.0) {
    const size_t b = i / hw;
    const int p = (int)(i - b * hw);
    float2 pv = pred_of(y, b, p, hw);
    if (rot) {
      const float2 r = rot[b];
      pv = make_float2(pv.x * r.x - pv.y * r.y, pv.x * r.y + pv.y * r.x);
    }
    const float pr = pv.x, pi = pv.y;
    const float2 t = tgt[i];
    const float rr = pr - t.x, ri = pi - t.y;
    const float mk = mask[p];
    l = (double)mk * ((double)rr * rr + (double)ri * ri);
    // g = conj(r) * pred
    const float gr = rr * pr + ri * pi, gi = rr * pi - ri * pr;
    dy[(b * 2) * hw + p] = 2.0f * mk * gr * inv_norm;
    dy[(b * 2 + 1) * hw + p] = -2.0f * mk * gi * inv_norm;
  }
  red[threadIdx.x] = l;
  __syncthreads();
  for (int s = CMSE_THREADS / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// the loss, and what the host has to know of the mask, into host memory the GPU writes
__global__ __launch_bounds__(1024) void cmse_loss_kernel(const double* __restrict__ x, int n,
                                                         const CmseHead* __restrict__ head, int batch,
                                                         CmseResult* __restrict__ out) {
  __shared__ double red[1024];
  double a = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) a += x[i];
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out->loss = red[0] * (1.0 / ((double)batch * head->msum));
    out->msum = head->msum;
    out->bad = head->bad;
  }
}

// ---------------------------------------------------------------------------
// Adam
// ---------------------------------------------------------------------------
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1,
                            float c2, int* __restrict__ wbad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *wbad = 0;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// ---------------------------------------------------------------------------
// Network input map
// ---------------------------------------------------------------------------
// |Q|^2 per probe pixel (FP64) and ||Q||_2.
__global__ __launch_bounds__(1024) void probe_norm_kernel(const double2* __restrict__ q, int mm,
                                                          double* __restrict__ out, double* __restrict__ a2) {
  __shared__ double red[1024];
  double a = 0.0;
  for (int i = threadIdx.x; i < mm; i += 1024) {
    const double2 v = q[i];
    const double w = v.x * v.x + v.y * v.y;
    a2[i] = w;
    a += w;
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sqrt(red[0]);
}

// Statistics of one position's pattern, read where the step kernel keeps sqrt(d): row
// ky is m contiguous floats in either order, and frequency kx = g CB + c + RA k2 of it
// sits at g RA + c RB + k2 (RA = CB RB), so a wave's reads stay inside whole rows.  The
// frequencies are summed in natural order: the result does not depend on the plan.
// 1600 positions of 64 x 64: 10.2 us, 26 MB at half the rate of a large copy: a position is a
// workgroup's one short run (16 values per thread, then the tree over four FP64 sums), so its
// loads do not cover its sums.  A re-layout to natural order in front of it had cost a
// second read and a write of the same bytes (18.5 us).
__global__ __launch_bounds__(256) void position_stats_kernel(const float* __restrict__ sqrtd, int lm, int lrb,
                                                             const double* __restrict__ qnorm,
                                                             double4* __restrict__ stats) {
  __shared__ double red[4][256];
  const int k = blockIdx.x, m = 1 << lm, lra = lm - lrb, lcb = lra - lrb;
  const float* s = sqrtd + ((size_t)k << (2 * lm));
  double sa = 0.0, sd = 0.0, sy = 0.0, sx = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < m * m; i += 256) {
    const int r = i >> lm, c = i & (m - 1);
    const int rem = c & ((1 << lra) - 1);
    const int at = ((rem >> lcb) << lra) + ((rem & ((1 << lcb) - 1)) << lrb) + (c >> lra);
    const double a = (double)s[(r << lm) + at];
    const double d = a * a;
    const double fy = (r < m / 2) ? r : r - m, fx = (c < m / 2) ? c : c - m;
    sa += a;
    sd += d;
    sy += fy * d;
    sx += fx * d;
  }
  red[0][threadIdx.x] = sa;
  red[1][threadIdx.x] = sd;
  red[2][threadIdx.x] = sy;
  red[3][threadIdx.x] = sx;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double tot = red[1][0];
    double4 o;
    o.x = red[0][0] / ((double)m * m) / qnorm[0];
    o.y = tot > 0.0 ? red[2][0] / tot : 0.0;
    o.z = tot > 0.0 ? red[3][0] / tot : 0.0;
    o.w = 0.0;
    stats[k] = o;
  }
}

// One workgroup per tile of the static position lists (tile_w = 32 columns, 8 rows of
// it at a time): the tile's positions and their statistics are staged in LDS, then
// every thread walks them for its pixel (the list order, as before) with one 8-byte
// read of |Q|^2 per covering position.  Walking the list from global memory per pixel,
// with blocks that spanned eight tiles' lists, took 36 us on a 512 x 512 object with
// 1600 windows of 64 x 64.
constexpr int MAP_CHUNK = 256;

__global__ __launch_bounds__(256) void map_fine_kernel(const double4* __restrict__ stats,
                                                       const double* __restrict__ a2, int m,
                                                       const int* __restrict__ tile_ptr,
                                                       const int4* __restrict__ tile_ent, int tiles_x, int tile_h,
                                                       int nr, int nc, double* __restrict__ fine) {
  __shared__ double sst[3][MAP_CHUNK];
  __shared__ int2 soff[MAP_CHUNK];
  const int tx = blockIdx.x, ty = blockIdx.y;
  const int c = tx * 32 + (threadIdx.x & 31);
  const int beg = tile_ptr[ty * tiles_x + tx], end = tile_ptr[ty * tiles_x + tx + 1];
  const size_t plane = (size_t)nr * nc;
  for (int r0 = ty * tile_h; r0 < (ty + 1) * tile_h; r0 += 8) {
    const int r = r0 + (threadIdx.x >> 5);
    double n0 = 0.0, n1 = 0.0, n2 = 0.0, den = 0.0;
    for (int e0 = beg; e0 < end; e0 += MAP_CHUNK) {
      const int n = min(MAP_CHUNK, end - e0);
      __syncthreads();
      if ((int)threadIdx.x < n) {
        const int4 en = tile_ent[e0 + threadIdx.x];
        const double4 s = stats[en.x];
        soff[threadIdx.x] = make_int2(en.y, en.z);
        sst[0][threadIdx.x] = s.x;
        sst[1][threadIdx.x] = s.y;
        sst[2][threadIdx.x] = s.z;
      }
      __syncthreads();
#pragma unroll 4
      for (int e = 0; e < n; ++e) {
        const int2 o = soff[e];
        const int dr = r - o.x, dc = c - o.y;
        if ((unsigned)dr < (unsigned)m && (unsigned)dc < (unsigned)m) {
          const double w = a2[dr * m + dc];
          n0 += w * sst[0][e];
          n1 += w * sst[1][e];
          n2 += w * sst[2][e];
          den += w;
        }
      }
    }
    if (r < nr && c < nc) {
      const size_t i = (size_t)r * nc + c;
      const bool pos = den > 0.0;
      fine[i] = pos ? n0 / den : 0.0;
      fine[plane + i] = pos ? n1 / den : 0.0;
      fine[2 * plane + i] = pos ? n2 / den : 0.0;
    }
  }
}

// One workgroup per run of cells of one cell row and channel: each thread sums a
// column of fr pixels (neighbouring threads read neighbouring columns), then the first
// threads sum fc columns per cell from LDS.
__global__ __launch_bounds__(256) void pool_kernel(const double* __restrict__ fine, int nr, int nc, int fr, int fc,
                                                   int cells, float* __restrict__ out) {
  __shared__ double cs[256];
  const int so = nc / fc, sr = nr / fr;
  const int i = blockIdx.y, ch = blockIdx.z, j0 = blockIdx.x * cells;
  const double* src = fine + (size_t)ch * nr * nc + (size_t)i * fr * nc;
  const int nj = min(cells, so - j0);
  double cell = 0.0;
  // cells = 256 / fc whole cells at a time; a cell wider than 256 columns alone, in pieces
  for (int x0 = 0; x0 < nj * fc; x0 += 256) {
    const int n = min(256, nj * fc - x0);
    double a = 0.0;
    if ((int)threadIdx.x < n)
#pragma unroll 8
      for (int y = 0; y < fr; ++y) a += src[(size_t)y * nc + (size_t)j0 * fc + x0 + threadIdx.x];
    __syncthreads();
    cs[threadIdx.x] = a;
    __syncthreads();
    if ((int)threadIdx.x < nj) {
      const int w = min(fc, n);
      for (int x = 0; x < w; ++x) cell += cs[threadIdx.x * fc + x];
    }
  }
  if ((int)threadIdx.x < nj) out[((size_t)ch * sr + i) * so + j0 + threadIdx.x] = (float)(cell / ((double)fr * fc));
}

// Phase channel: least-squares integration of the gradient field the two
// centre-of-mass channels measure (Frankot and Chellappa), in FP64.  The two real
// fields are transformed together as H = DFT(gy + i gx) and separated with the
// conjugate-symmetric parts; then phi^ = -i (wy Gy + wx Gx) / (wy^2 + wx^2) (0 at zero
// frequency) and phi = Re IDFT(phi^).  Direct DFT sums over rows and columns (S <= 64),
// in three launches of one workgroup per row or pair of columns: on one workgroup the
// S^3 sums of each pass ran from one CU's LDS (158 us at S = 64).
constexpr int PHI_MAX_S = 64;

// exp(-2 pi i j / S) for j < S by the first S threads
__device__ __forceinline__ void phi_twiddles(double2* W, int S) {
  if ((int)threadIdx.x < S) {
    double sn, cs;
    sincospi(-2.0 * (int)threadIdx.x / S, &sn, &cs);
    W[threadIdx.x] = make_double2(cs, sn);
  }
}

// sum_j v[j stride] W^(k j) (CONJ: conj(W)), j < S
template <bool CONJ>
__device__ __forceinline__ double2 phi_sum(const double2* v, const double2* W, int S, int k) {
  double2 acc = make_double2(0.0, 0.0);
  int idx = 0;
#pragma unroll 4
  for (int j = 0; j < S; ++j) {
    const double2 a = v[j], w = W[idx];
    const double wy = CONJ ? -w.y : w.y;
    acc.x += a.x * w.x - a.y * wy;
    acc.y += a.x * wy + a.y * w.x;
    idx += k;
    if (idx >= S) idx -= S;
  }
  return acc;
}

// rows of the forward transform, stored transposed: t[k][y]
__global__ __launch_bounds__(PHI_MAX_S) void phi_rows_kernel(const float* __restrict__ gy_in,
                                                             const float* __restrict__ gx_in, int S, double sy,
                                                             double sx, double2* __restrict__ t) {
  __shared__ double2 v[PHI_MAX_S], W[PHI_MAX_S];
  const int y = blockIdx.x, k = threadIdx.x;
  phi_twiddles(W, S);
  if (k < S) v[k] = make_double2(sy * gy_in[y * S + k], sx * gx_in[y * S + k]);
  __syncthreads();
  if (k < S) t[k * S + y] = phi_sum<false>(v, W, S, k);
}

// Columns k1 and -k1 (mod S): forward over y, phi^ (which pairs the frequencies k and
// -k), inverse over k0; in place (the workgroup owns both columns).
__global__ __launch_bounds__(2 * PHI_MAX_S) void phi_cols_kernel(int S, double2* __restrict__ t) {
  __shared__ double2 v[2][PHI_MAX_S], h[2][PHI_MAX_S], W[PHI_MAX_S];
  const int which = threadIdx.x / PHI_MAX_S, k0 = threadIdx.x % PHI_MAX_S;
  const int ka = blockIdx.x, kb = (S - ka) % S, k1 = which ? kb : ka;
  phi_twiddles(W, S);
  if (k0 < S) v[which][k0] = t[k1 * S + k0];
  __syncthreads();
  if (k0 < S) h[which][k0] = phi_sum<false>(v[which], W, S, k0);
  __syncthreads();
  if (k0 < S) {
    const double2 a = h[which][k0], am = h[1 - which][(S - k0) % S];
    // Gy = (h + conj(hm)) / 2, Gx = (h - conj(hm)) / (2 i)
    const double2 gy = make_double2(0.5 * (a.x + am.x), 0.5 * (a.y - am.y));
    const double2 gx = make_double2(0.5 * (a.y + am.y), -0.5 * (a.x - am.x));
    const int f0 = (k0 < (S + 1) / 2) ? k0 : k0 - S, f1 = (k1 < (S + 1) / 2) ? k1 : k1 - S;
    const double wy = 6.283185307179586 * f0 / S, wx = 6.283185307179586 * f1 / S;
    const double den = wy * wy + wx * wx;
    double2 ph = make_double2(0.0, 0.0);
    if (den > 0.0) {
      // -i (wy gy + wx gx) / den
      const double2 u = make_double2(wy * gy.x + wx * gx.x, wy * gy.y + wx * gx.y);
      ph = make_double2(u.y / den, -u.x / den);
    }
    v[which][k0] = ph;
  }
  __syncthreads();
  if (k0 < S && (which == 0 || kb != ka)) t[k1 * S + k0] = phi_sum<true>(v[which], W, S, k0);
}

// rows of the inverse: out[y][x] = Re sum_k1 t[k1][y] conj(W)^(k1 x) / S^2
__global__ __launch_bounds__(PHI_MAX_S) void phi_out_kernel(const double2* __restrict__ t, int S,
                                                            float* __restrict__ out) {
  __shared__ double2 v[PHI_MAX_S], W[PHI_MAX_S];
  const int y = blockIdx.x, x = threadIdx.x;
  phi_twiddles(W, S);
  if (x < S) v[x] = t[x * S + y];
  __syncthreads();
  if (x < S) out[y * S + x] = (float)(phi_sum<true>(v, W, S, x).x / ((double)S * S));
}

// ---------------------------------------------------------------------------
// Whole-object prolongation and restriction
// ---------------------------------------------------------------------------
__global__ void prolong_object_kernel(const void* __restrict__ coarse, int format, int sr, int sc, int f,
                                      float2* __restrict__ z, int nr, int nc) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (c >= nc) return;
  const int i = r / f, j = c / f;
  const size_t ci = (size_t)i * sc + j;
  float2 v;
  if (format == 0) {
    v = ((const float2*)coarse)[ci];
  } else if (format == 1) {
    const double2 d = ((const double2*)coarse)[ci];
    v = make_float2((float)d.x, (float)d.y);
  } else {
    const float* pl = (const float*)coarse;
    const float amp = expf(pl[ci]);
    float sn, cs;
    sincosf(pl[(size_t)sr * sc + ci], &sn, &cs);
    v = make_float2(amp * cs, amp * sn);
  }
  z[(size_t)r * nc + c] = v;
}

__global__ void restrict_object_kernel(const float2* __restrict__ z, int nr, int nc, int f, float2* __restrict__ out) {
  const int so = nc / f, sr = nr / f;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y;
  if (j >= so || i >= sr) return;
  double ax = 0.0, ay = 0.0;
  for (int y = 0; y < f; ++y)
    for (int x = 0; x < f; ++x) {
      const float2 v = z[(size_t)(i * f + y) * nc + j * f + x];
      ax += v.x;
      ay += v.y;
    }
  const double inv = 1.0 / ((double)f * f);
  out[(size_t)i * so + j] = make_float2((float)(ax * inv), (float)(ay * inv));
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
int cmse_blocks(int batch, int hw) { return (int)(((size_t)batch * hw + CMSE_THREADS - 1) / CMSE_THREADS); }

int cmse_ip_blocks(int hw) { return (hw + CMSE_THREADS - 1) / CMSE_THREADS; }

hipError_t launch_cmse(const float* y, const float2* target, const float* mask, float2* rot, double2* ip_part,
                       float* dy, double* part, int batch, int hw, CmseHead* head, CmseResult* out, hipStream_t s) {
  const int nb = cmse_blocks(batch, hw);
  if (nb <= 0) return hipSuccess;
  const int nbi = cmse_ip_blocks(hw);
  if (rot)
    hipLaunchKernelGGL(cmse_ip_kernel, dim3(nbi, batch), dim3(CMSE_THREADS), 0, s, y, target, mask, ip_part, hw);
  hipLaunchKernelGGL(cmse_head_kernel, dim3(rot ? batch + 1 : 1), dim3(256), 0, s, mask, hw, ip_part, nbi, rot, head);
  hipLaunchKernelGGL(cmse_kernel, dim3(nb), dim3(CMSE_THREADS), 0, s, y, target, mask, (const float2*)rot, dy, part,
                     batch, hw, (const CmseHead*)head);
  hipLaunchKernelGGL(cmse_loss_kernel, dim3(1), dim3(1024), 0, s, (const double*)part, nb, (const CmseHead*)head, batch,
                     out);
  return hipGetLastError();
}

__global__ void adam_reset_kernel(float* __restrict__ m, float* __restrict__ v, int64_t n, int* __restrict__ wbad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *wbad = 0;
  if (i < n) m[i] = v[i] = 0.0f;
}

hipError_t launch_adam_reset(float* m, float* v, int64_t n, int* wbad, hipStream_t s) {
  hipLaunchKernelGGL(adam_reset_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, m, v, n, wbad);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, int* wbad, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps,
                     c1, c2, wbad);
  return hipGetLastError();
}

hipError_t launch_probe_norm(const double2* q, int m, double* out, double* a2, hipStream_t s) {
  hipLaunchKernelGGL(probe_norm_kernel, dim3(1), dim3(1024), 0, s, q, m * m, out, a2);
  return hipGetLastError();
}

hipError_t launch_position_stats(const float* sqrtd, int n_pos, int m, int rb, const double* qnorm, double4* stats,
                                 hipStream_t s) {
  if (n_pos <= 0) return hipSuccess;
  auto log2i = [](int x) {
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
  };
  const int lm = log2i(m), lrb = log2i(rb);
  if ((1 << lm) != m || (1 << lrb) != rb || 2 * lrb > lm) return hipErrorInvalidValue;
  hipLaunchKernelGGL(position_stats_kernel, dim3(n_pos), dim3(256), 0, s, sqrtd, lm, lrb, qnorm, stats);
  return hipGetLastError();
}

hipError_t launch_map_fine(const double4* stats, const double* a2, int m, const int* tile_ptr, const int4* tile_ent,
                           int tiles_x, int tiles_y, int tile_w, int tile_h, int nr, int nc, double* fine,
                           hipStream_t s) {
  if (tile_w != 32 || tile_h % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(map_fine_kernel, dim3(tiles_x, tiles_y), dim3(256), 0, s, stats, a2, m, tile_ptr, tile_ent,
                     tiles_x, tile_h, nr, nc, fine);
  return hipGetLastError();
}

hipError_t launch_pool(const double* fine, int nr, int nc, int fr, int fc, float* out, hipStream_t s) {
  const int so = nc / fc, sr = nr / fr;
  const int cells = fc >= 256 ? 1 : 256 / fc;
  hipLaunchKernelGGL(pool_kernel, dim3((so + cells - 1) / cells, sr, 3), dim3(256), 0, s, fine, nr, nc, fr, fc, cells,
                     out);
  return hipGetLastError();
}

hipError_t launch_integrate_phase(const float* gy, const float* gx, int S, double sy, double sx, double2* scratch,
                                  float* out, hipStream_t s) {
  if (S < 1 || S > PHI_MAX_S) return hipErrorInvalidValue;
  hipLaunchKernelGGL(phi_rows_kernel, dim3(S), dim3(PHI_MAX_S), 0, s, gy, gx, S, sy, sx, scratch);
  hipLaunchKernelGGL(phi_cols_kernel, dim3(S / 2 + 1), dim3(2 * PHI_MAX_S), 0, s, S, scratch);
  hipLaunchKernelGGL(phi_out_kernel, dim3(S), dim3(PHI_MAX_S), 0, s, (const double2*)scratch, S, out);
  return hipGetLastError();
}

hipError_t launch_prolong_object(const void* coarse, int format, int sr, int sc, int f, float2* z, int nr, int nc,
                                 hipStream_t s) {
  hipLaunchKernelGGL(prolong_object_kernel, dim3((nc + 255) / 256, nr), dim3(256), 0, s, coarse, format, sr, sc, f, z,
                     nr, nc);
  return hipGetLastError();
}

hipError_t launch_restrict_object(const float2* z, int nr, int nc, int f, float2* out, hipStream_t s) {
  const int so = nc / f, sr = nr / f;
  hipLaunchKernelGGL(restrict_object_kernel, dim3((so + 63) / 64, sr), dim3(64), 0, s, z, nr, nc, f, out);
  return hipGetLastError();
}

}  // namespace cnn
