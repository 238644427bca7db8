// 3x3 convolutions of the coarse-object network and their gradients for gfx950.
//
// Activations between the layers are channels-last: [B][H][W][32] FP32 (the
// network's input, output and output gradient keep their [B][c][H][W] planes).
//
// Forward: every output is the FP32 FMA chain over (input channel, tap) from the bias,
// the 32 -> 32 layers as v_mfma_f32_16x16x4_f32 products: the instruction adds its four
// products one after another, k ascending, one rounding each, so the matrix cores give the
// chain's own bits (tested), at twice the rate of unpacked FP32 VALU.  The order is part of
// the interface: the phase output's bias has gradient zero by the loss's phase alignment, so
// what Adam makes of it is this rounding, and another summation would send the bias elsewhere.
//
// Backward: the 32 -> 32 products run as v_mfma_f32_32x32x16_bf16 of FP32 operands split
// exactly into three bf16 parts, x = x0 + x1 + x2, each the rest rounded to nearest (|x1| <=
// 2^-8, |x2| <= 2^-17 of x's power of two, of either sign).  Eight of the nine products are
// formed; the ninth, x2 w2, is below 2^-34 of the product.  bf16 weights are their own first
// part, so three products are exact.  What such an instruction adds to an accumulator is
// rounded to nearest where the accumulator is the larger, but an accumulator smaller than the
// products is cut off towards minus infinity at their low end (measured), so the first parts'
// products and the others are summed apart or one behind the other, see below.  Relative error
// against FP64 of the same operands, 32 samples of 128 x 128 (one FP32 FMA chain per output:
// in parentheses): weight gradients 1.4e-7 to 1.8e-7 (4.3e-7 to 5.2e-7); backward-data 0.7e-7
// to 0.95e-7 (1.7e-7 to 3.0e-7), with bf16 weights 1.0e-7 to 1.8e-7.  A product of split parts
// is not the FP32 product where a value is infinite (inf - inf in its second part) or rounds
// to infinity, so a workgroup that stages such a value, or whose weights hold one, takes the
// scalar FMA form of its tile instead.
//
// All reductions run in a fixed order: results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cmath.h"
#include "cnn.h"

namespace cnn {

namespace {

constexpr int C = 32;               // channels of the hidden layers
constexpr int CT = 16;              // output tile side of the convolutions
constexpr int HALO = CT + 2;
constexpr int HP = HALO * HALO;     // staged pixels of a tile

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mfma(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// bf16 pairs (even element in the low half) of two FP32 values, rounded to nearest
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float even, float odd) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{even, odd}, bf16x2));
}

// the three bf16 parts of eight values; `probe` becomes NaN if a first part is not finite (a
// value is not, or rounds to infinity)
__device__ __forceinline__ void split8(const float* v, uint4 (&s)[3], float& probe) {
  uint32_t p[3][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float even = v[2 * j], odd = v[2 * j + 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      p[q][j] = pack_bf16(even, odd);
      const float pe = __uint_as_float(p[q][j] << 16), po = __uint_as_float(p[q][j] & 0xffff0000u);
      if (q == 0) probe = fmaf(pe, 0.0f, fmaf(po, 0.0f, probe));
      even -= pe;
      odd -= po;
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) s[q] = make_uint4(p[q][0], p[q][1], p[q][2], p[q][3]);
}

__device__ __forceinline__ float round_bf16(float x) {
  const uint32_t u = __float_as_uint(x);
  return __uint_as_float((u + 0x7FFFu + ((u >> 16) & 1u)) & 0xffff0000u);
}

// ---------------------------------------------------------------------------
// The halo of a tile
// ---------------------------------------------------------------------------
// A tile of TH x 16 output pixels reads (TH + 2) x 18 pixels of a channels-last tensor (UP: of
// half the size, each pixel taken twice), split into PPP pieces per pixel; thread tid takes the
// pieces tid, tid + 256, ...: all its loads are issued together, without a branch.
template <bool UP, int TH, int PPP>
struct Halo {
  static constexpr int PIXELS = (TH + 2) * HALO, N = (PIXELS * PPP + 255) / 256;
  int vo[N];   // piece k: offset in bytes from the tile's first source pixel
  __device__ __forceinline__ void init(int tid, int Wi) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int i = tid + 256 * k, p = i / PPP, yy = p / HALO - 1, xx = p % HALO - 1;
      vo[k] = ((UP ? yy >> 1 : yy) * Wi + (UP ? xx >> 1 : xx)) * (C * 4) + i % PPP * (C * 4 / PPP);
    }
  }
  // The source of a tile of the output (H x W): a resource that covers the source rows that
  // exist, so that a row above the image is a negative offset, one below lies past the end, and
  // both read as zero.
  struct At {
    mg::rsrc_t rs;
    int base, x0, W;
  };
  static __device__ __forceinline__ At at(const float* in, int b, int y0, int x0, int H, int W) {
    const int Hi = UP ? H >> 1 : H, Wi = UP ? W >> 1 : W;
    const int ys = UP ? y0 >> 1 : y0, yb = max(ys - 1, 0), rows = min(Hi - yb, (UP ? TH / 2 : TH) + 2);
    return {mg::make_rsrc(in + ((size_t)b * Hi + yb) * Wi * C, (unsigned)rows * Wi * (C * 4)),
            ((ys - yb) * Wi + (UP ? x0 >> 1 : x0)) * (C * 4), x0, W};
  }
  // offset of piece k of thread tid (a column outside the image reads as zero)
  __device__ __forceinline__ int offset(const At& t, int k, int tid) const {
    const int x = t.x0 + (tid + 256 * k) / PPP % HALO - 1;
    return (unsigned)x < (unsigned)t.W ? t.base + vo[k] : -C * 4;
  }
  // get(k, resource, offset) for every piece
  template <typename F>
  __device__ __forceinline__ void load(const At& t, int tid, F get) const {
    if (t.x0 > 0 && t.x0 + CT < t.W) {
#pragma unroll
      for (int k = 0; k < N; ++k) get(k, t.rs, t.base + vo[k]);
    } else {
      asm volatile("" : "+v"(tid));   // the columns are formed again at an edge, not kept
#pragma unroll
      for (int k = 0; k < N; ++k) get(k, t.rs, offset(t, k, tid));
    }
  }
};

// tile q of a batch: sample, first row and column
struct TileAt {
  int b, y0, x0;
};
__device__ __forceinline__ TileAt tile_at(int q, int tx, int ty, int th) {
  const int b = q / (tx * ty), r = q - b * (tx * ty), ry = r / tx;
  return {b, ry * th, (r - ry * tx) * CT};
}

// ---------------------------------------------------------------------------
// 32 -> 32 convolution, forward
// ---------------------------------------------------------------------------
// Tiles of 16 x 4 P output pixels, four waves, each wave P rows.  The chain of an output runs
// over channels, taps within a channel: of the 36 steps of four channels, product p takes 4 p to
// 4 p + 3, one per lane group, so every lane holds operands of its own tap and channel (with
// K = 1 products the halves of a wave held the same weights, twice the reads per product).
// The halo is staged with the channels c, c + 4, c + 8, ... of a pixel side by side, 136 bytes
// per pixel: one 8-byte read gives the operand of the same product of two chunks of four
// channels, and 16 neighbouring pixels cover all banks (two of a lane's taps read 32 pairs).
// A weight or pixel register is loaded for the next two chunks right behind its last product
// (held there by scheduling barriers), 72 P products ahead of its use.
//
// P = 4: 512 workgroups (two per CU) walk the tiles, the next tile's halo on its way into
// registers while the products run.  Bound: 2 * 9 * 32 * 32 flops per pixel at the FP32
// matrix rate, 61 us at 2.4 GHz for 32 samples of 128 x 128, 69 us at the 2.1 GHz that the
// clock is at when a few such launches follow an idle time.  110 -> 88 us (a tile per
// workgroup with the halo loaded and stored piece by piece took as long to stage under the
// other workgroup's products as to multiply).
// P = 1, 2: where the 16 x 16 tiles would leave CUs idle, one tile of 4 or 8 rows per
// workgroup: up to 64 tiles 16 x 16 (one 128 x 128 sample) 17.0 -> 6.6 us with P = 1, up to
// 128 tiles 17.7 -> 8.8 us with P = 2 (P = 1: 11.8, P = 4: 13.3); above, P = 4 is faster (192 tiles:
// 14.0, with P = 2 16.5).
constexpr int FWD_TAPS = 9 * 2 * 64;   // float2 of the weights of two chunks

template <bool UP, int P>
__global__ __launch_bounds__(256, 2) void conv32_forward_kernel(const float* __restrict__ in,
                                                                const float2* __restrict__ w,
                                                                const float* __restrict__ bias,
                                                                float* __restrict__ out, int H, int W, int tx, int ty,
                                                                int total) {
  constexpr bool LOOP = P == 4;
  using HaloT = Halo<UP, 4 * P, 8>;
  constexpr int TH = 4 * P, HR = HaloT::PIXELS, LP = 34, NL = HaloT::N;
  __shared__ float2 T2[HR * LP / 2];
  float* T = reinterpret_cast<float*>(T2);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 15, kk = lane >> 4;
  const mg::rsrc_t wrs = mg::make_rsrc(w, 4 * FWD_TAPS * sizeof(float2));
  int wo = lane * (int)sizeof(float2);
  float2 wr[9][2];
#pragma unroll
  for (int p = 0; p < 9; ++p)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) wr[p][cb] = mg::bload2(wrs, wo, (p * 2 + cb) * 512);
  HaloT halo;
  halo.init(tid, UP ? W >> 1 : W);
  float4 hv[NL];
  auto load = [&](int q) {
    const TileAt t = tile_at(q, tx, ty, TH);
    halo.load(HaloT::at(in, t.b, t.y0, t.x0, H, W), tid, [&](int k, mg::rsrc_t rs, int off) { hv[k] = mg::bload4(rs, off, 0); });
  };
  int q = blockIdx.x;
  load(q);
  // this lane's operand of product p: step 4 p + kk of the 36
  const float2* xa[9];
#pragma unroll
  for (int p = 0; p < 9; ++p) {
    const int s = 4 * p + kk, c = s / 9, t = s - 9 * c;
    xa[p] = T2 + ((P * wave + t / 3) * HALO + n + t % 3) * (LP / 2) + 4 * c;
  }
  int ko = kk;
  for (; q < total; q += gridDim.x) {
    // opaque offsets: the weights and the bias are read again for each tile, not all held in registers
    asm volatile("" : "+v"(wo), "+v"(ko));
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int i = tid + 256 * k;
      if (i < HR * 8) {
        float* d = T + (i >> 3) * LP + (i & 7);
        d[0] = hv[k].x;
        d[8] = hv[k].y;
        d[16] = hv[k].z;
        d[24] = hv[k].w;
      }
    }
    float4 bb[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) bb[cb] = *reinterpret_cast<const float4*>(bias + 16 * cb + 4 * ko);
    __syncthreads();
    if (LOOP && q + (int)gridDim.x < total) load(q + gridDim.x);
    // lane (kk, n) holds channels 16 cb + 4 kk + (0..3) of pixel n of row r
    f32x4 acc[P][2];
#pragma unroll
    for (int r = 0; r < P; ++r)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[r][cb] = f32x4{bb[cb].x, bb[cb].y, bb[cb].z, bb[cb].w};
    float2 xr[9][P];
#pragma unroll
    for (int p = 0; p < 9; ++p)
#pragma unroll
      for (int r = 0; r < P; ++r) xr[p][r] = xa[p][r * HALO * (LP / 2)];
#pragma unroll
    for (int gp = 0; gp < 4; ++gp)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int p = 0; p < 9; ++p) {
#pragma unroll
          for (int r = 0; r < P; ++r)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
              acc[r][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(u ? wr[p][cb].y : wr[p][cb].x,
                                                                u ? xr[p][r].y : xr[p][r].x, acc[r][cb], 0, 0, 0);
          if (u) {
            if (gp < 3) {
#pragma unroll
              for (int r = 0; r < P; ++r) xr[p][r] = xa[p][r * HALO * (LP / 2) + gp + 1];
            }
            if (LOOP || gp < 3) {
#pragma unroll
              for (int cb = 0; cb < 2; ++cb)
                wr[p][cb] = mg::bload2(wrs, wo, ((((gp + 1) & 3) * 9 + p) * 2 + cb) * 512);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
    if (LOOP) __syncthreads();   // the tile is read; the next one may overwrite it
    const TileAt at = tile_at(q, tx, ty, TH);
#pragma unroll
    for (int r = 0; r < P; ++r) {
      const int y = at.y0 + P * wave + r, x = at.x0 + n;
      if (y < H && x < W) {
        float* d = out + (((size_t)at.b * H + y) * W + x) * C + 4 * kk;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          *reinterpret_cast<float4*>(d + 16 * cb) = make_float4(fmaxf(acc[r][cb][0], 0.0f), fmaxf(acc[r][cb][1], 0.0f),
                                                                fmaxf(acc[r][cb][2], 0.0f), fmaxf(acc[r][cb][3], 0.0f));
      }
    }
    if (!LOOP) break;
  }
}

// ---------------------------------------------------------------------------
// 32 -> 32 convolution, backward-data
// ---------------------------------------------------------------------------
// One workgroup of four waves per 16 x 16 output tile: the 18 x 18 x 32 halo is split
// while it is staged into LDS (three planes, 64 bytes per pixel, its four 16-byte
// chunks rotated by the pixel index so that the 16 lanes of a fragment read cover all
// banks), 62 KB, two workgroups per CU so that one's staging overlaps the other's
// products.  Products are D[co][pixel] += W[co][ci] X[ci][pixel] per tap and half of
// the input channels; a wave owns four rows of the tile (two blocks of 2 x 16 pixels), and
// the weights come as prepared fragments (54 KB, shared through L1 and L2).
// FP32 weights: the seven smaller products of all 18 steps come first and the first parts'
// product, three steps at a time, last, so that a sum takes 18 roundings at its own size
// (relative error 1.5e-7 to 2.5e-7 -> 0.65e-7 to 0.95e-7); the weights' first parts, read twice,
// are in LDS (18 KB, which still leaves two workgroups per CU: fragments from L2 for both
// passes 82 us, MODE 3 78).
// MODE 2: zero where omask <= 0.  3: sum of each 2 x 2 block (the adjoint of the
// upsampling), zero where omask <= 0, written at half the size.
// 512 workgroups (two per CU) walk the tiles: the next tile's halo is loaded, a piece every
// other step, while the products run, and the masks with the last ones.  (A tile per
// workgroup stood 9000 of its 33000 clocks at the loads, which all workgroups issued at once,
// and 8000 at the masks, read one after another; the fragments three steps ahead spill, and
// so do the first parts' sums in registers of their own.)
// Bound: 2 * 9 * 32 * 32 flops per pixel at the eight-product rate (31 us of MFMA issue for
// 32 samples of 128 x 128, 12 with bf16 weights) and the activations' traffic (42 us, 23 with
// MODE 3): 75 us, MODE 3 73 (six products of truncated parts 68 and 64).
template <int WS>
struct Pairs;
template <>
struct Pairs<3> {
  static constexpr int N = 8;
  static constexpr int x[8] = {2, 1, 2, 1, 0, 1, 0, 0}, w[8] = {1, 2, 0, 1, 2, 0, 1, 0};
};
template <>
struct Pairs<1> {
  static constexpr int N = 3;
  static constexpr int x[3] = {2, 1, 0}, w[3] = {0, 0, 0};
};

// The products of one K step, added to acc in two sums that start from zero, the first parts'
// product and the others, largest first: an accumulator that is smaller than the products is cut
// off (towards minus infinity) at the products' low end, and a larger one takes a rounding for
// each product, so neither form fits a running sum.  The adds are held here: the sums of
// several steps do not fit the registers.
__device__ __forceinline__ void add_products(const uint4 (&w)[3], const uint4 (&x)[3], f32x16& acc) {
  const f32x16 zero = {};
  const f32x16 first = mfma(w[0], x[0], zero);
  f32x16 t = {};
#pragma unroll
  for (int j = Pairs<3>::N - 2; j >= 0; --j) t = mfma(w[Pairs<3>::w[j]], x[Pairs<3>::x[j]], t);
  acc = (acc + first) + t;
  asm volatile("" : "+v"(acc));
}

struct Conv32Args {
  const float* in;        // [B][H][W][32]
  const uint4* frag;      // prepared fragments (see prep_kernel)
  const float* w;         // master weights of the layer [32][32][9]
  float* out;
  const float* omask;
  const int* wbad;        // nonzero: the weights hold a non-finite value
  int H, W;               // size of the convolution's output
};

// scalar form of one output value, weights transposed and flipped
template <int WS>
__device__ float conv32_at(const Conv32Args& a, int b, int o, int y, int x) {
  float acc = 0.0f;
  for (int c = 0; c < C; ++c)
    for (int t = 0; t < 9; ++t) {
      const int gy = y + t / 3 - 1, gx = x + t % 3 - 1;
      const bool in = gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
      float w = a.w[(c * C + o) * 9 + 8 - t];
      if (WS == 1) w = round_bf16(w);
      acc = fmaf(w, in ? a.in[(((size_t)b * a.H + gy) * a.W + gx) * C + c] : 0.0f, acc);
    }
  return acc;
}

template <int MODE, int WS>
__device__ __noinline__ void conv32_scalar(const Conv32Args& a, int b, int y0, int x0) {
  if constexpr (MODE == 3) {
    const int H2 = a.H >> 1, W2 = a.W >> 1;
    for (int i = threadIdx.x; i < (CT / 2) * (CT / 2) * C; i += 256) {
      const int o = i % C, p = i / C, y = y0 / 2 + p / (CT / 2), x = x0 / 2 + p % (CT / 2);
      if (y >= H2 || x >= W2) continue;
      const size_t at = (((size_t)b * H2 + y) * W2 + x) * C + o;
      float v[4];
      for (int q = 0; q < 4; ++q) v[q] = conv32_at<WS>(a, b, o, 2 * y + q / 2, 2 * x + q % 2);
      a.out[at] = a.omask[at] > 0.0f ? (v[0] + v[1]) + (v[2] + v[3]) : 0.0f;
    }
  } else {
    for (int i = threadIdx.x; i < CT * CT * C; i += 256) {
      const int o = i % C, p = i / C, y = y0 + p / CT, x = x0 + p % CT;
      if (y >= a.H || x >= a.W) continue;
      const size_t at = (((size_t)b * a.H + y) * a.W + x) * C + o;
      const float v = conv32_at<WS>(a, b, o, y, x);
      a.out[at] = a.omask[at] > 0.0f ? v : 0.0f;
    }
  }
}

__device__ __forceinline__ float lane_xor_f(float v, bool far) {
  return far ? __int_as_float(mg::xor_lane<16>(__float_as_int(v))) : __int_as_float(mg::xor_lane<1>(__float_as_int(v)));
}

template <int MODE, int WS>
__global__ __launch_bounds__(256, 2) void conv32_kernel(Conv32Args a, int tx, int ty, int total) {
  using HaloT = Halo<false, CT, 4>;
  constexpr int NS = HaloT::N;
  constexpr bool TWO = WS == 3;
  constexpr int G0 = TWO ? 1 : 0, WG = WS - G0;   // parts of the weights that come as fragments
  __shared__ uint4 T[3][HP * 4];
  __shared__ uint4 W0[TWO ? 18 * 64 : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, n = lane & 31;
  const int wbad = *a.wbad;
  const mg::rsrc_t frs = mg::make_rsrc(a.frag, 18 * WS * 64 * sizeof(uint4));
  int fo = lane * (int)sizeof(uint4);
  auto frag = [&](int step, int s) { return __builtin_bit_cast(uint4, mg::bload4(frs, fo, (step * WS + s) * 1024)); };
  if constexpr (TWO)
    for (int i = tid; i < 18 * 64; i += 256) W0[i] = a.frag[(i >> 6) * 192 + (i & 63)];

  // staging: thread i takes 8 channels (chunk i & 3) of halo pixel i >> 2
  HaloT halo;
  halo.init(tid, a.W);
  float4 st[NS][2];
  auto source = [&](int q) {
    const TileAt t = tile_at(q, tx, ty, CT);
    return HaloT::at(a.in, t.b, t.y0, t.x0, a.H, a.W);
  };
  int to = tid;
  auto load = [&](const typename HaloT::At& t, int k) {
    const int off = halo.offset(t, k, to);
    st[k][0] = mg::bload4(t.rs, off, 0);
    st[k][1] = mg::bload4(t.rs, off, 16);
  };
  int q0 = blockIdx.x;
  {
    const typename HaloT::At src = source(q0);
#pragma unroll
    for (int k = 0; k < NS; ++k) load(src, k);
  }
  const int p0 = (4 * wave + (n >> 4)) * HALO + (n & 15);
#pragma unroll 1
  for (; q0 < total; q0 += gridDim.x) {
    asm volatile("" : "+v"(fo), "+v"(to));   // the fragments are read again for each tile
    // fragments are loaded PF steps ahead of their products: they come from L2 (54 KB per
    // tile and wave, more than L1 holds); a piece of the next halo every SPREAD steps
    constexpr int PF = 2, SPREAD = 2;
    constexpr int STEPS = TWO ? 24 : 18;
    uint4 wf[PF + 1][WG], w0[2][3];
    float probe = 0.0f;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int i = tid + 256 * k, p = i >> 2;
      const float v[8] = {st[k][0].x, st[k][0].y, st[k][0].z, st[k][0].w, st[k][1].x, st[k][1].y, st[k][1].z, st[k][1].w};
      uint4 s[3];
      split8(v, s, probe);
      if (i < HP * 4) {
        const int at = 4 * p + ((i & 3) ^ ((p >> 2) & 3));
#pragma unroll
        for (int q = 0; q < 3; ++q) T[q][at] = s[q];
      }
    }
#pragma unroll
    for (int k = 0; k < PF; ++k)
#pragma unroll
      for (int s = 0; s < WG; ++s) wf[k][s] = frag(k, G0 + s);
    const bool bad = __syncthreads_or(!(probe == 0.0f) || wbad);
    // the last tile's own halo is loaded again, unused, rather than a branch around each load
    const typename HaloT::At next = source(min(q0 + (int)gridDim.x, total - 1));
    const TileAt tl = tile_at(q0, tx, ty, CT);
    if (bad) {
      conv32_scalar<MODE, WS>(a, tl.b, tl.y0, tl.x0);
#pragma unroll
      for (int k = 0; k < NS; ++k) load(next, k);
      __syncthreads();
      continue;
    }

    f32x16 acc[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[k][r] = 0.0f;
    // lane (h, n) holds channels 8 q + 4 h + (0..3) of pixel n of each block; the masks are loaded
    // with the last products still to come
    size_t at[2];
    bool in[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int y = tl.y0 + 4 * wave + 2 * k + (n >> 4), x = tl.x0 + (n & 15);
      in[k] = y < a.H && x < a.W && (MODE == 2 || !(n & 17));
      const int sh = MODE == 2 ? 0 : 1, ys = min(y, a.H - 1) >> sh, xs = min(x, a.W - 1) >> sh;
      at[k] = (((size_t)tl.b * (a.H >> sh) + ys) * (a.W >> sh) + xs) * C + 4 * h;
    }
    float4 mk[2][4];
    // software pipeline, held by scheduling barriers: step i issues the weights of step i +
    // PF and the LDS reads of step i + 1 before its own twelve products
    uint4 x[2][2][3];
    auto read = [&](int step, uint4 (&xs)[2][3], uint4 (&ws)[3]) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int i = step < 18 ? step : 3 * (step - 18) + q, t = i >> 1, kh = i & 1;
        if (TWO && (step >= 18 || q == 0)) ws[q] = W0[i * 64 + lane];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int p = p0 + (2 * k + t / 3) * HALO + t % 3;
          xs[k][q] = T[step < 18 ? q : 0][4 * p + ((2 * kh + h) ^ ((p >> 2) & 3))];
        }
      }
    };
    read(0, x[0], w0[0]);
#pragma unroll
    for (int step = 0; step < STEPS; ++step) {
      if (step + PF < 18) {
#pragma unroll
        for (int s = 0; s < WG; ++s) wf[(step + PF) % (PF + 1)][s] = frag(step + PF, G0 + s);
      }
      if (step + 1 < STEPS) read(step + 1, x[(step + 1) & 1], w0[(step + 1) & 1]);
      if (step % SPREAD == 0 && step / SPREAD < NS) load(next, step / SPREAD);
      if (step == (TWO ? 18 : 18 - PF)) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int q = 0; q < 4; ++q) mk[k][q] = *reinterpret_cast<const float4*>(a.omask + at[k] + 8 * q);
      }
      __builtin_amdgcn_sched_barrier(0);
      const uint4 (&xs)[2][3] = x[step & 1];
      if (TWO && step >= 18) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int k = 0; k < 2; ++k) acc[k] = mfma(w0[step & 1][q], xs[k][q], acc[k]);
      } else {
#pragma unroll
        for (int j = 0; j < Pairs<WS>::N - (TWO ? 1 : 0); ++j)
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int w = Pairs<WS>::w[j];
            acc[k] = mfma(w < G0 ? w0[step & 1][0] : wf[step % (PF + 1)][w - G0], xs[k][Pairs<WS>::x[j]], acc[k]);
          }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();   // the tile is read; the next one may overwrite it

#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float4 v = make_float4(acc[k][4 * q], acc[k][4 * q + 1], acc[k][4 * q + 2], acc[k][4 * q + 3]);
        if constexpr (MODE == 3) {
          // 2 x 2 sums: the horizontal neighbour, then the row below
          v = make_float4(v.x + lane_xor_f(v.x, false), v.y + lane_xor_f(v.y, false), v.z + lane_xor_f(v.z, false),
                          v.w + lane_xor_f(v.w, false));
          v = make_float4(v.x + lane_xor_f(v.x, true), v.y + lane_xor_f(v.y, true), v.z + lane_xor_f(v.z, true),
                          v.w + lane_xor_f(v.w, true));
        }
        const float4 m = mk[k][q];
        v = make_float4(m.x > 0.0f ? v.x : 0.0f, m.y > 0.0f ? v.y : 0.0f, m.z > 0.0f ? v.z : 0.0f,
                        m.w > 0.0f ? v.w : 0.0f);
        if (in[k]) *reinterpret_cast<float4*>(a.out + at[k] + 8 * q) = v;
      }
  }
}

// ---------------------------------------------------------------------------
// Few -> 32 channels (the first layer; backward-data of the last one)
// ---------------------------------------------------------------------------
// Planes in, channels-last out.  One workgroup per 16 x 4 pixels, each wave eight output
// channels of all 64 pixels, so its weights w[co][c][t] are uniform (scalar loads); the
// four waves share the input reads in L1.  9 CI FMAs per output value against 4 bytes
// written (and 4 of mask read): bound by memory.
template <int CI, bool MASK>
__global__ __launch_bounds__(256) void conv_thin_kernel(const float* __restrict__ in, const float* __restrict__ w,
                                                        const float* __restrict__ bias, float* __restrict__ out,
                                                        const float* __restrict__ omask, int H, int W) {
  const int lane = threadIdx.x & 63, cog = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x = blockIdx.x * 16 + (lane & 15), y = blockIdx.y * 4 + (lane >> 4), b = blockIdx.z;
  const float* inb = in + (size_t)b * CI * H * W;
  float v[CI][9];
#pragma unroll
  for (int c = 0; c < CI; ++c)
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int gy = y + t / 3 - 1, gx = x + t % 3 - 1;
      v[c][t] = (gy >= 0 && gy < H && gx >= 0 && gx < W) ? inb[((size_t)c * H + gy) * W + gx] : 0.0f;
    }
  float acc[8];
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    acc[o] = MASK ? 0.0f : bias[cog * 8 + o];
#pragma unroll
    for (int c = 0; c < CI; ++c)
#pragma unroll
      for (int t = 0; t < 9; ++t) acc[o] = fmaf(w[((cog * 8 + o) * CI + c) * 9 + t], v[c][t], acc[o]);
  }
  if (y >= H || x >= W) return;
  const size_t at = (((size_t)b * H + y) * W + x) * C + cog * 8;
  float4* dst = reinterpret_cast<float4*>(out + at);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float4 r = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    if constexpr (MASK) {
      const float4 mk = reinterpret_cast<const float4*>(omask + at)[q];
      r = make_float4(mk.x > 0.0f ? r.x : 0.0f, mk.y > 0.0f ? r.y : 0.0f, mk.z > 0.0f ? r.z : 0.0f,
                      mk.w > 0.0f ? r.w : 0.0f);
    } else {
      r = make_float4(fmaxf(r.x, 0.0f), fmaxf(r.y, 0.0f), fmaxf(r.z, 0.0f), fmaxf(r.w, 0.0f));
    }
    dst[q] = r;
  }
}

// ---------------------------------------------------------------------------
// 32 -> 2 channels (the head): channels-last in, planes out
// ---------------------------------------------------------------------------
// One workgroup per 16 x 16 tile, one pixel per thread; the halo is staged as it is (128
// bytes per pixel, chunks rotated against bank conflicts), the weights w[c][t][o] are
// uniform.  576 FMAs per 128 bytes read: bound by the read of the activations (13 us for 32
// samples of 128 x 128; 29.7 -> 22.2 us with the halo's loads in flight together).
__global__ __launch_bounds__(256) void conv_head_kernel(const float* __restrict__ in, const float* __restrict__ w,
                                                        const float* __restrict__ bias, float* __restrict__ out,
                                                        int H, int W) {
  __shared__ float4 T[HP * 8];
  const int x0 = blockIdx.x * CT, y0 = blockIdx.y * CT, b = blockIdx.z;
  Halo<false, CT, 8> halo;
  float4 hv[halo.N];
  halo.init(threadIdx.x, W);
  halo.load(halo.at(in, b, y0, x0, H, W), threadIdx.x, [&](int k, mg::rsrc_t rs, int off) { hv[k] = mg::bload4(rs, off, 0); });
#pragma unroll
  for (int k = 0; k < halo.N; ++k) {
    const int i = threadIdx.x + 256 * k, p = i >> 3;
    if (i < HP * 8) T[8 * p + ((i & 7) ^ ((p >> 1) & 7))] = hv[k];
  }
  __syncthreads();
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float a0 = bias[0], a1 = bias[1];
#pragma unroll 1
  for (int q = 0; q < 8; ++q) {
    float4 v[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int p = (ty + t / 3) * HALO + tx + t % 3;
      v[t] = T[8 * p + (q ^ ((p >> 1) & 7))];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const float xv = c == 0 ? v[t].x : c == 1 ? v[t].y : c == 2 ? v[t].z : v[t].w;
        const float* wq = w + ((4 * q + c) * 9 + t) * 2;
        a0 = fmaf(wq[0], xv, a0);
        a1 = fmaf(wq[1], xv, a1);
      }
  }
  const int y = y0 + ty, x = x0 + tx;
  if (y < H && x < W) {
    const size_t at = ((size_t)b * 2 * H + y) * W + x;
    out[at] = a0;
    out[at + (size_t)H * W] = a1;
  }
}

// ---------------------------------------------------------------------------
// Weight gradients
// ---------------------------------------------------------------------------
// Workgroups walk runs of 16 x 8 pixel tiles.  The tensors are staged
// transposed: channel by channel, 16 consecutive pixels of a row as split bf16 values
// (a staging thread reads eight pixels of its channel, 32 lanes reading the 128
// contiguous bytes of a pixel), so a row of a tile is one K = 16 step of
// D[row channel][column channel] += A[channel][pixel] B[pixel][channel].
constexpr int GH = 8;                                  // tile rows
constexpr int A_PITCH = GH * 32 + 16;                  // bytes per channel of a staged tile without halo
constexpr int B_ROW = 48;                              // bytes per row of the halo tile (24 pixels, 18 used)
constexpr int B_PITCH = (GH + 2) * B_ROW + 16;         // odd multiples of 16 bytes: no bank conflicts
constexpr int SQ_LDS = 3 * C * (A_PITCH + B_PITCH);    // 74 KB: one of a workgroup's two buffers

struct Wgrad32Args {
  const float* in;      // [B][Hi][Wi][32]
  const float* dout;    // [B][H][W][32]
  float* part;
  int H, W, tiles_x, tiles_per_sample, total_tiles, tiles_per_wg;
};

// n of 8 pixels (channel c, row y, from x): FP32 values, 0 outside
template <bool UP>
__device__ __forceinline__ void load8(const float* base, int H, int W, int y, int x, int c, int n, float* v) {
  const int Wi = UP ? W >> 1 : W;
  if (n == 8 && y >= 0 && y < H && x >= 0 && x + 8 <= W) {   // inside: one address, constant offsets
    const float* p = base + ((size_t)(UP ? y >> 1 : y) * Wi + (UP ? x >> 1 : x)) * C + c;
    if (UP) {   // pixels x .. x + 7 of the doubled row: the low-resolution columns x / 2 .. (x + 7) / 2
      const int odd = x & 1;
      float q[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) q[j] = (j < 4 || odd) ? p[j * C] : 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = odd ? q[(j + 1) >> 1] : q[j >> 1];
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p[j * C];
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int gx = x + j;
    v[j] = (j < n && y >= 0 && y < H && gx >= 0 && gx < W)
               ? base[((size_t)(UP ? y >> 1 : y) * Wi + (UP ? gx >> 1 : gx)) * C + c]
               : 0.0f;
  }
}

constexpr int SQ_THREADS = 768;

// The scalar form of a run of tiles: element e of its part row, summed pixel by pixel.
template <bool UP>
__device__ __noinline__ void wgrad32_scalar(const Wgrad32Args& a, int t_begin, int t_end) {
  const int Hi = UP ? a.H >> 1 : a.H, Wi = UP ? a.W >> 1 : a.W;
  float* pr = a.part + (size_t)blockIdx.x * SQ_ROW;
  for (int e = threadIdx.x; e < SQ_ROW; e += SQ_THREADS) {
    const int t = e >> 10, r = (e >> 6) & 15, lane = e & 63;
    const bool isb = e >= 9 * C * C;
    const int co = isb ? e - 9 * C * C : 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), ci = lane & 31;
    float acc = 0.0f;
    for (int tile = t_begin; tile < t_end; ++tile) {
      const int b = tile / a.tiles_per_sample, tr = tile - b * a.tiles_per_sample;
      for (int p = 0; p < GH * 16; ++p) {
        const int y = (tr / a.tiles_x) * GH + p / 16, x = (tr % a.tiles_x) * 16 + p % 16;
        if (y >= a.H || x >= a.W) continue;
        const float g = a.dout[(((size_t)b * a.H + y) * a.W + x) * C + co];
        if (isb) {
          acc += g;
          continue;
        }
        const int gy = y + t / 3 - 1, gx = x + t % 3 - 1;
        const bool in = gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
        acc = fmaf(g, in ? a.in[(((size_t)b * Hi + (UP ? gy >> 1 : gy)) * Wi + (UP ? gx >> 1 : gx)) * C + ci] : 0.0f,
                   acc);
      }
    }
    pr[e] = acc;
  }
}

// 32 x 32 channels.  A workgroup of twelve waves per CU: wave (rg, dy) takes rows 2 rg and
// 2 rg + 1 of the tile and the three taps of row dy, their horizontal shifts formed in
// registers from one row read (three 32 x 32 sums, 48 registers).  Tiles are staged into
// two LDS buffers in turn (147 KB), the next tile's values loaded to registers before the current
// one's products and split and stored after them, so that neither memory latency nor
// the staging's arithmetic stands between the products.  The row groups' sums
// are added in order through LDS at the end of the run.
// 32 samples of 128 x 128: 101 us, through the upsampling 99 (six products of truncated
// parts added to the running sums: 90 and 84, with a relative error of 7.4e-7 and 6.2e-7 against
// 1.8e-7 and 1.5e-7, see the top of this file; all eight in one sum per step, added once: 96 and
// 99, 2.2e-7 and 1.9e-7).
template <bool UP>
__global__ __launch_bounds__(SQ_THREADS, 3) void wgrad32_kernel(Wgrad32Args a) {
  extern __shared__ uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wave / 3, dy = wave - 3 * rg;
  const int Hi = UP ? a.H >> 1 : a.H, Wi = UP ? a.W >> 1 : a.W;
  f32x16 acc[3];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
  float bsum = 0.0f, probe = 0.0f;   // this thread's share of channel tid & 31's bias gradient
  const int t_begin = blockIdx.x * a.tiles_per_wg, t_end = min(a.total_tiles, t_begin + a.tiles_per_wg);
  int to = tid;   // the loops' own copy: index arithmetic is formed again for each tile, not held in registers
  // Staging: thread tid takes channel sc of pixel groups sg (0 .. 23) and sg + 24: groups
  // 0 .. 15 are the 8 x 2 of dout, 16 .. 45 the 10 x 3 of in (the third of 2 pixels).
  float v[2][8];
  auto load = [&](int tile) {
    const int sc = to & 31, sg = to >> 5;
    const int b = tile / a.tiles_per_sample, tr = tile - b * a.tiles_per_sample;
    const int y0 = (tr / a.tiles_x) * GH, x0 = (tr % a.tiles_x) * 16;
    const float* inb = a.in + (size_t)b * Hi * Wi * C;
    const float* dob = a.dout + (size_t)b * a.H * a.W * C;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = sg + 24 * k, q = i - 16, row = q / 3, gx = q - 3 * row;
      if (k == 0 && i < 16)
        load8<false>(dob, a.H, a.W, y0 + (i >> 1), x0 + 8 * (i & 1), sc, 8, v[k]);
      else
        load8<UP>(inb, a.H, a.W, i < 46 ? y0 + row - 1 : -1, x0 + 8 * gx - 1, sc, gx == 2 ? 2 : 8, v[k]);
    }
  };
  auto store = [&](int buf) {
    const int sc = to & 31, sg = to >> 5;
    unsigned char* const As = reinterpret_cast<unsigned char*>(smem) + buf * SQ_LDS;   // dout
    unsigned char* const Bs = As + 3 * C * A_PITCH;                                    // in, with halo
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = sg + 24 * k;
      uint4 s[3];
      split8(v[k], s, probe);
      if (k == 0 && i < 16) {
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(As + (q * C + sc) * A_PITCH + 16 * i) = s[q];
        bsum += ((v[k][0] + v[k][1]) + (v[k][2] + v[k][3])) + ((v[k][4] + v[k][5]) + (v[k][6] + v[k][7]));
      } else if (i < 46) {
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(Bs + (q * C + sc) * B_PITCH + 16 * (i - 16)) = s[q];
      }
    }
  };
  if (t_begin < t_end) {
    load(t_begin);
    store(0);
  }
  __syncthreads();
  for (int tile = t_begin; tile < t_end; ++tile) {
    asm volatile("" : "+v"(to));
    const int buf = (tile - t_begin) & 1;
    const unsigned char* const As = reinterpret_cast<const unsigned char*>(smem) + buf * SQ_LDS;
    const unsigned char* const Bs = As + 3 * C * A_PITCH;
    const bool more = tile + 1 < t_end;
    if (more) load(tile + 1);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int row = 2 * rg + k;
      uint4 g[3], d[3];
      uint32_t d4[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        g[q] = *reinterpret_cast<const uint4*>(As + (q * C + n) * A_PITCH + row * 32 + h * 16);
        const unsigned char* src = Bs + (q * C + n) * B_PITCH + (row + dy) * B_ROW + h * 16;
        d[q] = *reinterpret_cast<const uint4*>(src);
        d4[q] = *reinterpret_cast<const uint32_t*>(src + 16);
      }
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        uint4 x[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          if (dx == 0) x[q] = d[q];
          else if (dx == 2) x[q] = make_uint4(d[q].y, d[q].z, d[q].w, d4[q]);
          else x[q] = make_uint4(__builtin_amdgcn_alignbit(d[q].y, d[q].x, 16), __builtin_amdgcn_alignbit(d[q].z, d[q].y, 16),
                                 __builtin_amdgcn_alignbit(d[q].w, d[q].z, 16), __builtin_amdgcn_alignbit(d4[q], d[q].w, 16));
        }
        add_products(g, x, acc[dx]);
      }
    }
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  if (__syncthreads_or(!(probe == 0.0f))) {
    wgrad32_scalar<UP>(a, t_begin, t_end);
    return;
  }
  // the row groups' sums in order, then the row: fragment order [t][r][lane], then the bias
  float* const red = reinterpret_cast<float*>(smem);
  for (int w = 0; w < 4; ++w) {
    if (rg == w)
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float* d = red + ((3 * dy + t) * 16 + r) * 64 + lane;
          *d = w ? *d + acc[t][r] : acc[t][r];
        }
    __syncthreads();
  }
  float* pr = a.part + (size_t)blockIdx.x * SQ_ROW;
  for (int e = tid; e < 9 * C * C; e += SQ_THREADS) pr[e] = red[e];
  __syncthreads();
  red[tid] = bsum;   // zero in the threads that staged no dout
  __syncthreads();
  if (tid < C) {
    float s = red[tid];
    for (int k = 1; k < 16; ++k) s += red[tid + 32 * k];
    pr[9 * C * C + tid] = s;
  }
}

// A 32-channel tensor against one of few channels (the first layer's input, the head's
// output gradient): the columns of D are the (tap, channel) pairs, t CN + c, padded to
// 32 or 64, so one product of K = 16 covers all taps.  The few channels are staged as
// three copies shifted by one pixel each, so that every tap's 8 pixels are aligned.
// FLIP (head): wide = the layer's input x[p], thin = dy[p - d]; otherwise wide = dout[p],
// thin = x[p + d].  Bound by the read of the 32-channel tensor.
struct WgradThinArgs {
  const float* wide;    // [B][H][W][32]
  const float* thin;    // [B][CN][H][W]
  float* part;
  int H, W, tiles_x, tiles_per_sample, total_tiles, tiles_per_wg;
};

template <int CN, bool FLIP>
__device__ __noinline__ void wgrad_thin_scalar(const WgradThinArgs& a, int t_begin, int t_end) {
  constexpr int NB = (9 * CN + 31) / 32, ROW = thin_row(CN, FLIP);
  float* pr = a.part + (size_t)blockIdx.x * ROW;
  for (int e = threadIdx.x; e < ROW; e += 256) {
    const int r = (e >> 6) & 15, lane = e & 63, nn = 32 * (e >> 10) + (lane & 31), t = nn / CN, c = nn % CN;
    const bool isb = e >= NB * C * C;
    const int rowc = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), bc = e - NB * C * C;
    float acc = 0.0f;
    if (isb || nn < 9 * CN)
      for (int tile = t_begin; tile < t_end; ++tile) {
        const int b = tile / a.tiles_per_sample, tr = tile - b * a.tiles_per_sample;
        for (int p = 0; p < GH * 16; ++p) {
          const int y = (tr / a.tiles_x) * GH + p / 16, x = (tr % a.tiles_x) * 16 + p % 16;
          if (y >= a.H || x >= a.W) continue;
          const float* wide = a.wide + (((size_t)b * a.H + y) * a.W + x) * C;
          if (isb) {
            acc += wide[bc];
            continue;
          }
          const int sg = FLIP ? -1 : 1, gy = y + sg * (t / 3 - 1), gx = x + sg * (t % 3 - 1);
          const bool in = gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
          acc = fmaf(wide[rowc], in ? a.thin[(((size_t)b * CN + c) * a.H + gy) * a.W + gx] : 0.0f, acc);
        }
      }
    pr[e] = acc;
  }
}

// Bias gradient of the head: its phase channel's sum is zero but for rounding (see the
// top of this file), so the order is fixed for good: runs of 16 x 16 tiles pixel by pixel,
// the runs in four strided sets.  A workgroup stages a tile's two planes and two lanes add
// them up (256 dependent additions per tile); these workgroups come behind the weight
// gradient's own, whose memory traffic hides the chains.
struct HeadBias {
  float* part;   // [workgroups][2]
  int first, tiles_x, tiles_per_sample, total_tiles, tiles_per_wg;   // first: of these workgroups
};
__device__ void head_bias(const float* __restrict__ dy, const HeadBias& hb, int H, int W, float4 (*v)[CT * CT / 4]) {
  const int wg = blockIdx.x - hb.first;
  const int t_begin = wg * hb.tiles_per_wg, t_end = min(hb.total_tiles, t_begin + hb.tiles_per_wg);
  float acc = 0.0f;
  for (int tile = t_begin; tile < t_end; ++tile) {
    const int b = tile / hb.tiles_per_sample, tr = tile - b * hb.tiles_per_sample;
    const int y = (tr / hb.tiles_x) * CT + threadIdx.x / CT, x = (tr % hb.tiles_x) * CT + threadIdx.x % CT;
    const bool in = y < H && x < W;
    const float* src = dy + ((size_t)b * 2 * H + y) * W + x;
    const float d0 = in ? src[0] : 0.0f, d1 = in ? src[(size_t)H * W] : 0.0f;
    __syncthreads();
    reinterpret_cast<float*>(v[0])[threadIdx.x] = d0;
    reinterpret_cast<float*>(v[1])[threadIdx.x] = d1;
    __syncthreads();
    if (threadIdx.x < 2)
#pragma unroll 8
      for (int i = 0; i < CT * CT / 4; ++i) {
        const float4 q = v[threadIdx.x][i];
        acc += q.x;
        acc += q.y;
        acc += q.z;
        acc += q.w;
      }
  }
  if (threadIdx.x < 2) hb.part[2 * wg + threadIdx.x] = acc;
}

template <int CN, bool FLIP>
__global__ __launch_bounds__(256) void wgrad_thin_kernel(WgradThinArgs a, HeadBias hb) {
  constexpr int NB = (9 * CN + 31) / 32, ROW = thin_row(CN, FLIP);
  constexpr int COPY = (GH + 2) * 32;                            // one shifted copy: 10 rows of 16 pixels
  __shared__ uint4 As4[3 * C * A_PITCH / 16];
  __shared__ uint4 Ts4[3 * CN * 3 * COPY / 16];
  __shared__ float red[NB * C * C > 256 ? NB * C * C : 256];
  if (FLIP && (int)blockIdx.x >= hb.first) {
    head_bias(a.thin, hb, a.H, a.W, reinterpret_cast<float4 (*)[CT * CT / 4]>(As4));
    return;
  }
  unsigned char* const As = reinterpret_cast<unsigned char*>(As4);
  unsigned char* const Ts = reinterpret_cast<unsigned char*>(Ts4);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, n = lane & 31;
  f32x16 acc[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[k][r] = 0.0f;
  float bsum = 0.0f, probe = 0.0f;
  const int t_begin = blockIdx.x * a.tiles_per_wg, t_end = min(a.total_tiles, t_begin + a.tiles_per_wg);
  const int sc = tid & 31, sg = tid >> 5;
  // byte offset of column n's pixels in the staged copies (part 0, row 0); columns past
  // 9 CN read column 0's and are dropped
  int toff[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int nn = 32 * k + n < 9 * CN ? 32 * k + n : 0, t = nn / CN, c = nn % CN;
    const int dy = FLIP ? 2 - t / 3 : t / 3, dx = FLIP ? 2 - t % 3 : t % 3;
    toff[k] = (c * 3 + dx) * COPY + dy * 32 + h * 16;
  }
  for (int tile = t_begin; tile < t_end; ++tile) {
    const int b = tile / a.tiles_per_sample, tr = tile - b * a.tiles_per_sample;
    const int y0 = (tr / a.tiles_x) * GH, x0 = (tr % a.tiles_x) * 16;
    const float* wb = a.wide + (size_t)b * a.H * a.W * C;
    const float* tb = a.thin + (size_t)b * CN * a.H * a.W;
    float va[2][8];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = sg + 8 * k;
      load8<false>(wb, a.H, a.W, y0 + (i >> 1), x0 + 8 * (i & 1), sc, 8, va[k]);
    }
    // groups of 8 pixels: channel, copy dx, row, half
    for (int i = tid; i < CN * 3 * (GH + 2) * 2; i += 256) {
      const int half = i & 1, row = (i >> 1) % (GH + 2), cd = (i >> 1) / (GH + 2), c = cd / 3, dx = cd - 3 * c;
      const int gy = y0 + row - 1;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int gx = x0 + 8 * half + j + dx - 1;
        v[j] = (gy >= 0 && gy < a.H && gx >= 0 && gx < a.W) ? tb[((size_t)c * a.H + gy) * a.W + gx] : 0.0f;
      }
      uint4 s[3];
      split8(v, s, probe);
#pragma unroll
      for (int q = 0; q < 3; ++q)
        *reinterpret_cast<uint4*>(Ts + (q * CN * 3 + cd) * COPY + row * 32 + half * 16) = s[q];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = sg + 8 * k;
      uint4 s[3];
      split8(va[k], s, probe);
#pragma unroll
      for (int q = 0; q < 3; ++q)
        *reinterpret_cast<uint4*>(As + (q * C + sc) * A_PITCH + 16 * i) = s[q];
      if constexpr (!FLIP)
        bsum += ((va[k][0] + va[k][1]) + (va[k][2] + va[k][3])) + ((va[k][4] + va[k][5]) + (va[k][6] + va[k][7]));
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int row = 2 * wave + k;
      uint4 g[3];
#pragma unroll
      for (int q = 0; q < 3; ++q)
        g[q] = *reinterpret_cast<const uint4*>(As + (q * C + n) * A_PITCH + row * 32 + h * 16);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        uint4 x[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
          x[q] = *reinterpret_cast<const uint4*>(Ts + q * CN * 3 * COPY + toff[nb] + row * 32);
        add_products(g, x, acc[nb]);
      }
    }
    __syncthreads();
  }
  if (__syncthreads_or(!(probe == 0.0f))) {
    wgrad_thin_scalar<CN, FLIP>(a, t_begin, t_end);
    return;
  }
  for (int w = 0; w < 4; ++w) {
    if (wave == w)
#pragma unroll
      for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float* d = red + (k * 16 + r) * 64 + lane;
          *d = w ? *d + acc[k][r] : acc[k][r];
        }
    __syncthreads();
  }
  float* pr = a.part + (size_t)blockIdx.x * ROW;
  for (int e = tid; e < NB * C * C; e += 256) pr[e] = red[e];
  if constexpr (!FLIP) {
    __syncthreads();
    red[tid] = bsum;
    __syncthreads();
    if (tid < C) {
      float s = red[tid];
      for (int k = 1; k < 8; ++k) s += red[tid + 32 * k];
      pr[NB * C * C + tid] = s;
    }
  }
}

// grad = sum of the part rows, from fragment order to the layer's parameter order:
// column e of a row is (t, r, lane) of a square layer, (block, r, lane) of a thin one,
// then (not the head) the bias.  64 columns per workgroup, 16 strided row sets combined in order.
// KIND 0: square; 1: first layer (CN input channels); 2: head (CN output channels).
template <int KIND>
__global__ __launch_bounds__(1024) void rows_sum_kernel(const float* __restrict__ part, int n_rows, int row_len,
                                                        int n_w, int cn, float* __restrict__ grad,
                                                        const float* __restrict__ bias_part, int bias_rows) {
  __shared__ float red[16][64];
  if (KIND == 2 && blockIdx.x == gridDim.x - 1) {   // the head's bias, see head_bias
    const int j = threadIdx.x & 1, q = threadIdx.x >> 1;
    if (q < 4) {
      float acc = 0.0f;
#pragma unroll 16
      for (int r = q; r < bias_rows; r += 4) acc += bias_part[2 * r + j];
      red[q][j] = acc;
    }
    __syncthreads();
    if (q == 0) grad[2 * C * 9 + j] = ((red[0][j] + red[1][j]) + red[2][j]) + red[3][j];
    return;
  }
  const int jj = threadIdx.x & 63, s = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + jj;
  float acc = 0.0f;
  if (e < row_len)
#pragma unroll 8
    for (int r = s; r < n_rows; r += 16) acc += part[(size_t)r * row_len + e];
  red[s][jj] = acc;
  __syncthreads();
  if (s || e >= row_len) return;
  acc = red[0][jj];
#pragma unroll
  for (int k = 1; k < 16; ++k) acc += red[k][jj];
  if (e >= n_w) {
    grad[(KIND == 0 ? 9 * C * C : 9 * C * cn) + e - n_w] = acc;
    return;
  }
  const int r = (e >> 6) & 15, lane = e & 63, row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  if (KIND == 0) {
    grad[(row * C + (lane & 31)) * 9 + (e >> 10)] = acc;
  } else {
    const int nn = 32 * (e >> 10) + (lane & 31), t = nn / cn, c = nn % cn;
    if (nn < 9 * cn) grad[(KIND == 1 ? (row * cn + c) : (c * C + row)) * 9 + t] = acc;
  }
}

// ---------------------------------------------------------------------------
// Compute copies of the weights (all layers in one launch)
// ---------------------------------------------------------------------------
// Forward, per 32 -> 32 layer: [pair of chunks of four input channels][product p][half of co][lane]
// float2, lane (kk, n) holding the weights of step 4 p + kk (channel, tap) and co = 16 half + n in
// both chunks.  Backward-
// data: fragments [tap][half of its input channels][part][lane] of eight bf16 values, lane
// (h, co) holding input channels 16 half + 8 h + (0..7).
__global__ __launch_bounds__(256) void prep_kernel(PrepArgs a) {
  constexpr int NF = 3 * FWD_VECS, NB = 3 * 18 * 64;
  const int i = blockIdx.x * 256 + threadIdx.x;
  bool bad = false;
  if (i < NF) {
    const int layer = i / FWD_VECS, e = i - layer * FWD_VECS, lane = e & 63, half = (e >> 6) & 1, gp = e / FWD_TAPS;
    const int st = 4 * ((e >> 7) % 9) + (lane >> 4), c = st / 9, t = st - 9 * c, co = 16 * half + (lane & 15);
    const float* w = a.p + a.off_sq[layer] + (co * C + 8 * gp + c) * 9 + t;
    float2 v = make_float2(w[0], w[36]);
    if (a.bf16) v = make_float2(round_bf16(v.x), round_bf16(v.y));
    a.fwd[i] = v;
  } else if (i < NF + NB) {
    const int j0 = i - NF, layer = j0 / (18 * 64), e = j0 - layer * (18 * 64), step = e >> 6, lane = e & 63;
    const int t = step >> 1, k0 = 16 * (step & 1) + 8 * (lane >> 5), co = lane & 31;
    const float* w = a.p + a.off_sq[layer];
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = w[((k0 + j) * C + co) * 9 + 8 - t];
      if (a.bf16) v[j] = round_bf16(v[j]);
    }
    uint4 s[3];
    float probe = 0.0f;
    split8(v, s, probe);
    bad = !(probe == 0.0f);
    const int ws = a.bf16 ? 1 : 3;
    uint4* dst = a.frag + (size_t)layer * FRAG_VECS;
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q < ws) dst[(step * ws + q) * 64 + lane] = s[q];
  } else {
    // first layer as it is; head as [c][t][o] and, for backward-data, [c][o][8 - t]
    const int j = i - NF - NB, n0 = C * a.cin * 9, n4 = 2 * C * 9;
    if (j < n0) {
      const float v = a.p[a.off_first + j];
      a.first[j] = a.bf16 ? round_bf16(v) : v;
    } else if (j < n0 + n4) {
      const int q = j - n0, o = q / (C * 9), c = (q / 9) % C, t = q % 9;
      float v = a.p[a.off_head + q];
      v = a.bf16 ? round_bf16(v) : v;
      a.head[(c * 9 + t) * 2 + o] = v;
      a.head_t[(c * 2 + o) * 9 + 8 - t] = v;
    }
  }
  if (bad) atomicOr(a.wbad, 1);
}


template <int MODE>
hipError_t conv32_t(bool bf16, const Conv32Args& a, int batch, hipStream_t s) {
  const int tx = (a.W + CT - 1) / CT, ty = (a.H + CT - 1) / CT, total = tx * ty * batch;
  const dim3 grid(std::min(total, 512));
  if (bf16) hipLaunchKernelGGL((conv32_kernel<MODE, 1>), grid, dim3(256), 0, s, a, tx, ty, total);
  else hipLaunchKernelGGL((conv32_kernel<MODE, 3>), grid, dim3(256), 0, s, a, tx, ty, total);
  return hipGetLastError();
}

struct Tiling {
  int tiles_x, per_sample, total, per_wg, wgs;
};
Tiling wgrad_tiling(int batch, int H, int W, int most) {
  Tiling t;
  t.tiles_x = (W + 15) / 16;
  t.per_sample = t.tiles_x * ((H + GH - 1) / GH);
  t.total = batch * t.per_sample;
  t.per_wg = (t.total + most - 1) / most;
  t.wgs = (t.total + t.per_wg - 1) / t.per_wg;
  return t;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_prep(const PrepArgs& a, hipStream_t s) {
  const int n = 3 * FWD_VECS + 3 * 18 * 64 + C * a.cin * 9 + 2 * C * 9;
  hipLaunchKernelGGL(prep_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int P>
static void conv32_forward_t(bool up, const float* in, const float2* w, const float* bias, float* out, int batch, int H,
                             int W, hipStream_t s) {
  const int tx = (W + CT - 1) / CT, ty = (H + 4 * P - 1) / (4 * P), total = tx * ty * batch;
  const dim3 grid(P == 4 ? std::min(total, 512) : total);
  if (up)
    hipLaunchKernelGGL((conv32_forward_kernel<true, P>), grid, dim3(256), 0, s, in, w, bias, out, H, W, tx, ty, total);
  else
    hipLaunchKernelGGL((conv32_forward_kernel<false, P>), grid, dim3(256), 0, s, in, w, bias, out, H, W, tx, ty, total);
}

hipError_t launch_conv32(bool up, const float* in, const float2* w, const float* bias, float* out, int batch, int H,
                         int W, hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1 || (up && ((H | W) & 1))) return hipErrorInvalidValue;
  // the fewest rows per workgroup that still give every CU at most one (see the kernel)
  const long tiles = (long)batch * ((H + CT - 1) / CT) * ((W + CT - 1) / CT);
  if (tiles <= 64) conv32_forward_t<1>(up, in, w, bias, out, batch, H, W, s);
  else if (tiles <= 128) conv32_forward_t<2>(up, in, w, bias, out, batch, H, W, s);
  else conv32_forward_t<4>(up, in, w, bias, out, batch, H, W, s);
  return hipGetLastError();
}

hipError_t launch_conv32_backward(bool up, bool bf16, const float* in, const uint4* frag, const float* w, float* out,
                                  const float* omask, const int* wbad, int batch, int H, int W, hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1 || (up && ((H | W) & 1))) return hipErrorInvalidValue;
  const Conv32Args a{in, frag, w, out, omask, wbad, H, W};
  return up ? conv32_t<3>(bf16, a, batch, s) : conv32_t<2>(bf16, a, batch, s);
}

hipError_t launch_conv_first(int ci, const float* in, const float* w, const float* bias, float* out, int batch, int H,
                             int W, hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1) return hipErrorInvalidValue;
  const dim3 grid((W + 15) / 16, (H + 3) / 4, batch);
#define CNN_FIRST(CI)                                                                                              \
  if (ci == CI) {                                                                                                  \
    hipLaunchKernelGGL((conv_thin_kernel<CI, false>), grid, dim3(256), 0, s, in, w, bias, out, nullptr, H, W);     \
    return hipGetLastError();                                                                                      \
  }
  CNN_FIRST(1)
  CNN_FIRST(3)
  CNN_FIRST(4)
#undef CNN_FIRST
  return hipErrorInvalidValue;
}

hipError_t launch_conv_head(const float* in, const float* w, const float* bias, float* out, int batch, int H, int W,
                            hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(conv_head_kernel, dim3((W + CT - 1) / CT, (H + CT - 1) / CT, batch), dim3(256), 0, s, in, w, bias,
                     out, H, W);
  return hipGetLastError();
}

hipError_t launch_conv_head_backward(const float* dy, const float* w, float* out, const float* omask, int batch,
                                     int H, int W, hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL((conv_thin_kernel<2, true>), dim3((W + 15) / 16, (H + 3) / 4, batch), dim3(256), 0, s, dy, w,
                     nullptr, out, omask, H, W);
  return hipGetLastError();
}

hipError_t launch_wgrad32(bool up, const float* in, const float* dout, float* part, float* grad, int batch, int H,
                          int W, hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1 || (up && ((H | W) & 1))) return hipErrorInvalidValue;
  const Tiling t = wgrad_tiling(batch, H, W, WGRAD_MAX_WORKGROUPS / 2);   // one workgroup per CU
  const Wgrad32Args a{in, dout, part, H, W, t.tiles_x, t.per_sample, t.total, t.per_wg};
  const void* k = up ? (const void*)wgrad32_kernel<true> : (const void*)wgrad32_kernel<false>;
  const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * SQ_LDS);
  if (e != hipSuccess) return e;
  if (up) hipLaunchKernelGGL(wgrad32_kernel<true>, dim3(t.wgs), dim3(SQ_THREADS), 2 * SQ_LDS, s, a);
  else hipLaunchKernelGGL(wgrad32_kernel<false>, dim3(t.wgs), dim3(SQ_THREADS), 2 * SQ_LDS, s, a);
  hipLaunchKernelGGL(rows_sum_kernel<0>, dim3((SQ_ROW + 63) / 64), dim3(1024), 0, s, (const float*)part, t.wgs, SQ_ROW,
                     9 * C * C, C, grad, (const float*)nullptr, 0);
  return hipGetLastError();
}

hipError_t launch_wgrad_first(int ci, const float* in, const float* dout, float* part, float* grad, int batch, int H,
                              int W, hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1) return hipErrorInvalidValue;
  const Tiling t = wgrad_tiling(batch, H, W, WGRAD_MAX_WORKGROUPS);
  const WgradThinArgs a{dout, in, part, H, W, t.tiles_x, t.per_sample, t.total, t.per_wg};
  const int row = thin_row(ci, false);
#define CNN_WF(CI) \
  if (ci == CI) hipLaunchKernelGGL((wgrad_thin_kernel<CI, false>), dim3(t.wgs), dim3(256), 0, s, a, HeadBias{});
  CNN_WF(1) else CNN_WF(3) else CNN_WF(4) else return hipErrorInvalidValue;
#undef CNN_WF
  hipLaunchKernelGGL(rows_sum_kernel<1>, dim3((row + 63) / 64), dim3(1024), 0, s, (const float*)part, t.wgs, row,
                     row - C, ci, grad, (const float*)nullptr, 0);
  return hipGetLastError();
}

hipError_t launch_wgrad_head(const float* in, const float* dy, float* part, float* grad, int batch, int H, int W,
                             hipStream_t s) {
  if (batch < 1 || H < 1 || W < 1) return hipErrorInvalidValue;
  const Tiling t = wgrad_tiling(batch, H, W, WGRAD_MAX_WORKGROUPS);
  const WgradThinArgs a{in, dy, part, H, W, t.tiles_x, t.per_sample, t.total, t.per_wg};
  const int row = thin_row(2, true);
  // the bias: 16 x 16 tiles, its rows behind the weights' (at most 512 of 1024 floats)
  HeadBias hb;
  hb.part = part + (size_t)WGRAD_MAX_WORKGROUPS * row;
  hb.first = t.wgs;
  hb.tiles_x = (W + CT - 1) / CT;
  hb.tiles_per_sample = hb.tiles_x * ((H + CT - 1) / CT);
  hb.total_tiles = batch * hb.tiles_per_sample;
  hb.tiles_per_wg = (hb.total_tiles + WGRAD_MAX_WORKGROUPS - 1) / WGRAD_MAX_WORKGROUPS;
  const int wgs = (hb.total_tiles + hb.tiles_per_wg - 1) / hb.tiles_per_wg;
  hipLaunchKernelGGL((wgrad_thin_kernel<2, true>), dim3(t.wgs + wgs), dim3(256), 0, s, a, hb);
  hipLaunchKernelGGL(rows_sum_kernel<2>, dim3((row + 63) / 64 + 1), dim3(1024), 0, s, (const float*)part, t.wgs, row,
                     row, 2, grad, (const float*)hb.part, wgs);
  return hipGetLastError();
}

}  // namespace cnn
