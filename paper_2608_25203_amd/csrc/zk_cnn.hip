// zk_cnn.hip -- kernels of the closure network (layouts in zk_cnn.hpp).
//
// Layers 2 and 3 (32 -> 32 channels, 3 x 3) are implicit GEMMs on the
// gfx950 matrix cores: v_mfma_f32_32x32x16_bf16 with the 32 output channels
// as the M dimension, 32 pixels of one row as N, and K = 9 taps x 32 input
// channels in chunks of 16.  Operand lane layout of that instruction: lane l
// holds A[l % 32][8 (l / 32) + 0..7] and B[8 (l / 32) + 0..7][l % 32]; the
// 16 accumulators of lane l hold D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
// The weight gradients of layers 1 to 3 are GEMMs with K = pixels on the same
// instruction.  Layer 1 (3 -> 32) runs on the same instruction with K = 9
// taps x 4 channels (channel 3 and taps 9..11 zero) in three chunks.  Layer 4
// (32 -> 1) is split in two: the layer-3 kernel turns each pixel's 32
// activations into the 9 per-tap partial sums t[p][tap] = sum_c W4[tap][c]
// a3[p][c] (two more MFMAs, taps as the M dimension), and a small kernel sums
// y[p] = b4 + sum_tap t[p + off(tap)][tap].  GELU uses the erf
// approximation 7.1.26 of Abramowitz and Stegun (absolute error <= 1.5e-7,
// far below the bf16 rounding of the activations), branch-free.  Layer 4's
// backward pass runs on the vector ALUs.  Every kernel indexes only inside
// the buffers described in zk_cnn.hpp for the geometry it is given (checked
// by the host before launch); periodic wrap-around adds or subtracts one
// period (every offset is a single pixel).
#include <algorithm>

#include "zk_cnn.hpp"

namespace zk {
namespace cnn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// round to nearest even (the hardware conversion, v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// Standard normal CDF Phi(z) = (1 + erf(z / sqrt 2)) / 2 and e = exp(-z^2 / 2),
// with erf(a) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-a^2),
// t = 1 / (1 + p a), a >= 0 (Abramowitz and Stegun 7.1.26), odd in a.
__device__ __forceinline__ float norm_cdf(float z, float &e) {
  const float u = z * 0.70710678118654752f;
  const float a = fabsf(u);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, a, 1.0f));
  const float poly =
      t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
  e = __builtin_amdgcn_exp2f(-1.44269504088896341f * a * a);
  return fmaf(0.5f, copysignf(fmaf(-poly, e, 1.0f), u), 0.5f);
}
__device__ __forceinline__ float gelu(float z) {
  float e;
  return z * norm_cdf(z, e);
}
__device__ __forceinline__ float gelu_d(float z) {  // Phi(z) + z phi(z)
  float e;
  const float c = norm_cdf(z, e);
  return fmaf(z * 0.39894228040143268f, e, c);
}
// i in [-n, 2n) wrapped into [0, n): every wrapped index here is a grid
// index plus or minus one
__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }
__device__ __forceinline__ f32x16 mfma(u16x8 a, u16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                  0, 0);
}

__global__ __launch_bounds__(256) void pack_kernel(const float *__restrict__ smp, uint16_t *__restrict__ xin, int H,
                                                   int W, long long P) {
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  if (p >= P) return;
  const long long hw = (long long)H * W;
  const long long b = p / hw, r = p % hw;
  u16x4 v;
  v[0] = f2bf(smp[(b * 4 + 0) * hw + r]);
  v[1] = f2bf(smp[(b * 4 + 1) * hw + r]);
  v[2] = f2bf(smp[(b * 4 + 2) * hw + r]);
  v[3] = 0;
  *reinterpret_cast<u16x4 *>(xin + p * 4) = v;
}

// ---- layer 1: 3 -> 32 on MFMA --------------------------------------------------
// Each wavefront computes 32 pixels of one row (N) x 32 output channels (M);
// K = tap * 4 + channel over 48 (three chunks of 16), so a lane's 8 K values
// of a chunk are two taps' 4-channel pixel words (8 bytes each).  Block: 4
// wavefronts side by side along x.
__global__ __launch_bounds__(256) void conv1_kernel(const uint16_t *__restrict__ xin, const uint16_t *__restrict__ w1m,
                                                    const float *__restrict__ b1, float *__restrict__ z1,
                                                    uint16_t *__restrict__ a1, int H, int W) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  const int x = blockIdx.x * 128 + 32 * wv + col;
  if (blockIdx.x * 128 + 32 * wv >= W) return;  // W % 32 == 0: whole wavefronts
  const int y = blockIdx.y;
  const long long b = blockIdx.z;
  f32x16 acc = {};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const u16x8 wa = *reinterpret_cast<const u16x8 *>(w1m + col * 48 + 16 * q + 8 * half);
    u16x8 bv = {};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int t = 4 * q + 2 * half + j;
      if (t < 9) {
        const int yy = wrap(y + t / 3 - 1, H), xx = wrap(x + t % 3 - 1, W);
        const u16x4 v = *reinterpret_cast<const u16x4 *>(xin + ((b * H + yy) * W + xx) * 4);
#pragma unroll
        for (int k = 0; k < 4; ++k) bv[4 * j + k] = v[k];
      }
    }
    acc = mfma(wa, bv, acc);
  }
  const long long pix = (b * H + y) * (long long)W + x;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int c0 = 8 * g + 4 * half;
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = acc[4 * g + k] + b1[c0 + k];
    if (z1) *reinterpret_cast<float4 *>(z1 + pix * CH + c0) = make_float4(v[0], v[1], v[2], v[3]);
    u16x4 o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = f2bf(gelu(v[k]));
    *reinterpret_cast<u16x4 *>(a1 + pix * CH + c0) = o;
  }
}

// ---- layers 2, 3: 32 -> 32 on MFMA ------------------------------------------------
// Block: 4 wavefronts side by side along x (32 pixels each), `rows` rows
// (chosen by the host so that one round of blocks fills the chip).  Input
// rows (y-1, y, y+1) over kConvTileX + 2 pixels sit in a ring of four LDS
// slots; row y+2 is fetched into registers while row y is computed and
// written to the free slot afterwards, so one barrier per row covers both.
// The weights of the wavefront's A operand stay in registers.
constexpr int kLdsPx = kConvTileX + 2;
constexpr int kPxStride = 40;  // uint16 per pixel in LDS (32 + 8 padding: 80-byte rows)
constexpr int kRing = 4;
constexpr int kFetch = (kLdsPx * 4 + 255) / 256;  // 16-byte pieces of a ring row per thread

// Modes: forward (out = bf16(GELU(z)), z optional); forward of the last
// hidden layer, which writes layer 4's per-tap partial sums taps[p][12] (taps
// 0..8; the bf16 activations of the lane's 16 channels are the B operand of
// two MFMAs against W4, its rows the taps) in place of out; backward-data (out = bf16(conv'(din) * GELU'(zprev))).
enum ConvMode { kFwd = 0, kFwdTaps = 1, kBwd = 2 };

template <int MODE>
__global__ __launch_bounds__(256) void conv32_kernel(const uint16_t *__restrict__ in, const uint16_t *__restrict__ wk,
                                                     const float *__restrict__ bias, const float *__restrict__ zprev,
                                                     float *__restrict__ zout, uint16_t *__restrict__ out,
                                                     const uint16_t *__restrict__ w4m, float *__restrict__ taps, int H,
                                                     int W, int rows) {
  constexpr bool BWD = MODE == kBwd;
  __shared__ __attribute__((aligned(16))) uint16_t ring[kRing][kLdsPx * kPxStride];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  const int x0 = blockIdx.x * kConvTileX;
  const int y0 = blockIdx.y * rows;
  const int y1 = min(H, y0 + rows);
  const long long b = blockIdx.z;
  const bool active = x0 + 32 * wv < W;  // W % 32 == 0
  // ring pixels the active wavefronts read (32 per wavefront plus one on each side)
  const int npx = min(kLdsPx, W - x0 + 2);

  u16x8 wa[9][2];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      wa[t][q] = *reinterpret_cast<const u16x8 *>(wk + (col * 9 + t) * CH + 16 * q + 8 * half);

  // thread piece s: pixel p = (tid + 256 s) / 4 of the ring row, channels 8 q .. 8 q + 7
  auto fetch = [&](u16x8 (&r)[kFetch], int yy) {
    const uint16_t *src = in + ((b * H + wrap(yy, H)) * (long long)W) * CH;
#pragma unroll
    for (int s = 0; s < kFetch; ++s) {
      const int i = tid + 256 * s, p = i >> 2, q = i & 3;
      if (p < npx) r[s] = *reinterpret_cast<const u16x8 *>(src + (long long)wrap(x0 - 1 + p, W) * CH + q * 8);
    }
  };
  auto put = [&](const u16x8 (&r)[kFetch], int slot) {
#pragma unroll
    for (int s = 0; s < kFetch; ++s) {
      const int i = tid + 256 * s, p = i >> 2, q = i & 3;
      if (p < npx) *reinterpret_cast<u16x8 *>(&ring[slot][p * kPxStride + q * 8]) = r[s];
    }
  };

  {
    u16x8 r0[kFetch], r1[kFetch], r2[kFetch];
    fetch(r0, y0 - 1);
    fetch(r1, y0);
    fetch(r2, y0 + 1);
    put(r0, 0);
    put(r1, 1);
    put(r2, 2);
  }
  __syncthreads();
  u16x8 pre[kFetch];
  for (int y = y0; y < y1; ++y) {
    const int j = y - y0;
    const bool next = y + 1 < y1;  // row y + 1 of this block needs input row y + 2
    if (next) fetch(pre, y + 2);
    if (active) {
      f32x16 acc = {};
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const uint16_t *rp = ring[(j + u) % kRing];
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const u16x8 bv = *reinterpret_cast<const u16x8 *>(rp + (32 * wv + col + v) * kPxStride + 16 * q + 8 * half);
            acc = mfma(wa[u * 3 + v][q], bv, acc);
          }
      }
      const long long pix = (b * H + y) * (long long)W + x0 + 32 * wv + col;
      u16x8 act[2];  // kFwdTaps: this lane's bf16 activations as the B operand, chunk q = groups 2q, 2q + 1
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c0 = 8 * g + 4 * half;
        float v[4] = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        if constexpr (!BWD) {
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] += bias[c0 + k];
          if (zout) *reinterpret_cast<float4 *>(zout + pix * CH + c0) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = gelu(v[k]);
        } else {
          const float4 zp = *reinterpret_cast<const float4 *>(zprev + pix * CH + c0);
          v[0] *= gelu_d(zp.x);
          v[1] *= gelu_d(zp.y);
          v[2] *= gelu_d(zp.z);
          v[3] *= gelu_d(zp.w);
        }
        u16x4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = f2bf(v[k]);
        if constexpr (MODE != kFwdTaps) *reinterpret_cast<u16x4 *>(out + pix * CH + c0) = o;
        if constexpr (MODE == kFwdTaps) {
#pragma unroll
          for (int k = 0; k < 4; ++k) act[g / 2][4 * (g % 2) + k] = o[k];
        }
      }
      if constexpr (MODE == kFwdTaps) {
        f32x16 tp = {};
#pragma unroll
        for (int q = 0; q < 2; ++q)
          tp = mfma(*reinterpret_cast<const u16x8 *>(w4m + (col * 2 + q) * 16 + 8 * half), act[q], tp);
        // rows 4 half + 0..3 (taps 0..7) and, for half 0, row 8 (tap 8)
        *reinterpret_cast<float4 *>(taps + pix * 12 + 4 * half) = make_float4(tp[0], tp[1], tp[2], tp[3]);
        if (half == 0) taps[pix * 12 + 8] = tp[4];
      }
    }
    // the slot of input row y - 1, last read in the previous row's step
    if (next) put(pre, (j + 3) % kRing);
    __syncthreads();
  }
}

// ---- layer 4: 32 -> 1, from the per-tap partial sums ---------------------------------
__global__ __launch_bounds__(256) void conv4_kernel(const float *__restrict__ taps, const float *__restrict__ b4,
                                                    float *__restrict__ y, int H, int W, long long P) {
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  if (p >= P) return;
  const int x = (int)(p % W);
  const long long r = p / W;
  const int yy0 = (int)(r % H);
  const long long b = r / H;
  float acc = b4[0];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const int yy = wrap(yy0 + t / 3 - 1, H), xx = wrap(x + t % 3 - 1, W);
    acc += taps[((b * H + yy) * W + xx) * 12 + t];
  }
  y[p] = acc;
}

// ---- loss: masked mean squared error -----------------------------------------------
__global__ __launch_bounds__(256) void loss_kernel(const float *__restrict__ y, const float *__restrict__ smp, int halo,
                                                   double inv_n, uint16_t *__restrict__ dz4,
                                                   double *__restrict__ partial, int H, int W, long long P) {
  __shared__ double red[256];
  double s = 0.0;
  const long long hw = (long long)H * W;
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < P; p += (long long)gridDim.x * 256) {
    const int x = (int)(p % W);
    const long long r = p / W;
    const int yy = (int)(r % H);
    const long long b = r / H;
    const bool in = yy >= halo && yy < H - halo && x >= halo && x < W - halo;
    const double d = in ? (double)y[p] - (double)smp[(b * 4 + 3) * hw + (long long)yy * W + x] : 0.0;
    dz4[p] = f2bf((float)(2.0 * d * inv_n));
    s += d * d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// ---- layer 4 backward: dz3 = (W4^T dz4) * GELU'(z3) and dW4, db4 -----------------------
// One pass over z3 serves both: pixel p's neighbours d[t] = dz4[p - off(t)]
// that backward-data weights with W4 are also the factors of its activations
// a3[p] in dW4[c][t] = sum_p a3[p][c] d[t], and a3 = bf16(GELU(z3)) comes from
// the same normal CDF as GELU'(z3), so the forward pass stores no a3.  Thread:
// 4 channels of every 128 gridDim.x-th pixel, its 36 weights and 36 sums in
// registers.  Bounded by memory (128 B read, 64 B written a pixel): 23 us at 16
// x 128 x 128 pixels, where backward-data alone took 23 us and a weight-gradient
// kernel with one channel and tap a thread 420 us.
constexpr int kL4Threads = 1024;
__global__ __launch_bounds__(kL4Threads) void conv4_bwd_kernel(const uint16_t *__restrict__ dz4,
                                                               const float *__restrict__ w4f,
                                                               const float *__restrict__ z3,
                                                               uint16_t *__restrict__ dz3, float *__restrict__ part,
                                                               int H, int W, int P) {
  constexpr int NWV = kL4Threads / 64;
  __shared__ float red[NWV][PART4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c0 = 4 * (tid & 7);
  float w[9][4], acc[9][4], accb = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[t][k] = w4f[t * CH + c0 + k];
      acc[t][k] = 0.f;
    }
  for (int p = blockIdx.x * (kL4Threads / 8) + (tid >> 3); p < P; p += gridDim.x * (kL4Threads / 8)) {
    const int r = p / W, x = p - r * W;
    const int y = r % H, row0 = r - y;  // row0: first row of the image, in rows
    const float4 zp = *reinterpret_cast<const float4 *>(z3 + (long long)p * CH + c0);
    const float zz[4] = {zp.x, zp.y, zp.z, zp.w};
    float d[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)  // output pixel p - (u-1, v-1) read this pixel through tap (u, v)
      d[t] = bf2f(dz4[(long long)(row0 + wrap(y - t / 3 + 1, H)) * W + wrap(x - t % 3 + 1, W)]);
    accb += d[4];
    u16x4 o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float e;
      const float cdf = norm_cdf(zz[k], e);
      const float a = bf2f(f2bf(zz[k] * cdf));
      float s = 0.f;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        s += w[t][k] * d[t];
        acc[t][k] += a * d[t];
      }
      o[k] = f2bf(s * fmaf(zz[k] * 0.39894228040143268f, e, cdf));
    }
    *reinterpret_cast<u16x4 *>(dz3 + (long long)p * CH + c0) = o;
  }
  // the wavefront's 8 pixels, then the block's wavefronts, in a fixed order
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float v = acc[t][k];
      v += __shfl_xor(v, 8);
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 8) red[wv][t * CH + c0 + k] = v;
    }
  accb += __shfl_xor(accb, 8);
  accb += __shfl_xor(accb, 16);
  accb += __shfl_xor(accb, 32);
  if (lane == 0) red[wv][9 * CH] = accb;
  __syncthreads();
  if (tid < NW4 + NB4) {
    float v = 0.f;
    for (int k = 0; k < NWV; ++k) v += red[k][tid];
    part[(long long)blockIdx.x * kPartSlots + SLOT4 + tid] = v;
  }
}

// ---- weight gradients of layers 1, 2 and 3 on MFMA --------------------------------------
// dW[o][c][tap] = sum_p dz[p][o] in[p + off(tap)][c]: M = o, K = pixels,
// 16 at a time.  Both operands want 8 consecutive pixels of one channel per
// lane while memory holds pixels of 32 channels, so a wavefront copies its
// rows to LDS as they are (no transposing stores) and gathers an operand with
// 16-bit reads, 32 channels of one pixel a half wavefront: with 72 bytes a
// pixel the two halves (8 pixels apart) fall on different banks.  The three
// horizontal taps of a row are windows of the same 10 pixels, so a chunk of 16
// pixels takes 8 + 30 reads for 9 products.  A wavefront owns a strip of
// kSegPx pixels and walks down its rows with a ring of three input rows (the
// next row in registers), all in LDS of its own: no block barrier until the
// block sums its wavefronts' results.  At 16 x 128 x 128 pixels layers 2 and
// 3 take 19 us each (66 us with a block staging transposed copies by 2-byte
// stores behind two barriers a segment), layer 1 8.4 us (420 us on the vector
// ALUs); the bytes they read take 10 and 4 us.
constexpr int kDwWaves = 8;               // wavefronts per block
constexpr int kDwStride = 36;             // uint16 per pixel in LDS
constexpr int kDwPx = kSegPx + 2;         // pixels of an input row in LDS
constexpr int kDwFewestRows = 4;          // rows a wavefront walks at least

// Rows y0 .. y0 + nrows - 1 of one strip.
struct DwStrip {
  int b, y0, nrows, x0;
};
__device__ __forceinline__ DwStrip dw_strip(int item, int bands, int rows, int H, int W) {
  const int segs = W / kSegPx, s = item / bands, y0 = (item - s * bands) * rows;
  return {s / segs, y0, min(rows, H - y0), (s % segs) * kSegPx};
}
// Wavefront-private LDS: its operations complete in order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void put_pixel(uint16_t *dst, u16x8 v) {  // 8-byte aligned
  *reinterpret_cast<u16x4 *>(dst) = u16x4{v[0], v[1], v[2], v[3]};
  *reinterpret_cast<u16x4 *>(dst + 4) = u16x4{v[4], v[5], v[6], v[7]};
}

__global__ __launch_bounds__(64 * kDwWaves) void dw32_kernel(const uint16_t *__restrict__ dz,
                                                            const uint16_t *__restrict__ act,
                                                            float *__restrict__ part, int slot0, int items, int bands,
                                                            int rows, int H, int W) {
  constexpr int ROW = kDwPx * kDwStride, LDS1 = 3 * ROW + kSegPx * kDwStride;  // uint16 per wavefront
  __shared__ __attribute__((aligned(16))) uint16_t smem[kDwWaves * LDS1];
  static_assert(kDwWaves * LDS1 * 2 >= (kDwWaves / 2) * 9 * 1024 * 4, "the final sums fit");
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  uint16_t *ring = smem + wv * LDS1, *dzs = ring + 3 * ROW;
  f32x16 acc[9] = {};
  float accb = 0.f;
  for (int item = blockIdx.x + gridDim.x * wv; item < items; item += gridDim.x * kDwWaves) {
    const DwStrip st = dw_strip(item, bands, rows, H, W);
    const long long img = (long long)st.b * H;
    // 16-byte pieces: pixel i / 4, channels 8 (i % 4) ..; an input row holds pixels x0 - 1 .. x0 + kSegPx
    u16x8 ra[5], rd[4];
    auto fetch_a = [&](int yy) {
      const uint16_t *src = act + (img + wrap(yy, H)) * W * CH;
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int i = lane + 64 * s;
        if (i < 4 * kDwPx) ra[s] = *reinterpret_cast<const u16x8 *>(src + wrap(st.x0 - 1 + (i >> 2), W) * CH + (i & 3) * 8);
      }
    };
    auto put_a = [&](int slot) {
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int i = lane + 64 * s;
        if (i < 4 * kDwPx) put_pixel(ring + slot * ROW + (i >> 2) * kDwStride + (i & 3) * 8, ra[s]);
      }
    };
    auto fetch_d = [&](int y) {
      const uint16_t *src = dz + ((img + y) * W + st.x0) * CH;
#pragma unroll
      for (int s = 0; s < 4; ++s) rd[s] = *reinterpret_cast<const u16x8 *>(src + (lane + 64 * s) * 8);
    };
    fetch_a(st.y0 - 1);
    wave_sync();  // the previous strip's reads are done
    put_a(0);
    fetch_a(st.y0);
    put_a(1);
    fetch_a(st.y0 + 1);
    fetch_d(st.y0);
    for (int j = 0; j < st.nrows; ++j) {
      wave_sync();  // the previous row's reads are done
      put_a((j + 2) % 3);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int i = lane + 64 * s;
        put_pixel(dzs + (i >> 2) * kDwStride + (i & 3) * 8, rd[s]);
      }
      wave_sync();
      if (j + 1 < st.nrows) {
        fetch_a(st.y0 + j + 2);
        fetch_d(st.y0 + j + 1);
      }
#pragma unroll
      for (int kc = 0; kc < kSegPx / 16; ++kc) {
        const int px = 16 * kc + 8 * half;
        u16x8 av;
#pragma unroll
        for (int k = 0; k < 8; ++k) av[k] = dzs[(px + k) * kDwStride + col];
#pragma unroll
        for (int k = 0; k < 8; ++k) accb += bf2f(av[k]);
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          const uint16_t *rp = ring + ((j + u) % 3) * ROW + px * kDwStride + col;
          uint16_t w[10];
#pragma unroll
          for (int k = 0; k < 10; ++k) w[k] = rp[k * kDwStride];
#pragma unroll
          for (int v = 0; v < 3; ++v) {
            u16x8 bv;
#pragma unroll
            for (int k = 0; k < 8; ++k) bv[k] = w[v + k];
            acc[3 * u + v] = mfma(av, bv, acc[3 * u + v]);
          }
        }
      }
    }
  }
  // Block sum over wavefronts, in a fixed order: halve the wavefronts until one is left.
  accb += __shfl_xor(accb, 32);
  float *red = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int n = kDwWaves / 2; n > 0; n >>= 1) {
    __syncthreads();
    if (wv >= n && wv < 2 * n) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[((wv - n) * 144 + t * 16 + r) * 64 + lane] = acc[t][r];
    }
    __syncthreads();
    if (wv < n) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] += red[(wv * 144 + t * 16 + r) * 64 + lane];
    }
  }
  __syncthreads();
  if (lane < 32) red[wv * 32 + lane] = accb;
  __syncthreads();
  float *o = part + (long long)blockIdx.x * kPartSlots + slot0;
  if (wv == 0) {
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[t * 1024 + (8 * (r / 4) + 4 * half + r % 4) * 32 + col] = acc[t][r];
  }
  if (tid < 32) {
    float v = 0.f;
    for (int k = 0; k < kDwWaves; ++k) v += red[k * 32 + tid];
    o[9 * 1024 + tid] = v;
  }
}

// Layer 1: N = 9 taps x 3 channels (column 3 tap + c), column 27 a vector of
// ones (the bias), so one product a chunk.
__global__ __launch_bounds__(64 * kDwWaves) void dw1_kernel(const uint16_t *__restrict__ dz,
                                                           const uint16_t *__restrict__ xin,
                                                           float *__restrict__ part, int items, int bands, int rows,
                                                           int H, int W) {
  constexpr int ROW = kDwPx * 4, LDS1 = 3 * ROW + kSegPx * kDwStride;
  __shared__ __attribute__((aligned(16))) uint16_t smem[kDwWaves * LDS1 + 1024 * 2 * kDwWaves];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  uint16_t *ring = smem + wv * LDS1, *dzs = ring + 3 * ROW;
  const int tap = col < 27 ? col / 3 : 8, ch = col < 27 ? col % 3 : 3;  // columns from 27 on read channel 3
  const uint16_t fill = col == 27 ? 0x3f80 : 0;                         // bf16 one
  f32x16 acc = {};
  for (int item = blockIdx.x + gridDim.x * wv; item < items; item += gridDim.x * kDwWaves) {
    const DwStrip st = dw_strip(item, bands, rows, H, W);
    const long long img = (long long)st.b * H;
    u16x4 ra[2];
    u16x8 rd[4];
    auto fetch_a = [&](int yy) {
      const uint16_t *src = xin + (img + wrap(yy, H)) * W * 4;
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (lane + 64 * s < kDwPx) ra[s] = *reinterpret_cast<const u16x4 *>(src + wrap(st.x0 - 1 + lane + 64 * s, W) * 4);
    };
    auto put_a = [&](int slot) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (lane + 64 * s < kDwPx) *reinterpret_cast<u16x4 *>(ring + slot * ROW + (lane + 64 * s) * 4) = ra[s];
    };
    auto fetch_d = [&](int y) {
      const uint16_t *src = dz + ((img + y) * W + st.x0) * CH;
#pragma unroll
      for (int s = 0; s < 4; ++s) rd[s] = *reinterpret_cast<const u16x8 *>(src + (lane + 64 * s) * 8);
    };
    fetch_a(st.y0 - 1);
    wave_sync();  // the previous strip's reads are done
    put_a(0);
    fetch_a(st.y0);
    put_a(1);
    fetch_a(st.y0 + 1);
    fetch_d(st.y0);
    for (int j = 0; j < st.nrows; ++j) {
      wave_sync();  // the previous row's reads are done
      put_a((j + 2) % 3);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int i = lane + 64 * s;
        put_pixel(dzs + (i >> 2) * kDwStride + (i & 3) * 8, rd[s]);
      }
      wave_sync();
      if (j + 1 < st.nrows) {
        fetch_a(st.y0 + j + 2);
        fetch_d(st.y0 + j + 1);
      }
      const uint16_t *rp = ring + ((j + tap / 3) % 3) * ROW + (tap % 3) * 4 + ch;
#pragma unroll
      for (int kc = 0; kc < kSegPx / 16; ++kc) {
        const int px = 16 * kc + 8 * half;
        u16x8 av, bv;
#pragma unroll
        for (int k = 0; k < 8; ++k) av[k] = dzs[(px + k) * kDwStride + col];
#pragma unroll
        for (int k = 0; k < 8; ++k) bv[k] = col < 27 ? rp[(px + k) * 4] : fill;
        acc = mfma(av, bv, acc);
      }
    }
  }
  float *red = reinterpret_cast<float *>(smem + kDwWaves * LDS1);
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wv * 1024 + (8 * (r / 4) + 4 * half + r % 4) * 32 + col] = acc[r];
  __syncthreads();
  for (int i = tid; i < 1024; i += 64 * kDwWaves) {
    float v = 0.f;
    for (int k = 0; k < kDwWaves; ++k) v += red[k * 1024 + i];
    part[(long long)blockIdx.x * kPartSlots + SLOT1 + i] = v;
  }
}

// Sums the blocks' partial results of every layer and puts them in parameter
// order.  Block: 64 slots, 16 wavefronts of kPartBlocks / 16 partials each
// (5.6 us for all layers; one thread a slot summing all of them took 60 us a
// layer).
__global__ __launch_bounds__(1024) void reduce_kernel(const float *__restrict__ part, float *__restrict__ grad) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, i = blockIdx.x * 64 + lane;
  constexpr int N = kPartBlocks / 16;
  float v[N], s = 0.f;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = part[(long long)(wv * N + k) * kPartSlots + i];
#pragma unroll
  for (int k = 0; k < N; ++k) s += v[k];
  red[wv][lane] = s;
  __syncthreads();
  if (wv) return;
  s = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) s += red[k][lane];
  if (i < SLOT2) {  // layer 1: [co][3 tap + ci], column 27 the bias
    const int co = (i - SLOT1) / 32, n = (i - SLOT1) % 32;
    if (n < 27) grad[OFF_W1 + (co * 3 + n % 3) * 9 + n / 3] = s;
    else if (n == 27) grad[OFF_B1 + co] = s;
  } else if (i < SLOT4) {  // layers 2, 3: [tap][o][c], then the bias
    const bool l2 = i < SLOT3;
    const int k = i - (l2 ? SLOT2 : SLOT3);
    if (k < 9 * 1024) grad[(l2 ? OFF_W2 : OFF_W3) + (k % 1024) * 9 + k / 1024] = s;
    else grad[(l2 ? OFF_B2 : OFF_B3) + k - 9 * 1024] = s;
  } else {  // layer 4: [tap][c], then the bias
    const int k = i - SLOT4;
    if (k < NW4) grad[OFF_W4 + (k % CH) * 9 + k / CH] = s;
    else if (k == NW4) grad[OFF_B4] = s;
  }
}

__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                                                   const float *__restrict__ g, float lr, float b1, float b2, float eps,
                                                   float c1, float c2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= NPARAM) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ __launch_bounds__(256) void prep_kernel(const float *__restrict__ p, uint16_t *__restrict__ w1m,
                                                   uint16_t *__restrict__ w2f, uint16_t *__restrict__ w2b,
                                                   uint16_t *__restrict__ w3f, uint16_t *__restrict__ w3b,
                                                   float *__restrict__ w4f, uint16_t *__restrict__ w4m) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  // the zero slots of the MFMA operands (channel 3 and taps 9..11 of w1m; rows 9..31 of w4m)
  if (i < CH * 48 && (i % 4 == 3 || i % 48 >= 36)) w1m[i] = 0;
  if (i >= 9 * 32 && i < 32 * 32) w4m[i] = 0;
  if (i >= NPARAM) return;
  const uint16_t h = f2bf(p[i]);
  if (i >= OFF_W1 && i < OFF_W1 + NW1) {
    const int k = i - OFF_W1, co = k / 27, ci = (k / 9) % 3, t = k % 9;
    w1m[co * 48 + t * 4 + ci] = h;
  } else if ((i >= OFF_W2 && i < OFF_W2 + NW2) || (i >= OFF_W3 && i < OFF_W3 + NW3)) {
    const bool l2 = i < OFF_W2 + NW2;
    const int k = i - (l2 ? OFF_W2 : OFF_W3), o = k / (CH * 9), c = (k / 9) % CH, t = k % 9;
    (l2 ? w2f : w3f)[(o * 9 + t) * CH + c] = h;
    (l2 ? w2b : w3b)[(c * 9 + (8 - t)) * CH + o] = h;
  } else if (i >= OFF_W4 && i < OFF_W4 + NW4) {
    const int k = i - OFF_W4, c = k / 9, t = k % 9;
    w4f[t * CH + c] = bf2f(h);
    // MFMA operand: row t, chunk c / 16, K slot 8 h + j with c % 16 = 8 (j / 4) + 4 h + j % 4
    const int q = c / 16, hh = (c % 8) / 4, j = 4 * ((c % 16) / 8) + c % 4;
    w4m[(t * 2 + q) * 16 + 8 * hh + j] = h;
  }
}

unsigned blocks_for(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t pack_samples(const float *samples, uint16_t *xin, Geo g, hipStream_t s) {
  hipLaunchKernelGGL(pack_kernel, dim3(blocks_for(g.pixels())), dim3(256), 0, s, samples, xin, g.H, g.W, g.pixels());
  return hipGetLastError();
}
hipError_t conv1_fwd(const uint16_t *xin, const uint16_t *w1m, const float *b1, float *z1, uint16_t *a1, Geo g,
                     hipStream_t s) {
  const dim3 grid((g.W + 127) / 128, g.H, g.B);
  hipLaunchKernelGGL(conv1_kernel, grid, dim3(256), 0, s, xin, w1m, b1, z1, a1, g.H, g.W);
  return hipGetLastError();
}
// Rows per block of a layer-2/3 launch: enough that one round of resident
// blocks covers the grid (each block pays a three-row prologue), at least
// kConvRows.  `resident` = blocks of this kernel the whole chip holds at once.
template <int MODE>
int conv_rows(Geo g) {
  static int resident = 0;
  if (resident == 0) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, conv32_kernel<MODE>, 256, 0) != hipSuccess)
      cus = per_cu = 0;
    resident = cus > 0 && per_cu > 0 ? cus * per_cu : 1024;
  }
  const long long strips = (long long)g.B * ((g.W + kConvTileX - 1) / kConvTileX);  // blocks per row band
  const long long need = (strips * g.H + resident - 1) / resident;
  return (int)std::min<long long>(g.H, std::max<long long>(kConvRows, need));
}
template <int MODE>
hipError_t conv32_launch(const uint16_t *in, const uint16_t *wk, const float *bias, const float *zprev, float *z,
                         uint16_t *out, const uint16_t *w4m, float *taps, Geo g, hipStream_t s) {
  const int rows = conv_rows<MODE>(g);
  const dim3 grid((g.W + kConvTileX - 1) / kConvTileX, (g.H + rows - 1) / rows, g.B);
  hipLaunchKernelGGL(conv32_kernel<MODE>, grid, dim3(256), 0, s, in, wk, bias, zprev, z, out, w4m, taps, g.H, g.W,
                     rows);
  return hipGetLastError();
}
hipError_t conv32_fwd(const uint16_t *in, const uint16_t *wk, const float *bias, float *z, uint16_t *out, Geo g,
                      hipStream_t s) {
  return conv32_launch<kFwd>(in, wk, bias, nullptr, z, out, nullptr, nullptr, g, s);
}
hipError_t conv32_fwd_taps(const uint16_t *in, const uint16_t *wk, const float *bias, float *z, const uint16_t *w4m,
                           float *taps, Geo g, hipStream_t s) {
  return conv32_launch<kFwdTaps>(in, wk, bias, nullptr, z, nullptr, w4m, taps, g, s);
}
hipError_t conv32_bwd(const uint16_t *din, const uint16_t *wkt, const float *zprev, uint16_t *dout, Geo g,
                      hipStream_t s) {
  return conv32_launch<kBwd>(din, wkt, nullptr, zprev, nullptr, dout, nullptr, nullptr, g, s);
}
hipError_t conv4_fwd(const float *taps, const float *b4, float *y, Geo g, hipStream_t s) {
  hipLaunchKernelGGL(conv4_kernel, dim3(blocks_for(g.pixels())), dim3(256), 0, s, taps, b4, y, g.H, g.W, g.pixels());
  return hipGetLastError();
}
hipError_t loss_grad(const float *y, const float *samples, int halo, double inv_n, uint16_t *dz4, double *partial,
                     Geo g, hipStream_t s) {
  hipLaunchKernelGGL(loss_kernel, dim3(kLossBlocks), dim3(256), 0, s, y, samples, halo, inv_n, dz4, partial, g.H, g.W,
                     g.pixels());
  return hipGetLastError();
}
hipError_t conv4_bwd(const uint16_t *dz4, const float *w4f, const float *z3, uint16_t *dz3, float *part, Geo g,
                     hipStream_t s) {
  hipLaunchKernelGGL(conv4_bwd_kernel, dim3(kPartBlocks), dim3(kL4Threads), 0, s, dz4, w4f, z3, dz3, part, g.H, g.W,
                     (int)g.pixels());
  return hipGetLastError();
}
// Strips of kSegPx pixels, cut into bands of enough rows to give each wavefront one.
struct DwSplit {
  int items, bands, rows;
};
DwSplit dw_split(Geo g) {
  const long long strips = (long long)g.B * (g.W / kSegPx), waves = (long long)kPartBlocks * kDwWaves;
  const int rows = (int)std::min<long long>(g.H, std::max<long long>(kDwFewestRows, (strips * g.H + waves - 1) / waves));
  const int bands = (g.H + rows - 1) / rows;
  return {(int)(strips * bands), bands, rows};
}
hipError_t dw32(const uint16_t *dz, const uint16_t *a, float *part, int layer, Geo g, hipStream_t s) {
  const DwSplit d = dw_split(g);
  hipLaunchKernelGGL(dw32_kernel, dim3(kPartBlocks), dim3(64 * kDwWaves), 0, s, dz, a, part, layer == 2 ? SLOT2 : SLOT3,
                     d.items, d.bands, d.rows, g.H, g.W);
  return hipGetLastError();
}
hipError_t dw1(const uint16_t *dz1, const uint16_t *xin, float *part, Geo g, hipStream_t s) {
  const DwSplit d = dw_split(g);
  hipLaunchKernelGGL(dw1_kernel, dim3(kPartBlocks), dim3(64 * kDwWaves), 0, s, dz1, xin, part, d.items, d.bands, d.rows,
                     g.H, g.W);
  return hipGetLastError();
}
hipError_t reduce_parts(const float *part, float *grad, hipStream_t s) {
  hipLaunchKernelGGL(reduce_kernel, dim3(kPartSlots / 64), dim3(1024), 0, s, part, grad);
  return hipGetLastError();
}
hipError_t adam(float *p, float *m, float *v, const float *g, float lr, float b1, float b2, float eps, float c1,
                float c2, hipStream_t s) {
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(NPARAM)), dim3(256), 0, s, p, m, v, g, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}
hipError_t prep_weights(const float *p, uint16_t *w1m, uint16_t *w2f, uint16_t *w2b, uint16_t *w3f, uint16_t *w3b,
                        float *w4f, uint16_t *w4m, hipStream_t s) {
  hipLaunchKernelGGL(prep_kernel, dim3(blocks_for(NPARAM)), dim3(256), 0, s, p, w1m, w2f, w2b, w3f, w3b, w4f, w4m);
  return hipGetLastError();
}

}  // namespace cnn
}  // namespace zk
