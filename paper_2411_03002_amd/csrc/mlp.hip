// Learned precision indicator: per-atom features, a 4-64-64-64-1 tanh network trained in
// float32 (forward, backward, Adam) and evaluated with bfloat16 MFMA, and the switch from
// its prediction to an additional detection weight.
//
// The paper lets the detection argument of its switching function be replaced by another
// criterion (Appendix B, after eq. lambda_1_i); here the network predicts
// log(|F_ACE - F_EAM| + 1e-3) from [rho_EAM, min(CSP, 50), coordination (r < 3.08 A),
// |F_EAM|] and w0_extra = 1 - f_cut((yhat - tau_lo)/(tau_hi - tau_lo)) with
// yhat = exp(prediction) - 1e-3.  Atoms whose features lie outside the training range get
// w0_extra = 0, i.e. only the centro-symmetry criterion (the fallback).
#include <algorithm>
#include <cmath>
#include <cstring>

#include "common.h"
#include "device_util.h"

namespace apx {

constexpr int kH = 64;                 // hidden width
constexpr int kIn = 4;                 // inputs
constexpr int kOffW1 = 0;              // [64][4]
constexpr int kOffB1 = 256;
constexpr int kOffW2 = 320;            // [64][64]
constexpr int kOffB2 = 4416;
constexpr int kOffW3 = 4480;           // [64][64]
constexpr int kOffB3 = 8576;
constexpr int kOffW4 = 8640;           // [64]
constexpr int kOffB4 = 8704;
constexpr int kNParams = 8705;
constexpr float kCoordR2 = 3.08f * 3.08f;

struct Std4 {
  float mu[4], sd[4];
};

}  // namespace apx

struct apx_mlp {
  int device = 0;
  apx::DevBuf buf;    // params, m, v, loss, bf16 weights, sums of a training step
  float* params = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  float* loss = nullptr;
  float* sums = nullptr;         // [kPassBlocks][kSlabLd]
  unsigned short* wb = nullptr;  // bf16: W1 padded [64][16], W2 [64][64], W3 [64][64], W4 [64]
  bool wb_valid = false;
  long long step = 0;
  apx::Std4 st{};
  float fmin[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  float fmax[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
};

namespace apx {

// ----------------------------------------------------------------- features
template <int W>
__global__ void __launch_bounds__(64 * W) k_features(const double* __restrict__ pos, int n, BoxDev b,
                                                  const int* __restrict__ count, const int* __restrict__ idx,
                                                  int max_nb, const double* __restrict__ rho,
                                                  const double* __restrict__ csp, const double* __restrict__ f,
                                                  float* __restrict__ feat) {
  constexpr int kBatch = row_batch(W);
  const int row = row_atom<W>(xcd_block(blockIdx.x, gridDim.x)), wv = row_wave<W>();
  const int i = row < n ? row : n - 1;  // (a thread beyond the last atom repeats it)
  const double xi = pos[i], yi = pos[(size_t)n + i], zi = pos[2 * (size_t)n + i];
  int cnt = count[i];
  if (cnt > max_nb) cnt = max_nb;
  const double rc2 = 3.08 * 3.08;
  int coord = 0;
  for (int k0 = wv * kBatch; k0 < cnt; k0 += W * kBatch) {
    int jb[kBatch];
    double px[kBatch], py[kBatch], pz[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) jb[q] = k0 + q < cnt ? idx[(size_t)(k0 + q) * n + i] : i;
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      px[q] = pos[jb[q]];
      py[q] = pos[(size_t)n + jb[q]];
      pz[q] = pos[2 * (size_t)n + jb[q]];
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      const double dx = min_image(px[q] - xi, b.L[0], b.half[0], b.per[0]);
      const double dy = min_image(py[q] - yi, b.L[1], b.half[1], b.per[1]);
      const double dz = min_image(pz[q] - zi, b.L[2], b.half[2], b.per[2]);
      if (k0 + q < cnt && sq_dist_exact(dx, dy, dz) < rc2) ++coord;
    }
  }
  double sums[1] = {(double)coord};
  row_reduce<W, 1>(sums, wv);
  if (row >= n || wv > 0) return;
  coord = (int)sums[0];
  const double fx = f[i], fy = f[(size_t)n + i], fz = f[2 * (size_t)n + i];
  const double c = csp[i];
  feat[4 * (size_t)i + 0] = (float)rho[i];
  feat[4 * (size_t)i + 1] = (float)(c < 50.0 ? c : 50.0);
  feat[4 * (size_t)i + 2] = (float)coord;
  feat[4 * (size_t)i + 3] = (float)sqrt(fx * fx + fy * fy + fz * fz);
}

// ------------------------------------------------- float32 forward / backward
// Sixteen samples per tile, four waves, on the float32 matrix cores (16x16x4): wave w owns the
// sixteen neurons 16 w .. 16 w + 15 of every hidden layer.  The weights a wave multiplies with
// stay in its registers over the block's tiles (forward: column = own neuron; backward: column =
// own neuron of the layer below), the activations pass through LDS, and an accumulator's rows are
// samples, so that a wave meets its own activations again in the backward pass.  The weight
// gradients are products delta^T H over the samples, accumulated in registers over the tiles;
// every block writes its own sums (no atomics) and k_mlp_sum adds them in a fixed order.  Those sums are
// the caller's workspace or, for a training step, the network's: passes of other networks, streams and
// contexts run at the same time.  Without a workspace the blocks add to the outputs by atomics.
// Latency-bound (a chain of six small products a tile); at a batch of 4,096 the pass that read
// both factors of every multiply-add from LDS took 59 us on 64 blocks and needed its outputs
// cleared (9 us); this one 17 us on 256 blocks, the sum 4 us.  Without a workspace 32 us on 128 blocks
// (33 on 64, 44 on 256; 16,384 samples 88 / 59 / 57 on 64 / 128 / 256).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kTile = 16;                 // samples
constexpr int kActLd = kH + 4;            // activation rows in LDS: sixteen samples x four k on distinct banks
constexpr int kPassBlocks = 256;          // blocks of a gradient pass
constexpr int kAtomicBlocks = 128;        // of one without a workspace
constexpr int kSlabLd = kNParams + 7;     // a block's sums: the parameters, then the loss

__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// sum over k of act[sample][k] * w[k][neuron], w as operands of sixteen steps
__device__ __forceinline__ f32x4 layer(const float* act, const float (&w)[16], int lane) {
  f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
  const float* a = act + (lane & 15) * kActLd + (lane >> 4);
#pragma unroll
  for (int st = 0; st < 16; st += 2) {
    c0 = mma(a[4 * st], w[st], c0);
    c1 = mma(a[4 * st + 4], w[st + 1], c1);
  }
  return c0 + c1;
}

// The wave's rows j of delta^T H: column tile kt holds k = 16 kt + lane % 16.
__device__ __forceinline__ void outer(const float* delta, const float* act, int wv, int lane, f32x4 (&g)[4],
                                      float& bias) {
  const int r = lane >> 4, c = lane & 15;
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const int s = 4 * st + r;
    const float d = delta[s * kActLd + 16 * wv + c];
    bias += d;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) g[kt] = mma(d, act[s * kActLd + 16 * kt + c], g[kt]);
  }
}

// With BWD the block writes its share of the gradient of the mean squared error (mean over
// `total` samples) and of the error to its row of `slab`, or adds them to grad and loss (ATOMIC);
// otherwise the outputs to `out`.
template <bool BWD, bool ATOMIC = false>
__global__ void __launch_bounds__(256) k_mlp_pass(const float* __restrict__ feat, const float* __restrict__ target,
                                                  const int* __restrict__ sel, int nb, int total,
                                                  const float* __restrict__ P, Std4 st, float* __restrict__ slab,
                                                  float* __restrict__ grad, float* __restrict__ loss,
                                                  float* __restrict__ out) {
  constexpr int NB = BWD ? 5 : 2;
  __shared__ float X[kTile][8];
  __shared__ float buf[NB][kTile * kActLd];  // H1, H2, delta3, delta2, delta1
  __shared__ float ypart[4][kTile], dY[kTile];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r = lane >> 4, c = lane & 15, j = 16 * wv + c;
  float *H1 = buf[0], *H2 = buf[1];
  float w2[16], w3[16], v2[16], v3[16];  // forward and backward operands of layers 2 and 3
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int k = 4 * q + r;
    w2[q] = P[kOffW2 + j * kH + k];
    w3[q] = P[kOffW3 + j * kH + k];
    if constexpr (BWD) {
      v2[q] = P[kOffW2 + k * kH + j];
      v3[q] = P[kOffW3 + k * kH + j];
    }
  }
  const float w1 = P[kOffW1 + j * kIn + r], w4 = P[kOffW4 + j];
  const float b1 = P[kOffB1 + j], b2 = P[kOffB2 + j], b3 = P[kOffB3 + j], b4 = P[kOffB4];
  f32x4 g2[4], g3[4], g1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) g2[kt] = g3[kt] = g1;
  float gb1 = 0.f, gb2 = 0.f, gb3 = 0.f, g4 = 0.f, gb4 = 0.f, err = 0.f;
  const unsigned n = (unsigned)nb;  // (a stride beyond the last sample stays below 2^32)
  for (unsigned s0 = blockIdx.x * kTile; s0 < n; s0 += gridDim.x * kTile) {
    float y_target = 0.f;
    if (tid < kTile * kIn) {
      const int s = tid >> 2;
      const unsigned g = s0 + s;
      float x = 0.f;
      if (g < n) {
        const unsigned id = sel ? (unsigned)sel[g] : g;
        x = (feat[4 * (size_t)id + (tid & 3)] - st.mu[tid & 3]) / st.sd[tid & 3];
      }
      X[s][tid & 3] = x;
    }
    if (BWD && tid < kTile && s0 + tid < n) y_target = target[sel ? (unsigned)sel[s0 + tid] : s0 + tid];
    __syncthreads();
    // rows of the accumulators: sample 4 r + q
    f32x4 z = mma(X[c][r], w1, f32x4{b1, b1, b1, b1}), h1, h2, h3;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      h1[q] = tanhf(z[q]);
      H1[(4 * r + q) * kActLd + j] = h1[q];
    }
    __syncthreads();
    z = layer(H1, w2, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      h2[q] = tanhf(z[q] + b2);
      H2[(4 * r + q) * kActLd + j] = h2[q];
    }
    __syncthreads();
    z = layer(H2, w3, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      h3[q] = tanhf(z[q] + b3);
      float y = w4 * h3[q];  // summed over the wave's neurons
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) y += __shfl_xor(y, off, kWave);
      if (c == 0) ypart[wv][4 * r + q] = y;
    }
    __syncthreads();
    if (tid < kTile) {
      const float y = b4 + ((ypart[0][tid] + ypart[1][tid]) + (ypart[2][tid] + ypart[3][tid]));
      float d = 0.f;
      if (s0 + tid < n) {
        if (out) out[s0 + tid] = y;
        if (BWD) {
          const float e = y - y_target;
          d = 2.f * e / (float)total;
          err = fmaf(e, e, err);
        }
      }
      dY[tid] = d;
    }
    if constexpr (BWD) {
      float *D3 = buf[NB - 3], *D2 = buf[NB - 2], *D1 = buf[NB - 1];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float d = dY[4 * r + q];
        g4 = fmaf(d, h3[q], g4);
        D3[(4 * r + q) * kActLd + j] = d * w4 * (1.f - h3[q] * h3[q]);
      }
      if (tid < kTile) gb4 += dY[tid];
      __syncthreads();
      z = layer(D3, v3, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) D2[(4 * r + q) * kActLd + j] = z[q] * (1.f - h2[q] * h2[q]);
      outer(D3, H2, wv, lane, g3, gb3);
      __syncthreads();
      z = layer(D2, v2, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) D1[(4 * r + q) * kActLd + j] = z[q] * (1.f - h1[q] * h1[q]);
      outer(D2, H1, wv, lane, g2, gb2);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int s = 4 * q + r;
        const float d = D1[s * kActLd + j];
        gb1 += d;
        g1 = mma(d, c < kIn ? X[s][c] : 0.f, g1);
      }
    }
    __syncthreads();
  }
  if constexpr (BWD) {
    auto put = [&](int i, float v) {
      if constexpr (!ATOMIC) slab[(size_t)blockIdx.x * kSlabLd + i] = v;
      else if (i == kNParams) atomicAdd(loss, v / (float)total);
      else atomicAdd(grad + i, v);
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = 16 * wv + 4 * r + q;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        put(kOffW2 + row * kH + 16 * kt + c, g2[kt][q]);
        put(kOffW3 + row * kH + 16 * kt + c, g3[kt][q]);
      }
      if (c < kIn) put(kOffW1 + row * kIn + c, g1[q]);
    }
    auto over_rows = [](float v) {
      v += __shfl_xor(v, 16, kWave);
      return v + __shfl_xor(v, 32, kWave);
    };
    gb1 = over_rows(gb1);
    gb2 = over_rows(gb2);
    gb3 = over_rows(gb3);
    g4 = over_rows(g4);
    if (r == 0) {
      put(kOffB1 + j, gb1);
      put(kOffB2 + j, gb2);
      put(kOffB3 + j, gb3);
      put(kOffW4 + j, g4);
    }
    if (wv == 0) {
      gb4 = wave_sum(gb4);
      err = wave_sum(err);
      if (lane == 0) {
        put(kOffB4, gb4);
        put(kNParams, err);
      }
    }
  }
}

struct AdamArgs {
  float *p, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam(const AdamArgs& a, int i, float gi) {
  const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  const float mh = mi / a.c1, vh = vi / a.c2;
  a.p[i] = a.p[i] - a.lr * mh / (sqrtf(vh) + a.eps);
}

// Sums the blocks' gradients (and the mean squared error, entry kNParams): 32 entries by 8 shares
// of the blocks per block.  ADAM: the parameters are updated with the sum instead of storing it.
template <bool ADAM>
__global__ void __launch_bounds__(256) k_mlp_sum(const float* __restrict__ slab, int nblk, int total,
                                                 float* __restrict__ grad, float* __restrict__ loss, AdamArgs a) {
  __shared__ float sh[8][33];
  const int col = threadIdx.x & 31, part = threadIdx.x >> 5;
  const int i = blockIdx.x * 32 + col;
  float v = 0.f;
  if (i <= kNParams) {
#pragma unroll 8
    for (int b = part; b < nblk; b += 8) v += slab[(size_t)b * kSlabLd + i];
  }
  sh[part][col] = v;
  __syncthreads();
  if (part != 0 || i > kNParams) return;
  v = ((sh[0][col] + sh[1][col]) + (sh[2][col] + sh[3][col])) + ((sh[4][col] + sh[5][col]) + (sh[6][col] + sh[7][col]));
  if (i == kNParams) *loss = v / (float)total;
  else if (ADAM) adam(a, i, v);
  else grad[i] = v;
}

__global__ void k_mlp_clear(float* __restrict__ grad, float* __restrict__ loss) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kNParams) grad[i] = 0.f;
  else if (i == kNParams) *loss = 0.f;
}

// Adam with bias correction; clears the gradient for the next step.
__global__ void k_adam(AdamArgs a, float* __restrict__ g, int np) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  adam(a, i, g[i]);
  g[i] = 0.f;
}

// --------------------------------------------------------- bfloat16 inference
__device__ __forceinline__ unsigned short bf16_rne(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40);  // quiet NaN
  const unsigned lsb = (u >> 16) & 1u;
  u += 0x7fffu + lsb;
  return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

__global__ void k_pack_bf16(const float* __restrict__ P, unsigned short* __restrict__ wb) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  // W1 padded to [64][16]
  if (e < kH * 16) {
    const int j = e / 16, k = e % 16;
    wb[e] = k < kIn ? bf16_rne(P[kOffW1 + j * kIn + k]) : (unsigned short)0;
  }
  if (e < kH * kH) {
    wb[kH * 16 + e] = bf16_rne(P[kOffW2 + e]);
    wb[kH * 16 + kH * kH + e] = bf16_rne(P[kOffW3 + e]);
  }
  if (e < kH) wb[kH * 16 + 2 * kH * kH + e] = bf16_rne(P[kOffW4 + e]);
}

typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma_bf16_16x16x32(v8s a, v8s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// One wave evaluates 16 atoms: every hidden layer is a [16 x K] x [K x 64] product on the
// 16x16x32 bfloat16 matrix cores of gfx950 (four output tiles, K/32 steps; lane = row or
// column (lane % 16) and a group of eight K values (lane / 16)), bias + tanh in float32,
// the activations rounded to bfloat16 in LDS for the next layer.
__global__ void __launch_bounds__(256) k_mlp_bf16(const float* __restrict__ feat, int n, const float* __restrict__ P,
                                                  const unsigned short* __restrict__ wb, Std4 st,
                                                  float* __restrict__ out) {
  __shared__ unsigned short act[4][16][kH + 8];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int a0 = (blockIdx.x * 4 + wv) * 16;
  const int ri = lane & 15;   // row (atom) of A, column (neuron) of B and D
  const int kq = lane >> 4;   // k quad
  // inputs, standardised and rounded, K padded to 32 (the weights hold 16 columns)
  {
    v8s a;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = 8 * kq + r;
      float x = 0.f;
      if (k < kIn && a0 + ri < n) x = (feat[4 * (size_t)(a0 + ri) + k] - st.mu[k]) / st.sd[k];
      a[r] = (short)bf16_rne(x);
    }
    const unsigned short* W1 = wb;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      v8s bv;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int k = 8 * kq + r;
        bv[r] = k < 16 ? (short)W1[(nt * 16 + ri) * 16 + k] : (short)0;
      }
      v4f c = {0.f, 0.f, 0.f, 0.f};
      c = mfma_bf16_16x16x32(a, bv, c);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = nt * 16 + ri;
        act[wv][4 * kq + r][j] = bf16_rne(tanhf(c[r] + P[kOffB1 + j]));
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int layer = 0; layer < 2; ++layer) {
    const unsigned short* Wl = wb + kH * 16 + layer * kH * kH;
    const float* bias = P + (layer == 0 ? kOffB2 : kOffB3);
    v4f c[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) c[nt] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kH / 32; ++ks) {
      v8s a;
#pragma unroll
      for (int r = 0; r < 8; ++r) a[r] = (short)act[wv][ri][32 * ks + 8 * kq + r];
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        v8s bv;
#pragma unroll
        for (int r = 0; r < 8; ++r) bv[r] = (short)Wl[(nt * 16 + ri) * kH + 32 * ks + 8 * kq + r];
        c[nt] = mfma_bf16_16x16x32(a, bv, c[nt]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = nt * 16 + ri;
        act[wv][4 * kq + r][j] = bf16_rne(tanhf(c[nt][r] + bias[j]));
      }
    __syncthreads();
  }
  if (lane < 16 && a0 + lane < n) {
    const unsigned short* W4 = wb + kH * 16 + 2 * kH * kH;
    float y = P[kOffB4];
    for (int k = 0; k < kH; ++k) y = fmaf(bf16_to_f(W4[k]), bf16_to_f(act[wv][lane][k]), y);
    out[a0 + lane] = y;
  }
}

// prediction -> additional detection weight, with the range fallback
__global__ void k_mlp_w0(const float* __restrict__ pred, const float* __restrict__ feat, int n, double tau_lo,
                         double width, Std4 lims_lo, Std4 lims_hi, double* __restrict__ w0) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  bool in_range = true;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float f = feat[4 * (size_t)i + c];
    if (!(f >= lims_lo.mu[c] && f <= lims_hi.mu[c])) in_range = false;
  }
  double w = 0.0;
  if (in_range) {
    const double dF = exp((double)pred[i]) - 1e-3;
    w = 1.0 - fcut_exact((dF - tau_lo) / width);
  }
  w0[i] = w;
}

// Training labels: dF_i = |F^precise_i - F^fast_i| (float64), label_i = log(dF_i + 1e-3)
// rounded to float32.
__global__ void k_mlp_labels(long long n, const double* __restrict__ fp, const double* __restrict__ ff,
                             double* __restrict__ dF, float* __restrict__ label) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double dx = fp[i] - ff[i], dy = fp[n + i] - ff[n + i], dz = fp[2 * n + i] - ff[2 * n + i];
  const double d = sqrt(dx * dx + dy * dy + dz * dz);
  if (dF) dF[i] = d;
  label[i] = (float)log(d + 1e-3);
}

// Column statistics of the [n][4] float32 features, one block per column, float64 sums
// reduced in a fixed order: out[c] mean, out[4 + c] standard deviation with n - 1,
// out[8 + c] minimum, out[12 + c] maximum.
constexpr int kStatThreads = 1024;
__global__ void __launch_bounds__(kStatThreads) k_feature_stats(const float* __restrict__ feat, long long n,
                                                                double* __restrict__ out) {
  __shared__ double sh[kStatThreads / kWave];
  __shared__ double shm[kStatThreads / kWave], shx[kStatThreads / kWave];
  const int c = blockIdx.x;
  const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  double s = 0.0, mn = INFINITY, mx = -INFINITY;
  for (long long i = threadIdx.x; i < n; i += kStatThreads) {
    const double v = (double)feat[4 * i + c];
    s += v;
    mn = v < mn ? v : mn;
    mx = v > mx ? v : mx;
  }
  s = wave_sum(s);
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    const double a = __shfl_xor(mn, off, kWave), b = __shfl_xor(mx, off, kWave);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  if (lane == 0) {
    sh[w] = s;
    shm[w] = mn;
    shx[w] = mx;
  }
  __syncthreads();
  double tot = 0.0, tmin = INFINITY, tmax = -INFINITY;
  for (int k = 0; k < kStatThreads / kWave; ++k) {
    tot += sh[k];
    tmin = shm[k] < tmin ? shm[k] : tmin;
    tmax = shx[k] > tmax ? shx[k] : tmax;
  }
  const double mean = n > 0 ? tot / (double)n : 0.0;
  __syncthreads();
  double q = 0.0;
  for (long long i = threadIdx.x; i < n; i += kStatThreads) {
    const double d = (double)feat[4 * i + c] - mean;
    q += d * d;
  }
  q = wave_sum(q);
  if (lane == 0) sh[w] = q;
  __syncthreads();
  if (threadIdx.x == 0) {
    double qq = 0.0;
    for (int k = 0; k < kStatThreads / kWave; ++k) qq += sh[k];
    out[c] = mean;
    out[4 + c] = n > 1 ? sqrt(qq / (double)(n - 1)) : 0.0;
    out[8 + c] = tmin;
    out[12 + c] = tmax;
  }
}

}  // namespace apx

using namespace apx;

extern "C" {

apx_status apx_mlp_labels(apx_ctx* ctx, int64_t n, const double* f_precise, const double* f_fast, double* dF,
                          float* label) {
  if (!ctx) return APX_EINVAL;
  if (n < 0) return fail(ctx, APX_EINVAL, "negative size");
  if (n > 0 && (!f_precise || !f_fast || !label)) return fail(ctx, APX_EINVAL, "forces and label are required");
  if (n == 0) return APX_OK;
  k_mlp_labels<<<blocks_for(n, 256), 256, 0, ctx->stream>>>(n, f_precise, f_fast, dF, label);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

apx_status apx_mlp_feature_stats(apx_ctx* ctx, const float* feat, int64_t n, double* stats) {
  if (!ctx) return APX_EINVAL;
  if (n < 1 || !feat || !stats) return fail(ctx, APX_EINVAL, "features (n >= 1) and stats are required");
  k_feature_stats<<<4, kStatThreads, 0, ctx->stream>>>(feat, n, stats);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

apx_status apx_mlp_create(apx_ctx* ctx, const float* params, const float* mu, const float* sd, apx_mlp** out) {
  if (!ctx) return APX_EINVAL;
  if (!params || !mu || !sd || !out) return fail(ctx, APX_EINVAL, "params, mu, sd and out are required");
  *out = nullptr;
  for (int c = 0; c < 4; ++c)
    if (!(sd[c] > 0.f)) return fail(ctx, APX_EINVAL, "standard deviations must be positive");
  apx_mlp* m = new apx_mlp();
  m->device = ctx->device;
  const size_t nf = 3 * (size_t)kNParams + 61;  // the bfloat16 weights behind on 16 bytes
  const size_t nwb = kH * 16 + 2 * kH * kH + kH;
  static_assert((kH * 16 + 2 * kH * kH + kH) % 2 == 0, "the sums behind the bfloat16 weights lie on floats");
  if (m->buf.ensure((nf + (size_t)kPassBlocks * kSlabLd) * sizeof(float) + nwb * sizeof(unsigned short)) !=
      hipSuccess) {
    delete m;
    return fail(ctx, APX_ENOMEM, "MLP buffers");
  }
  float* base = m->buf.as<float>();
  m->params = base;
  m->m = base + kNParams;
  m->v = base + 2 * kNParams;
  m->loss = base + 3 * kNParams;
  m->wb = reinterpret_cast<unsigned short*>(base + nf);
  m->sums = reinterpret_cast<float*>(m->wb + nwb);
  for (int c = 0; c < 4; ++c) {
    m->st.mu[c] = mu[c];
    m->st.sd[c] = sd[c];
  }
  if (hipMemcpy(m->params, params, kNParams * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(m->m, 0, (2 * (size_t)kNParams + 1) * sizeof(float)) != hipSuccess) {
    delete m;
    return fail(ctx, APX_EDEVICE, "MLP upload");
  }
  *out = m;
  return APX_OK;
}

void apx_mlp_destroy(apx_mlp* m) {
  if (!m) return;
  (void)hipSetDevice(m->device);
  delete m;
}

apx_status apx_mlp_get_params(apx_ctx* ctx, const apx_mlp* m, float* params) {
  if (!ctx || !m || !params) return APX_EINVAL;
  APX_HIP(ctx, hipMemcpyAsync(params, m->params, kNParams * sizeof(float), hipMemcpyDeviceToHost, ctx->stream));
  APX_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return APX_OK;
}

apx_status apx_mlp_set_range(apx_mlp* m, const float* fmin, const float* fmax) {
  if (!m || !fmin || !fmax) return APX_EINVAL;
  for (int c = 0; c < 4; ++c) {
    m->fmin[c] = fmin[c];
    m->fmax[c] = fmax[c];
  }
  return APX_OK;
}

apx_status apx_features(apx_ctx* ctx, const apx_atoms* atoms, const apx_nlist* nl, const double* rho,
                        const double* csp, const double* f_eam, float* feat) {
  if (!ctx) return APX_EINVAL;
  apx_status s = check_atoms(ctx, atoms);
  if (s != APX_OK) return s;
  if (!nl || nl->n != atoms->n) return fail(ctx, APX_EINVAL, "nlist mismatch");
  if (nl->r_list < 3.08) return fail(ctx, APX_EINVAL, "neighbour list shorter than the coordination radius");
  const int n = (int)atoms->n;
  if (n == 0) return APX_OK;
  if (!rho || !csp || !f_eam || !feat) return fail(ctx, APX_EINVAL, "feature inputs are required");
  ProfScope ps(ctx, "mlp.features");
  auto launch = [&](auto kern, int W) {
    kern<<<row_blocks(n, W), row_threads(W), 0, ctx->stream>>>(atoms->pos, n, make_box(atoms), nl->count, nl->idx,
                                                               nl->max_nb, rho, csp, f_eam, feat);
  };
  if (row_waves(n) == 16)
    launch(k_features<16>, 16);
  else
    launch(k_features<4>, 4);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

apx_status apx_mlp_forward(apx_ctx* ctx, const apx_mlp* m, const float* feat, int64_t n, float* out) {
  if (!ctx || !m) return APX_EINVAL;
  if (n < 0 || n > 0x7fffffff) return fail(ctx, APX_EINVAL, "bad sample count");
  if (n == 0) return APX_OK;
  if (!feat || !out) return fail(ctx, APX_EINVAL, "feat and out are required");
  const int blocks = (int)std::min<int64_t>(8 * kPassBlocks, blocks_for(n, kTile));
  k_mlp_pass<false><<<blocks, 256, 0, ctx->stream>>>(feat, nullptr, nullptr, (int)n, (int)n, m->params, m->st, nullptr,
                                                     nullptr, nullptr, out);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

}  // extern "C"

namespace {

// Blocks of a gradient pass over nb samples; each writes one row of sums.
int pass_blocks(int64_t nb) { return (int)std::min<int64_t>(kPassBlocks, blocks_for(nb, kTile)); }

// The pass over the batch: rows of sums to `slab`, or (null) sums into grad and loss.
apx_status mlp_pass(apx_ctx* ctx, const apx_mlp* m, const float* feat, const float* target, const int32_t* sel,
                    int64_t nb, float* slab, float* grad, float* loss) {
  ProfScope ps(ctx, "mlp.train");
  auto launch = [&](auto kern, int blocks) {
    kern<<<blocks, 256, 0, ctx->stream>>>(feat, target, sel, (int)nb, (int)nb, m->params, m->st, slab, grad, loss,
                                          nullptr);
  };
  if (slab)
    launch(k_mlp_pass<true>, pass_blocks(nb));
  else
    launch(k_mlp_pass<true, true>, std::min(kAtomicBlocks, pass_blocks(nb)));
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

// The update of one step (the step counter already advanced).
AdamArgs adam_args(apx_mlp* m, float lr, float beta1, float beta2, float eps) {
  return AdamArgs{m->params, m->m,  m->v, lr, beta1, beta2, eps, 1.f - powf(beta1, (float)m->step),
                  1.f - powf(beta2, (float)m->step)};
}

constexpr int kSumBlocks = (kNParams + 1 + 31) / 32;

}  // namespace

extern "C" {

int64_t apx_mlp_work_size(int64_t nb) {
  return nb <= 0 || nb > 0x7fffffff ? 0 : (int64_t)pass_blocks(nb) * kSlabLd;
}

apx_status apx_mlp_gradients_ws(apx_ctx* ctx, apx_mlp* m, const float* feat, const float* target, const int32_t* sel,
                                int64_t nb, float* grad, float* loss, float* work) {
  if (!ctx || !m) return APX_EINVAL;
  if (nb <= 0 || nb > 0x7fffffff) return fail(ctx, APX_EINVAL, "batch size must be positive");
  if (!feat || !target || !grad || !loss) return fail(ctx, APX_EINVAL, "feat, target, grad and loss are required");
  if (!work) {
    k_mlp_clear<<<blocks_for(kNParams + 1, 256), 256, 0, ctx->stream>>>(grad, loss);
    APX_LAUNCH_CHECK(ctx);
    return mlp_pass(ctx, m, feat, target, sel, nb, nullptr, grad, loss);
  }
  const apx_status s = mlp_pass(ctx, m, feat, target, sel, nb, work, nullptr, nullptr);
  if (s != APX_OK) return s;
  k_mlp_sum<false><<<kSumBlocks, 256, 0, ctx->stream>>>(work, pass_blocks(nb), (int)nb, grad, loss, AdamArgs{});
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

apx_status apx_mlp_gradients(apx_ctx* ctx, apx_mlp* m, const float* feat, const float* target, const int32_t* sel,
                             int64_t nb, float* grad, float* loss) {
  return apx_mlp_gradients_ws(ctx, m, feat, target, sel, nb, grad, loss, nullptr);
}

apx_status apx_mlp_adam_step(apx_ctx* ctx, apx_mlp* m, const float* grad, float lr, float beta1, float beta2,
                             float eps) {
  if (!ctx || !m || !grad) return APX_EINVAL;
  m->step += 1;
  k_adam<<<blocks_for(kNParams, 256), 256, 0, ctx->stream>>>(adam_args(m, lr, beta1, beta2, eps),
                                                             const_cast<float*>(grad), kNParams);
  APX_LAUNCH_CHECK(ctx);
  m->wb_valid = false;
  return APX_OK;
}

apx_status apx_mlp_train_step(apx_ctx* ctx, apx_mlp* m, const float* feat, const float* target, const int32_t* sel,
                              int64_t nb, float lr, float* loss) {
  if (!ctx || !m) return APX_EINVAL;
  if (nb <= 0 || nb > 0x7fffffff) return fail(ctx, APX_EINVAL, "batch size must be positive");
  if (!feat || !target) return fail(ctx, APX_EINVAL, "feat and target are required");
  const apx_status s = mlp_pass(ctx, m, feat, target, sel, nb, m->sums, nullptr, nullptr);
  if (s != APX_OK) return s;
  m->step += 1;
  k_mlp_sum<true><<<kSumBlocks, 256, 0, ctx->stream>>>(m->sums, pass_blocks(nb), (int)nb, nullptr,
                                                       loss ? loss : m->loss, adam_args(m, lr, 0.9f, 0.999f, 1e-8f));
  APX_LAUNCH_CHECK(ctx);
  m->wb_valid = false;
  return APX_OK;
}

apx_status apx_mlp_infer_bf16(apx_ctx* ctx, apx_mlp* m, const float* feat, int64_t n, float* out) {
  if (!ctx || !m) return APX_EINVAL;
  if (n < 0 || n > 0x7fffffff) return fail(ctx, APX_EINVAL, "bad sample count");
  if (!m->wb_valid) {
    k_pack_bf16<<<blocks_for(kH * kH, 256), 256, 0, ctx->stream>>>(m->params, m->wb);
    APX_LAUNCH_CHECK(ctx);
    m->wb_valid = true;
  }
  if (n == 0) return APX_OK;
  if (!feat || !out) return fail(ctx, APX_EINVAL, "feat and out are required");
  ProfScope ps(ctx, "mlp.infer_bf16");
  k_mlp_bf16<<<blocks_for(n, 64), 256, 0, ctx->stream>>>(feat, (int)n, m->params, m->wb, m->st, out);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

apx_status apx_mlp_weight(apx_ctx* ctx, const apx_mlp* m, const float* pred, const float* feat, int64_t n,
                          double tau_lo, double tau_hi, double* w0_extra) {
  if (!ctx || !m) return APX_EINVAL;
  if (!(tau_hi > tau_lo)) return fail(ctx, APX_EINVAL, "tau_hi must exceed tau_lo");
  if (n < 0 || n > 0x7fffffff) return fail(ctx, APX_EINVAL, "bad sample count");
  if (n > 0 && (!pred || !feat || !w0_extra)) return fail(ctx, APX_EINVAL, "pred, feat and w0_extra are required");
  if (n == 0) return APX_OK;
  Std4 lo, hi;
  for (int c = 0; c < 4; ++c) {
    lo.mu[c] = m->fmin[c];
    hi.mu[c] = m->fmax[c];
    lo.sd[c] = hi.sd[c] = 0.f;
  }
  k_mlp_w0<<<blocks_for(n, 256), 256, 0, ctx->stream>>>(pred, feat, (int)n, tau_lo, tau_hi - tau_lo, lo, hi, w0_extra);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

apx_status apx_mlp_precision(apx_ctx* ctx, apx_mlp* m, const float* feat, int64_t n, double tau_lo, double tau_hi,
                             float* pred, double* w0_extra) {
  if (!ctx || !m) return APX_EINVAL;
  if (!(tau_hi > tau_lo)) return fail(ctx, APX_EINVAL, "tau_hi must exceed tau_lo");
  if (n > 0 && (!pred || !w0_extra)) return fail(ctx, APX_EINVAL, "pred and w0_extra are required");
  apx_status s = apx_mlp_infer_bf16(ctx, m, feat, n, pred);
  if (s != APX_OK || n == 0) return s;
  return apx_mlp_weight(ctx, m, pred, feat, n, tau_lo, tau_hi, w0_extra);
}

}  // extern "C"
