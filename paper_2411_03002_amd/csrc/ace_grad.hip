// Coefficient gradients of the atomic cluster expansion:
//   dE/dc1_v = sum_i w_i B_iv,   dE/dc2_v = sum_i w_i F_eps'(phi2_i) B_iv.
//
// A third-order function is B = sum_M A_n3M P_LM(q1, q2) with the products P of ace_sym.hip, so
// the gradients of one degree triple (l1, l2, L) are a matrix product over atoms and M: rows
// (n3, which sum), columns label pairs, both weights folded into the rows.  It runs on the
// float64 matrix cores, four atoms per instruction and sixteen pairs per accumulator; the
// triple is taken once, with the block of the smallest degree as its row.  Second-order
// functions have a single block as the column, first-order ones the constant 1.  The sums run
// in float64 for either precision of the atomic base.  A block keeps 32 atoms in LDS and its
// waves take the (type, sixteen pairs) items in turn; each block adds up its own gradient
// (no atomics, a fixed order), and a second kernel sums over blocks.
// At 3,982 atoms and (10, 4) the gradients with energy and adjoint took 1,300 us in the kernel
// that reduced every triple across the wave and added it with atomics.
#include <algorithm>
#include <type_traits>

#include "ace_coupling_gen.h"
#include "ace_sym.h"
#include "device_util.h"

namespace apx {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kGradAtoms = 32;             // atoms per chunk
constexpr int kGradStride = kGradAtoms + 4;  // row stride in LDS: consecutive n on distinct banks
constexpr int kGradWaves = 8;
constexpr int kGradBlocks = 256;           // blocks along the atoms (each holds a gradient)

template <class T>
struct GradArgs {
  const T* A;  // [n_act][stride]
  const T* slope;
  const double* w;
  const int* active;
  const int* pairs;  // n1 | n2 << 16, by type, sixteen a group
  const int* items;  // [n][3]: type (second order of degree L: 15 + L), first pair, first slot
  double* slab;      // [block][slots]
  int n_act, stride, n_max, n_items, slots;
};

// Rows o = 2 n3 + p over sixteen columns; d[r] holds row 4 r + lane / 16, e[k] row
// 16 + 4 k + lane / 16, column lane % 16.
template <int NMAX>
struct GradAcc {
  static constexpr int R = 2 * NMAX, NB = (R - 16) / 4;
  f64x4 d;
  double e[NB > 0 ? NB : 1];
  __device__ __forceinline__ void zero() {
    d = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NB; ++k) e[k] = 0.0;
  }
  // blk: the rows of one component, [n][kGradStride] at the lane's atom; the lane's rows are
  // o = lane % 16 and 16 + 4 k + lane % 4, all of the sum p = lane % 2 whose weight is s
  __device__ __forceinline__ void step(const double* blk, int n_max, int lane, double s, double P) {
    auto row = [&](int n3) { return n3 < n_max ? s * blk[n3 * kGradStride] : 0.0; };
    d = __builtin_amdgcn_mfma_f64_16x16x4f64(row((lane & 15) >> 1), P, d, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < NB; ++k)
      e[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(row(8 + 2 * k + ((lane & 3) >> 1)), P, e[k], 0, 0, 0);
  }
  __device__ __forceinline__ void add_to(double* out, int lane, bool first) const {
    auto put = [&](int row, double v) {
      double* q = out + row * 16 + (lane & 15);
      *q = first ? v : *q + v;
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) put(4 * r + (lane >> 4), d[r]);
#pragma unroll
    for (int k = 0; k < NB; ++k) put(16 + 4 * k + (lane >> 4), e[k]);
  }
};

// One item of third-order type (L1 <= L2): sixteen pairs, the rows of degrees L2 - L1 <= L <= L1.
template <int LMAX, int NMAX, int L1, int L2>
__device__ __forceinline__ void grad_item(const double* As, const double* sw, int n_max, int pair, double* out,
                                          int lane, bool first) {
  using Acc = GradAcc<NMAX>;
  constexpr int L0 = L2 - L1, NL = (L1 - L0) / 2 + 1;
  Acc acc[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) acc[k].zero();
  const int n1 = pair & 0xffff, n2 = pair >> 16, sub = lane >> 4;
  const double* pa = As + (L1 * L1 * n_max + n1) * kGradStride + sub;
  const double* pb = As + (L2 * L2 * n_max + n2) * kGradStride + sub;
  const int ms = n_max * kGradStride;
  for (int at = 0; at < kGradAtoms; at += 4) {
    double a[2 * L1 + 1], b[2 * L2 + 1];
#pragma unroll
    for (int m = 0; m < 2 * L1 + 1; ++m) a[m] = pa[m * ms + at];
#pragma unroll
    for (int m = 0; m < 2 * L2 + 1; ++m) b[m] = pb[m * ms + at];
    const double s = sw[(lane & 1) * kGradAtoms + at + sub];
    auto comp = [&](auto Mc) {
      constexpr int M = decltype(Mc)::value, AM = M < 0 ? -M : M;
      if constexpr (AM <= L1) {
        double P[5];
        SymP<L1, L2, M>::template p<LMAX, double>(a, b, P);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
          const int L = L0 + 2 * k;
          if (L >= AM) acc[k].step(As + (L * L + L + M) * ms + at + sub, n_max, lane, s, P[L]);
        }
      }
    };
    comp(std::integral_constant<int, -4>{});
    comp(std::integral_constant<int, -3>{});
    comp(std::integral_constant<int, -2>{});
    comp(std::integral_constant<int, -1>{});
    comp(std::integral_constant<int, 0>{});
    comp(std::integral_constant<int, 1>{});
    comp(std::integral_constant<int, 2>{});
    comp(std::integral_constant<int, 3>{});
    comp(std::integral_constant<int, 4>{});
  }
#pragma unroll
  for (int k = 0; k < NL; ++k) acc[k].add_to(out + k * Acc::R * 16, lane, first);
}

// Second order of degree L: the columns are the blocks n' = lane % 16; for L = 0 the column
// n_max is the constant 1 (first order).
template <int NMAX>
__device__ __forceinline__ void grad_low(const double* As, const double* sw, int n_max, int L, double* out, int lane,
                                         bool first) {
  using Acc = GradAcc<NMAX>;
  Acc acc;
  acc.zero();
  const int col = lane & 15, sub = lane >> 4, ms = n_max * kGradStride;
  for (int at = 0; at < kGradAtoms; at += 4) {
    const double s = sw[(lane & 1) * kGradAtoms + at + sub];
    for (int m = L * L; m < (L + 1) * (L + 1); ++m) {
      const double* blk = As + m * ms + at + sub;
      const double P = col < n_max ? blk[col * kGradStride] : (L == 0 && col == n_max ? 1.0 : 0.0);
      acc.step(blk, n_max, lane, s, P);
    }
  }
  acc.add_to(out, lane, first);
}

template <class T, int LMAX, int NMAX>
__global__ void __launch_bounds__(kGradWaves * 64, 4) k_ace_grad(GradArgs<T> g) {
  constexpr int LM = (LMAX + 1) * (LMAX + 1);
  extern __shared__ double As[];  // [lm][n][kGradStride]
  __shared__ double sw[2 * kGradAtoms];
  const int tid = threadIdx.x, lane = tid & 63, K = g.n_max;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* slab = g.slab + (size_t)blockIdx.x * g.slots;
  const int chunks = (g.n_act + kGradAtoms - 1) / kGradAtoms;
  for (int c = blockIdx.x; c < chunks; c += gridDim.x) {
    const int q0 = c * kGradAtoms;
    __syncthreads();
    // atoms beyond the last have weight 0 and a base of zeros
    for (int e = tid; e < kGradAtoms * K * LM; e += kGradWaves * 64) {
      const int t = e / (K * LM), r = e - t * K * LM, n = r / LM, lm = r - n * LM;
      As[(lm * K + n) * kGradStride + t] = q0 + t < g.n_act ? (double)g.A[(size_t)(q0 + t) * g.stride + r] : 0.0;
    }
    if (tid < kGradAtoms) {
      const int q = q0 + tid;
      double w = 0.0, f = 0.0;
      if (q < g.n_act) {
        w = g.w ? g.w[g.active[q]] : 1.0;
        f = w * (double)g.slope[q];
      }
      sw[tid] = w;
      sw[kGradAtoms + tid] = f;
    }
    __syncthreads();
    const bool first = c == (int)blockIdx.x;
    for (int it = wv + kGradWaves * blockIdx.y; it < g.n_items; it += kGradWaves * gridDim.y) {
      const int type = __builtin_amdgcn_readfirstlane(g.items[3 * it]);
      double* out = slab + __builtin_amdgcn_readfirstlane(g.items[3 * it + 2]);
      const int p0 = __builtin_amdgcn_readfirstlane(g.items[3 * it + 1]);
      const int pair = g.pairs[p0 + (lane & 15)];
#define APX_GRAD(A_, B_) \
  case B_ * (B_ + 1) / 2 + A_: grad_item<LMAX, NMAX, A_, B_>(As, sw, K, pair, out, lane, first); break;
      switch (type) {
        APX_GRAD(0, 0)
        APX_GRAD(1, 1)
        APX_GRAD(1, 2)
        APX_GRAD(2, 2)
        APX_GRAD(2, 3)
        APX_GRAD(3, 3)
        default:
          if constexpr (LMAX >= 4) {
            switch (type) {
              APX_GRAD(2, 4)
              APX_GRAD(3, 4)
              APX_GRAD(4, 4)
              default: break;
            }
          }
          if (type >= 15) grad_low<NMAX>(As, sw, K, type - 15, out, lane, first);
      }
#undef APX_GRAD
    }
  }
}

// Sums the blocks' gradients: sixteen slots of one row per quarter wave, sixteen shares of the
// blocks per slot; slot -> 2 v + p (-1: not a function of its own) with the scale of P.
__global__ void __launch_bounds__(256) k_ace_grad_sum(const double* __restrict__ slab, int nblk, int slots,
                                                      const int* __restrict__ at, const double* __restrict__ scale,
                                                      double* __restrict__ dc1, double* __restrict__ dc2) {
  __shared__ double sh[16][17];
  const int col = threadIdx.x & 15, part = threadIdx.x >> 4;
  const int k = blockIdx.x * 16 + col;
  double v = 0.0;
#pragma unroll 4
  for (int b = part; b < nblk; b += 16) v += slab[(size_t)b * slots + k];
  sh[part][col] = v;
  __syncthreads();
  if (part == 0) {
    double s = 0.0;
    for (int p = 0; p < 16; ++p) s += sh[p][col];
    const int o = at[k];
    if (o >= 0) (o & 1 ? dc2 : dc1)[o >> 1] = scale[k] * s;
  }
}

namespace {
inline int grad_blocks(int n_act) { return std::min(kGradBlocks, (n_act + kGradAtoms - 1) / kGradAtoms); }
}  // namespace

size_t ace_grad_scratch(const apx_ace_model* m, int n_act) {
  return sizeof(double) * (size_t)grad_blocks(n_act) * m->grad.slots;
}

template <class T>
apx_status ace_grad(apx_ctx* ctx, const apx_ace_model* m, const T* A, const T* slope, const double* w,
                    const int* active, int n_act, double* dc1, double* dc2, void* scratch) {
  const GradTables& tb = m->grad;
  GradArgs<T> g{A,       slope, w, active, tb.pairs, tb.items, static_cast<double*>(scratch), n_act, sym_stride(m->na),
                m->n_max, tb.n_items, tb.slots};
  const int nb = grad_blocks(n_act);
  // few atoms: the items of a chunk are spread over blocks too
  const int parts = std::max(1, std::min(4, 512 / nb));
  const size_t lds = sizeof(double) * (size_t)m->na * kGradStride;
  ProfScope ps(ctx, "ace.grad");
  const int nm = sym_nmax(m->n_max);
  // (the most of the instantiation: the attribute is the process's, and another thread's model may be smaller)
  const size_t most = sizeof(double) * (size_t)nm * (m->l_max + 1) * (m->l_max + 1) * kGradStride;
  auto launch = [&](auto kern) -> apx_status {
    APX_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most));
    kern<<<dim3(nb, parts), kGradWaves * 64, lds, ctx->stream>>>(g);
    APX_LAUNCH_CHECK(ctx);
    k_ace_grad_sum<<<tb.slots / 16, 256, 0, ctx->stream>>>(g.slab, nb, tb.slots, tb.at, tb.scale, dc1, dc2);
    APX_LAUNCH_CHECK(ctx);
    return APX_OK;
  };
  if (m->l_max == 3 && nm == 8) return launch(k_ace_grad<T, 3, 8>);
  if (m->l_max == 3 && nm == 10) return launch(k_ace_grad<T, 3, 10>);
  if (m->l_max == 3) return launch(k_ace_grad<T, 3, 12>);
  if (nm == 8) return launch(k_ace_grad<T, 4, 8>);
  if (nm == 10) return launch(k_ace_grad<T, 4, 10>);
  return launch(k_ace_grad<T, 4, 12>);
}

template apx_status ace_grad<float>(apx_ctx*, const apx_ace_model*, const float*, const float*, const double*,
                                    const int*, int, double*, double*, void*);
template apx_status ace_grad<double>(apx_ctx*, const apx_ace_model*, const double*, const double*, const double*,
                                     const int*, int, double*, double*, void*);

}  // namespace apx
