// Atomic cluster expansion on the active atoms: atomic base, product basis with energy
// and adjoint, force scatter.
//
// Kernels of an evaluation (Sec. III A form E = phi1 + F_eps(phi2), basis defined in the ABI
// header):
//  1. k_ace_basis    one wave per active atom: per neighbour the Chebyshev radial values
//                    and real solid harmonics, A'[k][lm] = sum_j g_k S_lm, then the radial
//                    mixing A[n][lm] = sum_k Wp[l][n][k] A'[k][lm] (Wp folds W, N_l, 1/s_a).
//  2. ace_sym.hip    energies and the adjoint projected back on the radial functions;
//     ace_grad.hip   coefficient gradients.
//  3. k_ace_force    one wave per active atom: per neighbour the gradient of sum Abar'' g_k
//                    S_lm, scattered as F_j -= w_i dE_i/dr_ij, F_i += w_i dE_i/dr_ij (float64
//                    atomics).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ace_model.h"
#include "ace_sym.h"
#include "device_util.h"

namespace apx {

struct AnchorDev {
  double A, alpha, beta, r0, rc, inv_h, rc2;
  int on;
};

template <class T>
struct AceScratch {
  T* A;             // [n_act][stride] atomic base
  const T* B;       // [n_act][stride] projected adjoint B'[lm][k] = sum_n Wp[l][n][k] Abar[n][lm]
  int stride;
  double* e_anch;   // [n_act]
  double* fp_anch;  // [n_act]
};

// ------------------------------------------------------------ shared helpers
// Real solid harmonics S_lm of (x, y, z) with x^2 + y^2 + z^2 = 1, in the order l^2 + l + m.
template <class T, int LMAX>
__device__ __forceinline__ void solid_harmonics(T x, T y, T z, T* S) {
  S[0] = T(1);
#pragma unroll
  for (int l = 0; l < LMAX; ++l) {
    const T c = (l == 0) ? T(1) : T(sqrt((2.0 * l + 1.0) / (2.0 * l + 2.0)));
    const int sll = l * l + 2 * l;  // (l, l)
    const int slm = l * l;          // (l, -l)
    const int tp = (l + 1) * (l + 1) + 2 * (l + 1);
    const int bt = (l + 1) * (l + 1);
    if (l == 0) {
      S[tp] = c * x * S[sll];
      S[bt] = c * y * S[sll];
    } else {
      S[tp] = c * (x * S[sll] - y * S[slm]);
      S[bt] = c * (y * S[sll] + x * S[slm]);
    }
#pragma unroll
    for (int m = -l; m <= l; ++m) {
      const int dst = (l + 1) * (l + 1) + (l + 1) + m;
      const int s1 = l * l + l + m;
      const T a = T((2.0 * l + 1.0) / sqrt((l + m + 1.0) * (l - m + 1.0)));
      if (m >= -(l - 1) && m <= l - 1) {
        const int s2 = (l - 1) * (l - 1) + (l - 1) + m;
        const T b = T(sqrt((l + m) * (l - m) * 1.0) / sqrt((l + m + 1.0) * (l - m + 1.0)));
        S[dst] = a * z * S[s1] - b * S[s2];
      } else {
        S[dst] = a * z * S[s1];
      }
    }
  }
}

// Gradient of sum_lm W_lm S_lm at (x, y, z): the recurrence above backwards, degree by degree (W is
// used up).  S_lm of the lower degree enters with x^2 + y^2 + z^2, hence the terms in q.  It takes 130
// operations and a second array of values, where S with three derivatives took 370 and four arrays.
template <class T, int LMAX>
__device__ __forceinline__ void harmonics_gradient(T x, T y, T z, const T* S, T* W, T& gx, T& gy, T& gz) {
  T q = T(0);
  gx = gy = gz = T(0);
#pragma unroll
  for (int l = LMAX - 1; l >= 0; --l) {
    const T c = (l == 0) ? T(1) : T(sqrt((2.0 * l + 1.0) / (2.0 * l + 2.0)));
    const int sll = l * l + 2 * l;
    const int slm = l * l;
    const T wt = c * W[(l + 1) * (l + 1) + 2 * (l + 1)];
    const T wb = c * W[(l + 1) * (l + 1)];
    gx = fma(wt, S[sll], gx);
    gy = fma(wb, S[sll], gy);
    if (l > 0) {
      gx = fma(wb, S[slm], gx);
      gy = fma(-wt, S[slm], gy);
      W[sll] = fma(x, wt, fma(y, wb, W[sll]));
      W[slm] = fma(x, wb, fma(-y, wt, W[slm]));
    }
#pragma unroll
    for (int m = -l; m <= l; ++m) {
      const int dst = (l + 1) * (l + 1) + (l + 1) + m;
      const int s1 = l * l + l + m;
      const T a = T((2.0 * l + 1.0) / sqrt((l + m + 1.0) * (l - m + 1.0)));
      const T wa = a * W[dst];
      gz = fma(wa, S[s1], gz);
      if (l > 0) W[s1] = fma(wa, z, W[s1]);
      if (m >= -(l - 1) && m <= l - 1) {
        const int s2 = (l - 1) * (l - 1) + (l - 1) + m;
        const T b = T(sqrt((l + m) * (l - m) * 1.0) / sqrt((l + m + 1.0) * (l - m + 1.0)));
        const T wc = b * W[dst];
        q = fma(wc, S[s2], q);
        if (l > 1) W[s2] -= wc;
      }
    }
  }
  gx = fma(T(-2) * x, q, gx);
  gy = fma(T(-2) * y, q, gy);
  gz = fma(T(-2) * z, q, gz);
}

// Reciprocal in the evaluation type: the hardware estimate (1 ulp) in float32, two Newton
// steps on it in float64.
template <class T>
__device__ __forceinline__ T rcp_t(T a) {
  if constexpr (sizeof(T) == 4) return __builtin_amdgcn_rcpf(a);
  else return rcp_nr(a);
}

__device__ __forceinline__ void taper_d(double x, double& p, double& dp) {
  const double x2 = x * x;
  const double x4 = x2 * x2;
  const double den = rcp_nr(1.0 + x4);
  p = x4 * den;
  dp = 4.0 * x2 * x * den * den;
}

template <class T>
__device__ __forceinline__ void taper_t(T x, T& p, T& dp) {
  const T x2 = x * x;
  const T x4 = x2 * x2;
  const T den = rcp_t<T>(T(1) + x4);
  p = x4 * den;
  dp = T(4) * x2 * x * den * den;
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// One step of the atomic base on the matrix cores: 16 x 16 outputs, four neighbour slots.
__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 d) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, d, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mfma16(double a, double b, doublex4 d) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0);
}

// LDS layout of the atomic-base kernel: per neighbour slot (columns, row stride kStride: rows and the
// slots of a step fall on distinct banks) the radial values g_k (NMAX rows) and solid harmonics S_lm;
// A' reuses the space once the contraction is done.  48 slots at a time (42 neighbours lie within 5 A in
// copper; more take a second round) leave room for more waves than 64 would.
template <class T, int LMAX, int NMAX>
struct BasisLds {
  static constexpr int LM = (LMAX + 1) * (LMAX + 1);
  static constexpr int kSlots = 48;
  static constexpr int kStride = sizeof(T) == 4 ? 52 : 50;
  static constexpr size_t bytes() { return sizeof(T) * (size_t)(NMAX + LM) * kStride; }
};

// ------------------------------------------------------------------ kernel 1
// One wave per active atom, lanes over its neighbours for the radial values and harmonics; the
// contraction over the neighbours inside the cutoff (compacted to the front) runs on the matrix cores of
// either type, rows = k, columns = lm.  Then a lane holds one lm of A' and mixes it for every other n, so
// that a column is read from LDS once.
// Bound by vector instructions in float32 and by the float64 matrix instructions (64 cycles for 1,024
// multiply-adds, of which K x (l_max + 1)^2 of 16 x 32 outputs are used).  Measured at (10, 4) (us):
// float32, 29,150 atoms 69 before / 44, 16,309 atoms 50 / 33; float64, 29,150 atoms 183 / 91 (on the vector
// unit each multiply-add read two values from LDS), 3,982 atoms 35 / 21.
template <class T, int LMAX, int NMAX>
__global__ void __launch_bounds__(64) k_ace_basis(const double* __restrict__ pos, int n, BoxDev b,
                                                  const int* __restrict__ count, const int* __restrict__ idx,
                                                  int max_nb, const int* __restrict__ active, int n_act,
                                                  int K, double rc, double inv_h, double rc2,
                                                  const T* __restrict__ Wp,
                                                  AnchorDev an, AceScratch<T> sc) {
  constexpr int LM = (LMAX + 1) * (LMAX + 1);
  constexpr int ST = BasisLds<T, LMAX, NMAX>::kStride, kSlots = BasisLds<T, LMAX, NMAX>::kSlots;
  using V4 = std::conditional_t<sizeof(T) == 4, floatx4, doublex4>;
  extern __shared__ double smem_raw[];
  T* gS = reinterpret_cast<T*>(smem_raw);  // [NMAX][ST]: g_k per neighbour slot
  T* sS = gS + NMAX * ST;                  // [LM][ST]: S_lm per neighbour slot
  T* Ap = gS;                              // [K][LM], after the contraction
  __shared__ double etab[32];
  const int q = xcd_block(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x;
  const int i = active[q];
  if (an.on) stage_exp_table(etab);
  const double xi = pos[i], yi = pos[(size_t)n + i], zi = pos[2 * (size_t)n + i];
  int cnt = count[i];
  if (cnt > max_nb) cnt = max_nb;
  const int col = lane & 15, sub = lane >> 4;
  V4 D0 = {T(0), T(0), T(0), T(0)}, D1 = {T(0), T(0), T(0), T(0)};
  double rho_a = 0.0, pair_a = 0.0;
  const double two_rc = 2.0 / rc;
  for (int c0 = 0; c0 < cnt; c0 += 64) {
    const int k = c0 + lane;
    T g[NMAX];
    T S[LM];
    bool inside = false;
#pragma unroll
    for (int a = 0; a < NMAX; ++a) g[a] = T(0);
#pragma unroll
    for (int a = 0; a < LM; ++a) S[a] = T(0);
    if (k < cnt) {
      const int j = idx[(size_t)k * n + i];
      const double dx = min_image_sel(pos[j] - xi, b.L[0], b.half[0], b.per[0]);
      const double dy = min_image_sel(pos[(size_t)n + j] - yi, b.L[1], b.half[1], b.per[1]);
      const double dz = min_image_sel(pos[2 * (size_t)n + j] - zi, b.L[2], b.half[2], b.per[2]);
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double ird = rsq_nr(r2);
      const double rd = r2 * ird;
      inside = r2 < rc2;
      if (inside) {
        // (rounded to T once, here and in the direction: the polynomials magnify an error of their argument.
        // From a rounded distance the float32 forces were off by 2.7 times as much, for the same time)
        const T x = T(rd * two_rc - 1.0);
        T ps, dps;
        taper_t<T>(T((rd - rc) * inv_h), ps, dps);
        T t0 = T(1), t1 = x;
        g[0] = ps;
        g[1] = x * ps;
#pragma unroll
        for (int a = 2; a < NMAX; ++a) {
          const T t2 = T(2) * x * t1 - t0;
          g[a] = t2 * ps;
          t0 = t1;
          t1 = t2;
        }
        solid_harmonics<T, LMAX>(T(dx * ird), T(dy * ird), T(dz * ird), S);
      }
      if (an.on && r2 < an.rc2) {
        double ps, dps;
        taper_d((rd - an.rc) * an.inv_h, ps, dps);
        rho_a += exp_tab(-an.beta * (rd - an.r0), etab) * ps;
        pair_a += exp_tab(-an.alpha * (rd - an.r0), etab) * ps;
      }
    }
    // the neighbours inside the cutoff take the first slots, the next ones (all zero) fill up the last
    // step of four
    const unsigned long long m = __ballot(inside);
    const int nv = __popcll(m), steps = (nv + 3) >> 2;
    const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    const int slot = inside ? below : nv + (lane - below);
    // lane = row / column (lane % 16) and slot in the step (lane / 16); rows past NMAX and columns past
    // LM repeat others, and what they give is not used
    const T* ga = gS + (col < NMAX ? col : 0) * ST + sub;
    const T* sa = sS + col * ST + sub;
    const T* sb = sS + (16 + col < LM ? 16 + col : col) * ST + sub;
    for (int at = 0; at < 4 * steps; at += kSlots) {
      const int end = 4 * steps - at < kSlots ? 4 * steps - at : kSlots;
      if (slot >= at && slot < at + end) {
#pragma unroll
        for (int a = 0; a < NMAX; ++a) gS[a * ST + slot - at] = g[a];
#pragma unroll
        for (int a = 0; a < LM; ++a) sS[a * ST + slot - at] = S[a];
      }
      __syncthreads();
      for (int st = 0; st < end; st += 4) {
        const T av = ga[st];
        D0 = mfma16(av, sa[st], D0);
        if constexpr (LM > 16) D1 = mfma16(av, sb[st], D1);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    // accumulator layout: column lane % 16 (+ 16 for D1), row 4 (lane / 16) + r in float32,
    // 4 r + lane / 16 in float64
    const int k = sizeof(T) == 4 ? 4 * sub + r : 4 * r + sub;
    if (k < K) {
      Ap[k * LM + col] = D0[r];
      if (16 + col < LM) Ap[k * LM + 16 + col] = D1[r];
    }
  }
  __syncthreads();
  const int half = lane >> 5, lm = lane & 31;
  if (lm < LM) {
    int l = 0;
#pragma unroll
    for (int t = 1; t <= LMAX; ++t) l += lm >= t * t ? 1 : 0;
    T a[NMAX];
#pragma unroll
    for (int kk = 0; kk < NMAX; ++kk) a[kk] = kk < K ? Ap[kk * LM + lm] : T(0);
    T* Arow = sc.A + (size_t)q * sc.stride + lm;
    constexpr int H = (NMAX + 1) / 2;
    T v[H];
    auto mix = [&](auto full_c) {  // (full: whole rows of the table, read in wide loads)
      constexpr bool FULL = decltype(full_c)::value;
      const int kc = FULL ? NMAX : K;
      const T* wl = Wp + (size_t)l * kc * kc;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int nn = 2 * h + half, row = nn < kc ? nn : 0;
        v[h] = T(0);
#pragma unroll
        for (int kk = 0; kk < NMAX; ++kk) v[h] = fma(wl[row * kc + (FULL || kk < K ? kk : 0)], a[kk], v[h]);
      }
    };
    if (K == NMAX)
      mix(std::true_type{});
    else
      mix(std::false_type{});
#pragma unroll
    for (int h = 0; h < H; ++h)
      if (2 * h + half < K) Arow[(2 * h + half) * LM] = v[h];
  }
  if (an.on) {
    rho_a = wave_sum_dpp(rho_a);
    pair_a = wave_sum_dpp(pair_a);
    if (lane == 0) {
      const double sq = sqrt(rho_a);
      sc.e_anch[q] = (rho_a > 0.0 ? -sq : 0.0) + 0.5 * an.A * pair_a;
      sc.fp_anch[q] = rho_a > 0.0 ? -0.5 / sq : 0.0;
    }
  } else if (lane == 0) {
    sc.e_anch[q] = 0.0;
    sc.fp_anch[q] = 0.0;
  }
}

// ------------------------------------------------------------------ kernel 2
// Ā' of one atom in LDS: lm-major rows of KP radial values (K rounded up to whole 16-byte
// groups, the padding zero), so that a row is read by a few wide broadcast loads.
template <class T, int NMAX>
struct ForceLds {
  static constexpr int KP = (NMAX * (int)sizeof(T) + 15) / 16 * 16 / (int)sizeof(T);
};

// One wave per active atom, lanes over its neighbours.  The scatter is what bounds it: 162 float64
// atomics per atom, which the L2 takes a cache line at a time.  PACKED: the wave's contributions are
// turned in LDS so that three neighbouring lanes add the three components of one atom, 32 bytes apart
// from the next (fp[n][4]), instead of three instructions of 64 lanes on 64 lines each; k_unpack lays the
// sums out.  Measured at (10, 4), per component / packed (us): float32, 16,309 atoms 78 / 62, float64,
// 29,150 atoms 176 / 129 (without any scatter 43 and 123).
// Float32 is held to 128 VGPRs, four waves per SIMD.
template <class T, int LMAX, int NMAX, bool PACKED>
__global__ void __launch_bounds__(64, sizeof(T) == 4 ? 4 : 1) k_ace_force(const double* __restrict__ pos, int n, BoxDev b,
                                                  const int* __restrict__ count, const int* __restrict__ idx,
                                                  int max_nb, const int* __restrict__ active, int n_act, int K,
                                                  double rc, double inv_h, double rc2, AnchorDev an,
                                                  AceScratch<T> sc, const double* __restrict__ w,
                                                  double* __restrict__ f, const double* __restrict__ w2,
                                                  double* __restrict__ f2) {
  constexpr int LM = (LMAX + 1) * (LMAX + 1);
  constexpr int kMaxK = NMAX;
  constexpr int KP = ForceLds<T, NMAX>::KP;
  extern __shared__ double smem_raw[];
  T* Ab2 = reinterpret_cast<T*>(smem_raw);  // [LM][KP]: Ab2[lm * KP + k], zero for k >= K
  __shared__ double etab[32];
  __shared__ double turn[PACKED ? 192 : 1];
  __shared__ int turn_j[PACKED ? 64 : 1];
  if (an.on) stage_exp_table(etab);
  const int q = xcd_block(blockIdx.x, gridDim.x);
  const double two_rc = 2.0 / rc;
  const int lane = threadIdx.x;
  const int i = active[q];
  const double wi = w ? w[i] : 1.0;
  // second weight set (the integrator's weight difference): scattered only where non-zero
  const double w2i = f2 ? w2[i] : 0.0;
  const int na = K * LM;
  for (int o = lane; o < LM * KP; o += 64) Ab2[o] = T(0);
  __syncthreads();
  const T* B = sc.B + (size_t)q * sc.stride;
  for (int o = lane; o < na; o += 64) {
    const int lm = o / K;
    Ab2[lm * KP + o - lm * K] = B[o];
  }
  __syncthreads();
  const double fpa = an.on ? sc.fp_anch[q] : 0.0;
  const double xi = pos[i], yi = pos[(size_t)n + i], zi = pos[2 * (size_t)n + i];
  int cnt = count[i];
  if (cnt > max_nb) cnt = max_nb;
  double fix = 0.0, fiy = 0.0, fiz = 0.0;
  double f2x = 0.0, f2y = 0.0, f2z = 0.0;
  for (int c0 = 0; c0 < cnt; c0 += 64) {
    const int k = c0 + lane;
    double gx = 0.0, gy = 0.0, gz = 0.0;
    int j = i;
    if (k < cnt) {
      j = idx[(size_t)k * n + i];
      const double dx = min_image_sel(pos[j] - xi, b.L[0], b.half[0], b.per[0]);
      const double dy = min_image_sel(pos[(size_t)n + j] - yi, b.L[1], b.half[1], b.per[1]);
      const double dz = min_image_sel(pos[2 * (size_t)n + j] - zi, b.L[2], b.half[2], b.per[2]);
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double ird = rsq_nr(r2);
      const double rd = r2 * ird;
      if (r2 < rc2) {
        const T ir = T(ird);
        const T ux = T(dx * ird), uy = T(dy * ird), uz = T(dz * ird);
        const T dxdr = T(two_rc);
        const T x = T(rd * two_rc - 1.0);
        T ps, dps;
        taper_t<T>(T((rd - rc) * inv_h), ps, dps);
        dps *= T(inv_h);
        T g[kMaxK], gd[kMaxK];
        T t0 = T(1), t1 = x, d0 = T(0), d1 = T(1);
        g[0] = ps;
        gd[0] = dps;
        g[1] = x * ps;
        gd[1] = d1 * dxdr * ps + x * dps;
#pragma unroll
        for (int a = 2; a < kMaxK; ++a) {
          const T t2 = T(2) * x * t1 - t0;
          const T d2 = T(2) * t1 + T(2) * x * d1 - d0;
          g[a] = t2 * ps;
          gd[a] = d2 * dxdr * ps + t2 * dps;
          t0 = t1;
          t1 = t2;
          d0 = d1;
          d1 = d2;
        }
        T S[LM], W[LM];
        solid_harmonics<T, LMAX>(ux, uy, uz, S);
        T radial = T(0);
#pragma unroll
        for (int lm = 0; lm < LM; ++lm) {
          // the row is the same for every lane (broadcast); entries beyond K are zero
          T c[KP];
#pragma unroll
          for (int kk = 0; kk < KP; kk += 16 / (int)sizeof(T)) {
            if constexpr (sizeof(T) == 4) {
              const float4 v = *reinterpret_cast<const float4*>(&Ab2[lm * KP + kk]);
              c[kk] = v.x;
              c[kk + 1] = v.y;
              c[kk + 2] = v.z;
              c[kk + 3] = v.w;
            } else {
              const double2 v = *reinterpret_cast<const double2*>(&Ab2[lm * KP + kk]);
              c[kk] = v.x;
              c[kk + 1] = v.y;
            }
          }
          T av = T(0), bv = T(0);
#pragma unroll
          for (int kk = 0; kk < NMAX; ++kk) {
            av = fma(c[kk], g[kk], av);
            bv = fma(c[kk], gd[kk], bv);
          }
          radial = fma(bv, S[lm], radial);
          W[lm] = av;
        }
        // sum_lm av S_lm depends on the direction only: its gradient is the one in (x, y, z), less the
        // part along the direction, over r
        T vx, vy, vz;
        harmonics_gradient<T, LMAX>(ux, uy, uz, S, W, vx, vy, vz);
        radial -= (vx * ux + vy * uy + vz * uz) * ir;
        gx = (double)fma(radial, ux, vx * ir);
        gy = (double)fma(radial, uy, vy * ir);
        gz = (double)fma(radial, uz, vz * ir);
      }
      if (an.on && r2 < an.rc2) {
        double ps, dps;
        taper_d((rd - an.rc) * an.inv_h, ps, dps);
        dps *= an.inv_h;
        const double eb = exp_tab(-an.beta * (rd - an.r0), etab);
        const double ea = exp_tab(-an.alpha * (rd - an.r0), etab);
        const double drho = eb * (dps - an.beta * ps);
        const double dphi = an.A * ea * (dps - an.alpha * ps);
        const double s = (fpa * drho + 0.5 * dphi) * ird;
        gx += s * dx;
        gy += s * dy;
        gz += s * dz;
      }
      if (w2i != 0.0) {
        const double hx = gx * w2i, hy = gy * w2i, hz = gz * w2i;
        if (hx != 0.0 || hy != 0.0 || hz != 0.0) {
          unsafeAtomicAdd(&f2[j], -hx);
          unsafeAtomicAdd(&f2[(size_t)n + j], -hy);
          unsafeAtomicAdd(&f2[2 * (size_t)n + j], -hz);
        }
        f2x += hx;
        f2y += hy;
        f2z += hz;
      }
      gx *= wi;
      gy *= wi;
      gz *= wi;
      if (!PACKED && (gx != 0.0 || gy != 0.0 || gz != 0.0)) {
        unsafeAtomicAdd(&f[j], -gx);
        unsafeAtomicAdd(&f[(size_t)n + j], -gy);
        unsafeAtomicAdd(&f[2 * (size_t)n + j], -gz);
      }
      fix += gx;
      fiy += gy;
      fiz += gz;
    }
    if constexpr (PACKED) {
      turn[3 * lane] = -gx;
      turn[3 * lane + 1] = -gy;
      turn[3 * lane + 2] = -gz;
      turn_j[lane] = j;
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        const int e = 64 * h + lane, s = e / 3, c = e - 3 * s;
        const double v = turn[e];
        if (v != 0.0) unsafeAtomicAdd(&f[4 * (size_t)turn_j[s] + c], v);
      }
      __syncthreads();
    }
  }
  fix = wave_sum_dpp(fix);
  fiy = wave_sum_dpp(fiy);
  fiz = wave_sum_dpp(fiz);
  if (PACKED ? lane < 3 : lane == 0) {
    if constexpr (PACKED) {
      unsafeAtomicAdd(&f[4 * (size_t)i + lane], lane == 0 ? fix : (lane == 1 ? fiy : fiz));
    } else {
      unsafeAtomicAdd(&f[i], fix);
      unsafeAtomicAdd(&f[(size_t)n + i], fiy);
      unsafeAtomicAdd(&f[2 * (size_t)n + i], fiz);
    }
  }
  if (w2i != 0.0) {  // uniform across the wave
    f2x = wave_sum_dpp(f2x);
    f2y = wave_sum_dpp(f2y);
    f2z = wave_sum_dpp(f2z);
    if (lane == 0) {
      unsafeAtomicAdd(&f2[i], f2x);
      unsafeAtomicAdd(&f2[(size_t)n + i], f2y);
      unsafeAtomicAdd(&f2[2 * (size_t)n + i], f2z);
    }
  }
}

__global__ void k_fill_zero(double* __restrict__ p, long long m) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) p[i] = 0.0;
}

// f[3][n] from fp[n][4].
__global__ void k_unpack(const double* __restrict__ fp, int n, double* __restrict__ f) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 xy = reinterpret_cast<const double2*>(fp)[2 * (size_t)i];
  f[i] = xy.x;
  f[(size_t)n + i] = xy.y;
  f[2 * (size_t)n + i] = fp[4 * (size_t)i + 2];
}

// Forces gathered as [n][4] first: a packed scatter saves about 1 ns per active atom; clearing the third
// more and unpacking cost 4 us and 0.02 ns per atom.  Float32 with these passes, direct / packed (us):
// 16,309 active atoms 78 / 67, 29,150 of 130,466 123 / 86; below 8,192 the saving is no larger than a
// launch.
constexpr int kPackedLeast = 8192, kPackedShare = 32;
bool packed_forces(int n, int n_act) { return n_act >= kPackedLeast && n_act >= n / kPackedShare; }

template <class T, int LMAX>
apx_status ace_run(apx_ctx* ctx, const apx_atoms* atoms, const apx_nlist* nl, const apx_ace_model* m,
                   const double* w, const int* active, int n_act, double* e_site,
                   double* f, double* dc1, double* dc2, apx::DevBuf& buf, const double* w2 = nullptr,
                   double* f2 = nullptr) {
  constexpr int LM = (LMAX + 1) * (LMAX + 1);
  const int n = (int)atoms->n;
  const SymTables<T>& tb = sym_tables<T>(m);
  AceScratch<T> sc;
  sc.stride = sym_stride(m->na);
  // the projected adjoint overwrites the atomic base, which only the coefficient gradients need
  // afterwards (with the embedding's slopes)
  auto whole = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t bytes_A = whole(sizeof(T) * (size_t)n_act * sc.stride);
  const size_t bytes_anch = whole(sizeof(double) * 2 * (size_t)n_act);
  const size_t bytes_slope = dc1 ? whole(sizeof(T) * (size_t)n_act) : 0;
  const size_t bytes_more = std::max(sym_scratch<T>(m, n_act), dc1 ? ace_grad_scratch(m, n_act) : 0);
  const bool packed = packed_forces(n, n_act);
  const size_t bytes_fp = packed ? whole(sizeof(double) * 4 * (size_t)n) : 0;
  const size_t need = (dc1 ? 2 : 1) * bytes_A + bytes_anch + bytes_slope + bytes_fp + bytes_more;
  // What is allocated grows with n_act alone and is no less in float64 than in float32, so that after a
  // call no other of at most its n_act allocates (and can be recorded into a graph): whatever its number
  // of atoms, with or without coefficient gradients, and where fewer tiles' pairs are shared among blocks.
  const size_t most = 2 * bytes_A + bytes_anch + whole(sizeof(T) * (size_t)n_act) +
                      (n_act >= kPackedLeast ? whole(sizeof(double) * 4 * kPackedShare * ((size_t)n_act + 1)) : 0) +
                      std::max(sym_scratch_most(m, n_act), ace_grad_scratch(m, n_act));
  if (buf.bytes < need && buf.ensure(std::max(need, most)) != hipSuccess) {
    (void)hipGetLastError();
    APX_ALLOC(ctx, buf, need);
  }
  char* p = static_cast<char*>(buf.p);
  auto take = [&](size_t b) {
    char* at = p;
    p += b;
    return at;
  };
  sc.A = reinterpret_cast<T*>(take(bytes_A));
  T* B = dc1 ? reinterpret_cast<T*>(take(bytes_A)) : sc.A;
  sc.B = B;
  sc.e_anch = reinterpret_cast<double*>(take(bytes_anch));
  sc.fp_anch = sc.e_anch + n_act;
  T* slope = dc1 ? reinterpret_cast<T*>(take(bytes_slope)) : nullptr;
  double* fp = packed ? reinterpret_cast<double*>(take(bytes_fp)) : nullptr;
  void* more = p;
  if (packed) k_fill_zero<<<blocks_for(4LL * n, 256), 256, 0, ctx->stream>>>(fp, 4LL * n);
  BoxDev b = make_box(atoms);
  AnchorDev an{};
  an.on = m->anchored;
  if (an.on) {
    an.A = m->anchor.A;
    an.alpha = m->anchor.alpha;
    an.beta = m->anchor.beta;
    an.r0 = m->anchor.r0;
    an.rc = m->anchor.r_cut;
    an.inv_h = 1.0 / m->anchor.h;
    an.rc2 = m->anchor.r_cut * m->anchor.r_cut;
  }
  const double rc = m->r_cut, inv_h = 1.0 / m->h;
  const double rc2 = m->r_cut * m->r_cut;
  auto by_radial = [&](auto body) {
    if (m->n_max <= 8) body(std::integral_constant<int, 8>{});
    else if (m->n_max <= 10) body(std::integral_constant<int, 10>{});
    else body(std::integral_constant<int, 12>{});
  };
  {
    ProfScope ps(ctx, "ace.basis");
    by_radial([&](auto nmax_c) {
      constexpr int NM = decltype(nmax_c)::value;
      k_ace_basis<T, LMAX, NM><<<n_act, 64, BasisLds<T, LMAX, NM>::bytes(), ctx->stream>>>(
          atoms->pos, n, b, nl->count, nl->idx, nl->max_nb, active, n_act, m->n_max, rc, inv_h, rc2, tb.Wp, an, sc);
    });
    APX_LAUNCH_CHECK(ctx);
  }
  apx_status s = sym_products<T>(ctx, m, sc.A, B, slope, n_act, sc.e_anch, active, e_site, more);
  if (s == APX_OK && dc1) s = ace_grad<T>(ctx, m, sc.A, slope, w, active, n_act, dc1, dc2, more);
  if (s != APX_OK) return s;
  ProfScope ps(ctx, "ace.force");
  by_radial([&](auto nmax_c) {
    constexpr int NM = decltype(nmax_c)::value;
    const size_t lds3 = sizeof(T) * (size_t)ForceLds<T, NM>::KP * LM;
    auto launch = [&](auto kern, double* out) {
      kern<<<n_act, 64, lds3, ctx->stream>>>(atoms->pos, n, b, nl->count, nl->idx, nl->max_nb, active, n_act, m->n_max,
                                             rc, inv_h, rc2, an, sc, w, out, w2, f2);
    };
    if (packed)
      launch(k_ace_force<T, LMAX, NM, true>, fp);
    else
      launch(k_ace_force<T, LMAX, NM, false>, f);
  });
  if (packed) k_unpack<<<blocks_for(n, 256), 256, 0, ctx->stream>>>(fp, n, f);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

}  // namespace apx

using namespace apx;

namespace {
apx::DevBuf& ace_buffer(apx_ctx* ctx) { return ctx->ace_buf; }
}  // namespace

namespace {
apx_status ace_impl(apx_ctx* ctx, const apx_atoms* atoms, const apx_nlist* nl, const apx_ace_model* m, const double* w,
                    const int32_t* active, int64_t n_active, int32_t precision, double* e_site, double* f,
                    double* dE_dc1, double* dE_dc2, const double* w2, double* f2) {
  if (!ctx) return APX_EINVAL;
  apx_status s = check_atoms(ctx, atoms);
  if (s != APX_OK) return s;
  if (!nl || !m) return fail(ctx, APX_EINVAL, "nl and model are required");
  if (nl->n != atoms->n) return fail(ctx, APX_EINVAL, "nlist size mismatch");
  if (nl->max_nb < 1 || nl->max_nb > 128) return fail(ctx, APX_EINVAL, "nlist max_nb must be in 1..128");
  if (m->r_cut > nl->r_list || (m->anchored && m->anchor.r_cut > nl->r_list))
    return fail(ctx, APX_EINVAL, "ACE cutoff exceeds the neighbour-list cutoff");
  if (precision != APX_FP64 && precision != APX_FP32) return fail(ctx, APX_EINVAL, "precision must be APX_FP64 or APX_FP32");
  if (n_active < 0 || n_active > atoms->n) return fail(ctx, APX_EINVAL, "n_active out of range");
  if ((dE_dc1 == nullptr) != (dE_dc2 == nullptr)) return fail(ctx, APX_EINVAL, "dE_dc1 and dE_dc2 go together");
  const int n = (int)atoms->n;
  if (n > 0 && (!e_site || !f)) return fail(ctx, APX_EINVAL, "e_site and f are required");
  if (n_active > 0 && !active) return fail(ctx, APX_EINVAL, "active is NULL");
  if (n > 0) {
    if (!packed_forces(n, (int)n_active)) k_fill_zero<<<blocks_for(3LL * n, 256), 256, 0, ctx->stream>>>(f, 3LL * n);
    k_fill_zero<<<blocks_for(n, 256), 256, 0, ctx->stream>>>(e_site, n);
    if (f2) k_fill_zero<<<blocks_for(3LL * n, 256), 256, 0, ctx->stream>>>(f2, 3LL * n);
    APX_LAUNCH_CHECK(ctx);
  }
  if (dE_dc1) {
    k_fill_zero<<<blocks_for(m->n_basis, 256), 256, 0, ctx->stream>>>(dE_dc1, m->n_basis);
    k_fill_zero<<<blocks_for(m->n_basis, 256), 256, 0, ctx->stream>>>(dE_dc2, m->n_basis);
    APX_LAUNCH_CHECK(ctx);
  }
  if (n_active == 0) return APX_OK;
  const int na_ = (int)n_active;
  if (precision == APX_FP64) {
    if (m->l_max == 3)
      return ace_run<double, 3>(ctx, atoms, nl, m, w, active, na_, e_site, f, dE_dc1, dE_dc2, ace_buffer(ctx),
                                w2, f2);
    return ace_run<double, 4>(ctx, atoms, nl, m, w, active, na_, e_site, f, dE_dc1, dE_dc2, ace_buffer(ctx),
                              w2, f2);
  }
  if (m->l_max == 3)
    return ace_run<float, 3>(ctx, atoms, nl, m, w, active, na_, e_site, f, dE_dc1, dE_dc2, ace_buffer(ctx),
                             w2, f2);
  return ace_run<float, 4>(ctx, atoms, nl, m, w, active, na_, e_site, f, dE_dc1, dE_dc2, ace_buffer(ctx),
                           w2, f2);
}
}  // namespace

namespace apx {
apx_status ace_energy_forces_dual(apx_ctx* ctx, const apx_atoms* atoms, const apx_nlist* nl, const apx_ace_model* m,
                                  const double* w, const double* w2, const int32_t* active, int64_t n_active,
                                  int32_t precision, double* e_site, double* f, double* f2) {
  if (!w2 || !f2) return fail(ctx, APX_EINVAL, "the second weight set and its force array are required");
  return ace_impl(ctx, atoms, nl, m, w, active, n_active, precision, e_site, f, nullptr, nullptr, w2, f2);
}
}  // namespace apx

extern "C" apx_status apx_ace_energy_forces(apx_ctx* ctx, const apx_atoms* atoms, const apx_nlist* nl,
                                            const apx_ace_model* m, const double* w, const int32_t* active,
                                            int64_t n_active, int32_t precision, double* e_site, double* f,
                                            double* dE_dc1, double* dE_dc2) {
  return ace_impl(ctx, atoms, nl, m, w, active, n_active, precision, e_site, f, dE_dc1, dE_dc2, nullptr, nullptr);
}
