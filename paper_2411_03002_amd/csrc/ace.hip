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
template <class T, int LMAX, bool GRAD>
__device__ __forceinline__ void solid_harmonics(T x, T y, T z, T* S, T* Sx, T* Sy, T* Sz) {
  S[0] = T(1);
  if constexpr (GRAD) { Sx[0] = T(0); Sy[0] = T(0); Sz[0] = T(0); }
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
      if constexpr (GRAD) {
        Sx[tp] = c * S[sll]; Sy[tp] = T(0); Sz[tp] = T(0);
        Sx[bt] = T(0); Sy[bt] = c * S[sll]; Sz[bt] = T(0);
      }
    } else {
      S[tp] = c * (x * S[sll] - y * S[slm]);
      S[bt] = c * (y * S[sll] + x * S[slm]);
      if constexpr (GRAD) {
        Sx[tp] = c * (S[sll] + x * Sx[sll] - y * Sx[slm]);
        Sy[tp] = c * (x * Sy[sll] - S[slm] - y * Sy[slm]);
        Sz[tp] = c * (x * Sz[sll] - y * Sz[slm]);
        Sx[bt] = c * (y * Sx[sll] + S[slm] + x * Sx[slm]);
        Sy[bt] = c * (S[sll] + y * Sy[sll] + x * Sy[slm]);
        Sz[bt] = c * (y * Sz[sll] + x * Sz[slm]);
      }
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
        if constexpr (GRAD) {
          Sx[dst] = a * z * Sx[s1] - b * (T(2) * x * S[s2] + Sx[s2]);
          Sy[dst] = a * z * Sy[s1] - b * (T(2) * y * S[s2] + Sy[s2]);
          Sz[dst] = a * (S[s1] + z * Sz[s1]) - b * (T(2) * z * S[s2] + Sz[s2]);
        }
      } else {
        S[dst] = a * z * S[s1];
        if constexpr (GRAD) {
          Sx[dst] = a * z * Sx[s1];
          Sy[dst] = a * z * Sy[s1];
          Sz[dst] = a * (S[s1] + z * Sz[s1]);
        }
      }
    }
  }
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

// LDS layout of the atomic-base kernel: per neighbour slot (columns, row stride kStride)
// the radial values g_k (12 rows) and solid harmonics S_lm (LM rows); A' reuses the space
// once the contraction is done.  Float32 contracts on the matrix cores.
template <class T, int LMAX>
struct BasisLds {
  static constexpr int LM = (LMAX + 1) * (LMAX + 1);
  static constexpr bool kMfma = sizeof(T) == 4;
  static constexpr int kStride = kMfma ? 66 : 65;
  static constexpr int kGRows = 12;
  static constexpr int kSRows = LM;
  static constexpr size_t bytes() { return sizeof(T) * ((size_t)(kGRows + kSRows) * kStride); }
  static_assert(12 * LM <= (kGRows + kSRows) * kStride, "A' fits in the neighbour tables");
};

// ------------------------------------------------------------------ kernel 1
template <class T, int LMAX>
__global__ void __launch_bounds__(64) k_ace_basis(const double* __restrict__ pos, int n, BoxDev b,
                                                  const int* __restrict__ count, const int* __restrict__ idx,
                                                  int max_nb, const int* __restrict__ active, int n_act,
                                                  int K, T rc, T inv_h, double rc2, const T* __restrict__ Wp,
                                                  AnchorDev an, AceScratch<T> sc) {
  constexpr int LM = (LMAX + 1) * (LMAX + 1);
  constexpr int kMaxK = 12;
  constexpr bool MF = BasisLds<T, LMAX>::kMfma;
  constexpr int ST = BasisLds<T, LMAX>::kStride, GR = BasisLds<T, LMAX>::kGRows, SR = BasisLds<T, LMAX>::kSRows;
  extern __shared__ double smem_raw[];
  T* gS = reinterpret_cast<T*>(smem_raw);  // [GR][ST]: g_k per neighbour slot
  T* sS = gS + GR * ST;                    // [SR][ST]: S_lm per neighbour slot
  T* Ap = gS;                              // [K*LM], after the contraction
  __shared__ double etab[32];
  stage_exp_table(etab);
  const int q = xcd_block(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x;
  const int i = active[q];
  const double xi = pos[i], yi = pos[(size_t)n + i], zi = pos[2 * (size_t)n + i];
  int cnt = count[i];
  if (cnt > max_nb) cnt = max_nb;
  const int nout = K * LM;
  T acc[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) acc[s] = T(0);
  floatx4 D0 = {0.f, 0.f, 0.f, 0.f}, D1 = {0.f, 0.f, 0.f, 0.f};
  double rho_a = 0.0, pair_a = 0.0;
  const T two_rc = T(2) / rc;
  for (int c0 = 0; c0 < cnt; c0 += 64) {
    const int k = c0 + lane;
    T g[kMaxK];
    T S[LM];
    bool inside = false;
#pragma unroll
    for (int a = 0; a < kMaxK; ++a) g[a] = T(0);
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
        const T r = T(rd);
        const T ir = T(ird);
        const T x = r * two_rc - T(1);
        T ps, dps;
        taper_t<T>((r - rc) * inv_h, ps, dps);
        T t0 = T(1), t1 = x;
        g[0] = ps;
        if (K > 1) g[1] = x * ps;
#pragma unroll
        for (int a = 2; a < kMaxK; ++a) {
          const T t2 = T(2) * x * t1 - t0;
          if (a < K) g[a] = t2 * ps;
          t0 = t1;
          t1 = t2;
        }
        solid_harmonics<T, LMAX, false>(T(dx) * ir, T(dy) * ir, T(dz) * ir, S, nullptr, nullptr, nullptr);
      }
      if (an.on && r2 < an.rc2) {
        double ps, dps;
        taper_d((rd - an.rc) * an.inv_h, ps, dps);
        rho_a += exp_tab(-an.beta * (rd - an.r0), etab) * ps;
        pair_a += exp_tab(-an.alpha * (rd - an.r0), etab) * ps;
      }
    }
    // neighbour slot of the lane: float32 compacts the neighbours inside the cutoff to the
    // front (the others, all zero, follow), so that the matrix steps stop after them
    int slot = lane, steps = 0;
    if constexpr (MF) {
      const unsigned long long m = __ballot(inside);
      const int nv = __popcll(m);
      const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      slot = inside ? below : nv + (lane - below);
      steps = (nv + 3) >> 2;
    }
#pragma unroll
    for (int a = 0; a < kMaxK; ++a)
      if (a < K) gS[a * ST + slot] = g[a];
#pragma unroll
    for (int a = 0; a < LM; ++a) sS[a * ST + slot] = S[a];
    __syncthreads();
    if constexpr (MF) {
      // A'[k][lm] += sum over 4 slots per step of g[k][slot] S[lm][slot] on the matrix
      // cores (16 x 16 x 4 float32): lane = row/column (lane % 16) and slot in the step
      // (lane / 16), operand rows beyond K and LM are zero; the row stride of 66 keeps
      // the two lane halves on distinct banks
      const int col = lane & 15, sub = lane >> 4;
      const bool g_row = col < K, s_row = 16 + col < LM;
      for (int st = 0; st < steps; ++st) {
        const int sl = 4 * st + sub;
        const float av = g_row ? gS[col * ST + sl] : 0.f;
        D0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av, sS[col * ST + sl], D0, 0, 0, 0);
        if constexpr (LM > 16)
          D1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av, s_row ? sS[(16 + col) * ST + sl] : 0.f, D1, 0, 0, 0);
      }
    } else {
      const int lim = (cnt - c0) < 64 ? (cnt - c0) : 64;
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int o = lane + 64 * s;
        if (o < nout) {
          const int kk = o / LM, lm = o - kk * LM;
          T v = acc[s];
          for (int nb = 0; nb < lim; ++nb) v += gS[kk * ST + nb] * sS[lm * ST + nb];
          acc[s] = v;
        }
      }
    }
    __syncthreads();
  }
  if constexpr (MF) {
    // accumulator layout: row k = 4 (lane / 16) + r, column lane % 16 (+ 16 for D1)
    const int col = lane & 15, sub = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = 4 * sub + r;
      if (k < K) {
        Ap[k * LM + col] = D0[r];
        if (16 + col < LM) Ap[k * LM + 16 + col] = D1[r];
      }
    }
  } else {
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      const int o = lane + 64 * s;
      if (o < nout) Ap[o] = acc[s];
    }
  }
  __syncthreads();
  const int na = K * LM;
  T* Arow = sc.A + (size_t)q * sc.stride;
  for (int o = lane; o < na; o += 64) {
    const int nn = o / LM, lm = o - nn * LM;
    int l = 0;
    while ((l + 1) * (l + 1) <= lm) ++l;
    const T* w = Wp + ((size_t)l * K + nn) * K;
    T v = T(0);
    for (int kk = 0; kk < K; ++kk) v += w[kk] * Ap[kk * LM + lm];
    Arow[o] = v;
  }
  if (an.on) {
    rho_a = wave_sum(rho_a);
    pair_a = wave_sum(pair_a);
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

// Float32 is held to 128 VGPRs, four waves per SIMD (a few registers spill; three waves left
// the gathers' latency exposed).
template <class T, int LMAX, int NMAX>
__global__ void __launch_bounds__(64, sizeof(T) == 4 ? 4 : 1) k_ace_force(const double* __restrict__ pos, int n, BoxDev b,
                                                  const int* __restrict__ count, const int* __restrict__ idx,
                                                  int max_nb, const int* __restrict__ active, int n_act, int K,
                                                  T rc, T inv_h, double rc2, AnchorDev an,
                                                  AceScratch<T> sc, const double* __restrict__ w,
                                                  double* __restrict__ f, const double* __restrict__ w2,
                                                  double* __restrict__ f2) {
  constexpr int LM = (LMAX + 1) * (LMAX + 1);
  constexpr int kMaxK = NMAX;
  constexpr int KP = ForceLds<T, NMAX>::KP;
  extern __shared__ double smem_raw[];
  T* Ab2 = reinterpret_cast<T*>(smem_raw);  // [LM][KP]: Ab2[lm * KP + k], zero for k >= K
  __shared__ double etab[32];
  stage_exp_table(etab);
  const int q = xcd_block(blockIdx.x, gridDim.x);
  const T two_rc = T(2) / rc;
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
    if (k < cnt) {
      const int j = idx[(size_t)k * n + i];
      const double dx = min_image_sel(pos[j] - xi, b.L[0], b.half[0], b.per[0]);
      const double dy = min_image_sel(pos[(size_t)n + j] - yi, b.L[1], b.half[1], b.per[1]);
      const double dz = min_image_sel(pos[2 * (size_t)n + j] - zi, b.L[2], b.half[2], b.per[2]);
      const double r2 = dx * dx + dy * dy + dz * dz;
      double gx = 0.0, gy = 0.0, gz = 0.0;
      const double ird = rsq_nr(r2);
      const double rd = r2 * ird;
      if (r2 < rc2) {
        const T r = T(rd), ir = T(ird);
        const T ux = T(dx) * ir, uy = T(dy) * ir, uz = T(dz) * ir;
        const T dxdr = two_rc;
        const T x = r * dxdr - T(1);
        T ps, dps;
        taper_t<T>((r - rc) * inv_h, ps, dps);
        dps *= inv_h;
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
        T S[LM], Sx[LM], Sy[LM], Sz[LM];
        solid_harmonics<T, LMAX, true>(ux, uy, uz, S, Sx, Sy, Sz);
        T radial = T(0), vx = T(0), vy = T(0), vz = T(0);
#pragma unroll
        for (int lm = 0; lm < LM; ++lm) {
          int l = 0;
          while ((l + 1) * (l + 1) <= lm) ++l;
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
          radial += (bv - av * T(l) * ir) * S[lm];
          const T ar = av * ir;
          vx = fma(ar, Sx[lm], vx);
          vy = fma(ar, Sy[lm], vy);
          vz = fma(ar, Sz[lm], vz);
        }
        gx = (double)(radial * ux + vx);
        gy = (double)(radial * uy + vy);
        gz = (double)(radial * uz + vz);
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
      if (gx != 0.0 || gy != 0.0 || gz != 0.0) {
        unsafeAtomicAdd(&f[j], -gx);
        unsafeAtomicAdd(&f[(size_t)n + j], -gy);
        unsafeAtomicAdd(&f[2 * (size_t)n + j], -gz);
      }
      fix += gx;
      fiy += gy;
      fiz += gz;
    }
  }
  fix = wave_sum(fix);
  fiy = wave_sum(fiy);
  fiz = wave_sum(fiz);
  if (lane == 0) {
    unsafeAtomicAdd(&f[i], fix);
    unsafeAtomicAdd(&f[(size_t)n + i], fiy);
    unsafeAtomicAdd(&f[2 * (size_t)n + i], fiz);
  }
  if (w2i != 0.0) {  // uniform across the wave
    f2x = wave_sum(f2x);
    f2y = wave_sum(f2y);
    f2z = wave_sum(f2z);
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
  APX_ALLOC(ctx, buf, (dc1 ? 2 : 1) * bytes_A + bytes_anch + bytes_slope + bytes_more);
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
  void* more = p;
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
  const T rc = (T)m->r_cut, inv_h = (T)(1.0 / m->h);
  const double rc2 = m->r_cut * m->r_cut;
  const size_t lds1 = BasisLds<T, LMAX>::bytes();
  {
  ProfScope ps(ctx, "ace.basis");
  k_ace_basis<T, LMAX><<<n_act, 64, lds1, ctx->stream>>>(atoms->pos, n, b, nl->count, nl->idx, nl->max_nb, active,
                                                         n_act, m->n_max, rc, inv_h, rc2, tb.Wp, an, sc);
  APX_LAUNCH_CHECK(ctx);
  }
  apx_status s = sym_products<T>(ctx, m, sc.A, B, slope, n_act, sc.e_anch, active, e_site, more);
  if (s == APX_OK && dc1) s = ace_grad<T>(ctx, m, sc.A, slope, w, active, n_act, dc1, dc2, more);
  if (s != APX_OK) return s;
  ProfScope ps(ctx, "ace.force");
  auto force = [&](auto nmax_c) {
    constexpr int NM = decltype(nmax_c)::value;
    const size_t lds3 = sizeof(T) * (size_t)ForceLds<T, NM>::KP * LM;
    k_ace_force<T, LMAX, NM><<<n_act, 64, lds3, ctx->stream>>>(atoms->pos, n, b, nl->count, nl->idx, nl->max_nb,
                                                               active, n_act, m->n_max, rc, inv_h, rc2, an, sc, w,
                                                               f, w2, f2);
  };
  if (m->n_max <= 8) force(std::integral_constant<int, 8>{});
  else if (m->n_max <= 10) force(std::integral_constant<int, 10>{});
  else force(std::integral_constant<int, 12>{});
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
    k_fill_zero<<<blocks_for(3LL * n, 256), 256, 0, ctx->stream>>>(f, 3LL * n);
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
