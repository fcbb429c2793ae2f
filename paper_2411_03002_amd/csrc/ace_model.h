// ACE model: device copies of the radial mixing and the coefficient tables.
#pragma once

#include "common.h"

namespace apx {

// Tables of the product kernels (ace_sym.hip).  Types t = l2 (l2 + 1) / 2 + l1 are the degree
// pairs l1 <= l2; the label pairs of a type are (n1, n2) with n2 (of l2) outermost, n1 = 0 ..
// n_max - 1, or n1 >= n2 where l1 = l2.
// off: [t * 5 + L] first coefficient of (t, L); [kSymB2 + L] of the second-order rows of degree L;
// [kSymPairs + t] first entry of the type's pairs; [kSymNg + t] its number of pair groups (one
// pair a group in float32, four in float64).
constexpr int kSymB2 = 75, kSymPairs = 80, kSymNg = 95, kSymOff = 110;

// Radial indices the product kernels are instantiated for.
__host__ __device__ constexpr int sym_nmax(int n_max) { return n_max <= 8 ? 8 : (n_max <= 10 ? 10 : 12); }

// Values of a row of SymTables::low.
__host__ __device__ constexpr int sym_low(int nmax) { return 2 * nmax + 4; }

template <class T>
struct SymTables {
  const T* Wp;       // [l_max+1][n_max][n_max], W[l][n][k] * N_l / s_a
  const T* coef;     // rows of 2 sym_nmax values (c1 and c2 of n3 = 0, 1, ...), one group after the other
  const T* b1;       // [n_max][2], behind coef
  // float32, behind coef: a row for every pair of one degree (l, then the pairs of type (l, l)):
  // second-order c1 and c2, then c1 and c2 of the third-order functions with n3 = 0, 1, ... of
  // degree 0 beside the pair (each function in one row)
  const T* low;
  const int* pairs;  // atomic-base row of the l1 block | row of the l2 block << 16
  const int* off;
  // per value of coef, low and b1: 2 * basis index + (0: c1, 1: c2), or -1 (zero), and its factor
  const int* slot;
  const double* factor;
  int n;
};

// Tables of the coefficient gradients (ace_grad.hip).
struct GradTables {
  const int* pairs;     // n1 | n2 << 16 by type, padded to sixteens
  const int* items;     // [n_items][3]: type (15 + L: second order), first pair, first slot
  const int* at;        // [slots] 2 * basis index + (0: c1, 1: c2), or -1
  const double* scale;  // [slots]
  int n_items, slots;
};

}  // namespace apx

struct apx_ace_model {
  int device = 0;
  int n_max = 0, l_max = 0, na = 0;
  long long n_basis = 0;
  int npairs = 0, ntrip = 0;
  long long coupling_terms = 0, triple_width = 0;  // of apx_ace_model_stats, as npairs and ntrip
  double r_cut = 5.0, h = 0.5, s_a = 1.0, eps = 0.1;
  int anchored = 0;
  apx_eam_params anchor{};
  apx::DevBuf ints, doubles;  // index tables; Wp, factors and scales
  apx::DevBuf wp32, c;        // float32 Wp; the coefficients [c1, c2][n_basis]
  apx::DevBuf coef64, coef32;
  apx::SymTables<double> s64{};
  apx::SymTables<float> s32{};
  apx::GradTables grad{};
};

namespace apx {
template <class T>
const SymTables<T>& sym_tables(const apx_ace_model* m);
template <>
inline const SymTables<double>& sym_tables<double>(const apx_ace_model* m) { return m->s64; }
template <>
inline const SymTables<float>& sym_tables<float>(const apx_ace_model* m) { return m->s32; }
}  // namespace apx
