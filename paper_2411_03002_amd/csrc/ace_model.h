// ACE model: device copies of the radial mixing and the coupling tables.
#pragma once

#include "common.h"

namespace apx {

// Waves per block of the product-basis kernel: 16 for float32 (<= 128 VGPRs), 8 for
// float64 (<= 256 VGPRs).
constexpr int kAceWaves32 = 16;
constexpr int kAceWaves64 = 8;
// ints per pair record: [0] off1, [1] off2, [2] type = l1*(l_max+1)+l2, [3] n1,
// [4+L] first triple of degree L (L = 0..l_max+1, the last entry closes the list),
// [10+L] atomic-base offset of the first third block of degree L, [15] n2.
constexpr int kPairRec = 16;
template <class T>
struct alignas(2 * sizeof(T)) Coef2 {
  T c1, c2;
};

// Pointers into one precision's copy of the tables.
constexpr int kTcPad = 12;  // zero coefficient pairs around the triple table (>= the largest n_max)

template <class T>
struct AceTables {
  const T* Wp;        // [l_max+1][n_max][n_max], W[l][n][k] * N_l / s_a
  const int* pairs;   // [npairs][kPairRec], sorted by type
  const int* t_v;     // [ntrip] basis index
  const Coef2<T>* tc; // [ntrip] (c1, c2) per triple, kTcPad zero entries before and after
  const int* b1_off;  // [nb1]
  const int* b1_v;
  const T* b1_c1;
  const T* b1_c2;
  const int* b2_off;  // [nb2][3]: off1, off2, l
  const int* b2_v;
  const T* b2_c1;
  const T* b2_c2;
  int npairs;
};

// Tables of the symmetric product kernels (ace_sym.hip).  Types t = l2 (l2 + 1) / 2 + l1 are the
// degree pairs l1 <= l2; the label pairs of a type are (n1, n2) with n2 (of l2) outermost, n1 = 0
// .. n_max - 1, or n1 >= n2 where l1 = l2.
// off: [t * 5 + L] first coefficient of (t, L); [kSymB2 + L] of the second-order rows of degree L;
// [kSymPairs + t] first entry of the type's pairs; [kSymNg + t] its number of pair groups (one
// pair a group in float32, four in float64).
constexpr int kSymB2 = 75, kSymPairs = 80, kSymNg = 95, kSymOff = 110;

// Radial indices the product kernels are instantiated for.
__host__ __device__ constexpr int sym_nmax(int n_max) { return n_max <= 8 ? 8 : (n_max <= 10 ? 10 : 12); }

template <class T>
struct SymTables {
  const T* Wp;       // as AceTables
  const T* coef;     // rows of 2 sym_nmax values (c1 and c2 of n3 = 0, 1, ...), one group after the other
  const T* b1;       // [n_max][2]
  const int* pairs;  // atomic-base row of the l1 block | row of the l2 block << 16
  const int* off;
};

}  // namespace apx

struct apx_ace_model {
  int device = 0;
  int n_max = 0, l_max = 0, na = 0;
  long long n_basis = 0;
  int npairs = 0, ntrip = 0, nb1 = 0, nb2 = 0;
  long long coupling_terms = 0, triple_width = 0;  // per-atom work counts
  double r_cut = 5.0, h = 0.5, s_a = 1.0, eps = 0.1;
  int anchored = 0;
  apx_eam_params anchor{};
  apx::DevBuf ints;           // pairs, t_v, b1_off, b1_v, b2_off, b2_v
  apx::DevBuf reals64, reals32;
  apx::AceTables<double> t64{};
  apx::AceTables<float> t32{};
  std::vector<double> W;      // host copy [l][n][k]
  std::vector<int> t_v, b1_v, b2_v;  // basis index of every coefficient slot (host)
  // symmetric product kernels: per coefficient slot the basis index (-1: zero) and its factor
  std::vector<int> sym_v32, sym_v64;
  std::vector<double> sym_m32, sym_m64;
  apx::DevBuf sym_i32, sym_i64, sym_r32, sym_r64;
  apx::SymTables<double> s64{};
  apx::SymTables<float> s32{};
};

namespace apx {
template <class T>
const SymTables<T>& sym_tables(const apx_ace_model* m);
template <>
inline const SymTables<double>& sym_tables<double>(const apx_ace_model* m) { return m->s64; }
template <>
inline const SymTables<float>& sym_tables<float>(const apx_ace_model* m) { return m->s32; }
}  // namespace apx
