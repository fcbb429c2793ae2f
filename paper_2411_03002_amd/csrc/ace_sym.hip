// Product basis of the atomic cluster expansion and its adjoint, without a backward pass.
//
// The energy is phi1 + F_eps(phi2) with phi_p = sum c_p B over the first-, second- and
// third-order functions (Sec. III A).  A third-order function is symmetric in its three
// blocks, so the derivative with respect to block r = (n3, L) is a sum over ALL unordered
// label pairs {q1, q2} that couple to L,
//     dphi_p/dA_rM = sum_{q1 <= q2} C_p[r; q1 q2] P_LM(q1, q2),
//     P_LM(q1, q2) = sum_{m1 m2} G(l1 l2 L; m1 m2 M) A_q1m1 A_q2m2,
// where C_p is the function's coefficient times the number of times r occurs in {r, q1, q2}.
// The coefficients are the same for every atom: with the pairs as the reduction index this is
// a matrix product of C (rows: n3 and p) with P (columns: atoms), and it runs on the matrix
// cores, one pair (float32) or four (float64) per instruction.  Second-order functions join as
// pairs whose P is the block itself.  No coupling is back-propagated: by Euler's rule for
// homogeneous functions phi_p = A . (D3 / 3 + D2 / 2 + D1) with D_k = the derivative of the
// k-th order part.
//
// In float32 the accumulators round at the size of their sums, most of which are functions with a
// block of degree 0 (an isotropic density): their terms are added last, and their energies, with the
// second order's, are formed apart in float64 sums (low_energy); Euler's rule is left the functions
// without such a block.  Rounding of the energy for 192 thermal environments (emulated, eV RMS), the
// rule for every function and one accumulator / here / compensated float32 sums over the pairs of
// triples: 1.8e-8 / 4.4e-9 / 8.0e-9 at (10, 4), 2.1e-8 / 4.1e-9 / 4.6e-9 at (12, 3), 3.0e-8 / 6.4e-9 /
// 7.3e-9 at (6, 4).
//
// Against an evaluation over a minimal set of triples with an explicit
// backward coupling (forward 30 k and backward 90 k multiply-adds per atom at n_max 10,
// l_max 4, and float atomics on the adjoint) the coupling is evaluated for 2,160 (pair, L)
// entries instead of 995, but forwards only (68 k vector instructions a tile), and the 235 k
// multiply-adds with the coefficients run as 11,760 pairs of one 16x16x1 and one 4x4x1
// instruction.  Measured, 821,266 atoms of the indentation block in float32: energy, five
// adjoint launches, their zero fill and the back-projection took 16.9 ms; this kernel alone,
// which does all of it, 5.5 ms (counters: 0.48 M matrix and 0.38 M vector cycles of a SIMD for a
// tile of 64, of 0.99 M).  In float64, 29,150 atoms: 2,850 us in the kernel that dealt
// pairs to waves and added adjoints in LDS, 477 us here (16x16x4 and 4x4x4 instructions).
//
// A block holds one tile of atoms in LDS; its eight waves each own a few components (L, M)
// of every third block, so that sums of products shared by the degrees L of one M are formed
// once and no two waves add to the same output.  Accumulators stay in registers through all
// label pairs.  The waves run different code between common barriers.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "ace_coupling_gen.h"
#include "ace_sym.h"
#include "device_util.h"

namespace apx {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kSymWaves = 8;
constexpr int kSymMaxSplit = 8;             // blocks that share a tile's pairs
constexpr int kSymBlocks = 512;             // blocks of a launch up to which tiles are shared

template <class T>
struct SymArgs {
  const T* A;      // [tile * TA + atom][stride] atomic base
  T* B;            // the same rows: projected adjoint (may be A: a tile is read before it is written)
  T* slope;        // [atom] F_eps'(phi2), or null
  const T* Wp;
  const T* coef;   // rows of C, see SymTables
  const T* b1;     // [n_max][2]
  const T* low;    // rows of the pairs of one degree (float32)
  const int* pairs;
  const int* off;  // see SymTables
  T* slab;         // [split][tile][lm][2 NMAX][TA]
  double* epart;   // [split][tile][2][TA]
  const double* e_anch;
  const int* active;
  double* e_site;
  double eps;
  int n_act, stride, n_max, nsplit;
};

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(std::forward<F>(f));
  }
}

// Uniform read of a table entry through the constant address space (a scalar load).
__device__ __forceinline__ int sld(const int* p) { return *(const __attribute__((address_space(4))) int*)p; }
__device__ __forceinline__ float sld(const float* p) { return *(const __attribute__((address_space(4))) float*)p; }

// One component's accumulators: rows o = 2 n3 + p of C (p = 0: c1, 1: c2), columns = atoms.
// Rows 0..15 by a 16-row instruction, further rows four at a time.
template <class T, int NMAX>
struct SymAcc;

// float32: one pair per step, lane = atom (P as the B operand of the four-block 16x16x1 and
// sixteen-block 4x4x1 forms); a coefficient row sits in lanes 0 .. 2 NMAX - 1 of one register
// and is broadcast to all blocks (cbsz, abid).  d[4 blk + r] holds row 4 (lane / 16) + r of
// atom 16 blk + lane % 16; e[k][r] holds row 16 + 4 k + r of atom `lane`.
template <int NMAX>
struct SymAcc<float, NMAX> {
  static constexpr int R = 2 * NMAX, NB = (R - 16) / 4, TA = 64, kPairs = 1;
  f32x16 d;
  f32x4 e[NB > 0 ? NB : 1];
  struct Coef {
    float c;
  };
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = 0.f;
#pragma unroll
    for (int k = 0; k < NB; ++k) e[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // byte offset of the lane's coefficient within a row, and row group g of the table `rows`
  // (wave-uniform: the load takes a scalar base and the lane's offset)
  static __device__ __forceinline__ unsigned lane_bytes(int lane) { return 4u * (unsigned)(lane < R ? lane : R - 1); }
  static __device__ __forceinline__ Coef load(const float* rows, int g, unsigned bytes) {
    return Coef{*reinterpret_cast<const float*>(reinterpret_cast<const char*>(rows + g * R) + bytes)};
  }
  __device__ __forceinline__ void step(const Coef& c, float P) {
    d = __builtin_amdgcn_mfma_f32_16x16x1f32(c.c, P, d, 2, 0, 0);
    if constexpr (NB > 0) e[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(c.c, P, e[0], 4, 4, 0);
    if constexpr (NB > 1) e[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(c.c, P, e[1], 4, 5, 0);
  }
  __device__ __forceinline__ void store(float* out, int lane) const {
    const int sub = lane >> 4, col = lane & 15;
#pragma unroll
    for (int k = 0; k < 16; ++k) out[(4 * sub + (k & 3)) * TA + 16 * (k >> 2) + col] = d[k];
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(16 + 4 * k + r) * TA + lane] = e[k][r];
  }
  // the slopes F'(phi2) of the atoms a lane's rows belong to
  static constexpr int kFp = 5;
  static __device__ __forceinline__ void slopes(const float* fp, int lane, float (&f)[kFp]) {
#pragma unroll
    for (int b = 0; b < 4; ++b) f[b] = fp[16 * b + (lane & 15)];
    f[4] = fp[lane];
  }
  // out[n3 * step] = D1_n3 + F'(phi2) D2_n3
  __device__ __forceinline__ void combine(float* out, int step, int n_max, const float (&fp)[kFp], int lane) const {
    const int sub = lane >> 4, col = lane & 15;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float f = fp[b];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int n3 = 2 * sub + h;
        if (n3 < n_max) out[n3 * step + 16 * b + col] = fmaf(f, d[4 * b + 2 * h + 1], d[4 * b + 2 * h]);
      }
    }
    const float f = fp[4];
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int n3 = 8 + 2 * k + h;
        if (n3 < n_max) out[n3 * step + lane] = fmaf(f, e[k][2 * h + 1], e[k][2 * h]);
      }
  }
  // s += sum_n3 A_n3 D[n3][p] of the component whose rows of A start at `a` (n3
  // steps by `step`), in float64: s4[p] for atom `lane`, s16[p][blk] partial over the lane's rows
  struct Dot {
    double s16[2][4], s4[2];
  };
  __device__ __forceinline__ void dot(Dot& s, const float* a, int step, int n_max, int lane) const {
    const int sub = lane >> 4, col = lane & 15;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int n3 = min(2 * sub + h, n_max - 1);  // rows of D beyond n_max are zero
        const double x = (double)a[n3 * step + 16 * b + col];
        float d0 = d[4 * b + 2 * h], d1 = d[4 * b + 2 * h + 1];
        // converted one pair at a time: the accumulators leave few registers
        asm volatile("" : "+v"(d0), "+v"(d1)::"memory");
        s.s16[0][b] = fma(x, (double)d0, s.s16[0][b]);
        s.s16[1][b] = fma(x, (double)d1, s.s16[1][b]);
      }
      asm volatile("" : "+v"(s.s16[0][b]), "+v"(s.s16[1][b])::"memory");
    }
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int n3 = min(8 + 2 * k + h, n_max - 1);
        const double x = (double)a[n3 * step + lane];
        float d0 = e[k][2 * h], d1 = e[k][2 * h + 1];
        asm volatile("" : "+v"(d0), "+v"(d1)::"memory");
        s.s4[0] = fma(x, (double)d0, s.s4[0]);
        s.s4[1] = fma(x, (double)d1, s.s4[1]);
      }
    asm volatile("" : "+v"(s.s4[0]), "+v"(s.s4[1])::"memory");
  }
  // a wave's share of the sums: p = 0, 1 of atom `lane`
  struct Part {
    double e[2];
  };
  static __device__ __forceinline__ Part part(const Dot& s, int lane, double scale) {
    const int sub = lane >> 4;
    Part r;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      double v = 0.0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        double x = s.s16[p][b];
        x += __shfl_xor(x, 16, kWave);
        x += __shfl_xor(x, 32, kWave);
        v = b == sub ? x : v;
      }
      r.e[p] = scale * (v + s.s4[p]);
    }
    return r;
  }
  static __device__ __forceinline__ void put(const Part& s, int lane, double* red) {
#pragma unroll
    for (int p = 0; p < 2; ++p) red[p * TA + lane] = s.e[p];
  }
};

// float64: four pairs per step, lane = (pair lane / 16, atom lane % 16) (P as the B operand of
// the 16x16x4 and of the four-block 4x4x4 form, which covers the same atoms four columns a
// block).  d[r] holds row 4 r + lane / 16 of atom lane % 16, e[k] row 16 + 4 k + lane / 16.  A
// lane's rows thus belong to one sum, p = (lane / 16) % 2.
template <int NMAX>
struct SymAcc<double, NMAX> {
  static constexpr int R = 2 * NMAX, NB = (R - 16) / 4, TA = 16, kPairs = 4;
  f64x4 d;
  double e[NB > 0 ? NB : 1];
  struct Coef {
    double c, c4[NB > 0 ? NB : 1];
  };
  __device__ __forceinline__ void zero() {
    d = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NB; ++k) e[k] = 0.0;
  }
  static __device__ __forceinline__ unsigned lane_bytes(int lane) { return (unsigned)lane; }
  static __device__ __forceinline__ Coef load(const double* rows, int g, unsigned lane) {
    const double* r = rows + g * 4 * R;
    Coef c;
    c.c = r[lane];
#pragma unroll
    for (int k = 0; k < NB; ++k) c.c4[k] = (r + 64 + 16 * k)[(lane >> 4) * 4 + (lane & 3)];
    return c;
  }
  __device__ __forceinline__ void step(const Coef& c, double P) {
    d = __builtin_amdgcn_mfma_f64_16x16x4f64(c.c, P, d, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < NB; ++k) e[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(c.c4[k], P, e[k], 0, 0, 0);
  }
  __device__ __forceinline__ void store(double* out, int lane) const {
    const int sub = lane >> 4, col = lane & 15;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(4 * r + sub) * TA + col] = d[r];
#pragma unroll
    for (int k = 0; k < NB; ++k) out[(16 + 4 * k + sub) * TA + col] = e[k];
  }
  static constexpr int kFp = 1;
  static __device__ __forceinline__ void slopes(const double* fp, int lane, double (&f)[kFp]) { f[0] = fp[lane & 15]; }
  __device__ __forceinline__ void combine(double* out, int step, int n_max, const double (&fp)[kFp], int lane) const {
    const int sub = lane >> 4, col = lane & 15;
    auto put = [&](int n3, double v) {
      v = sub & 1 ? fp[0] * v : v;
      v += __shfl_xor(v, 16, kWave);
      if (!(sub & 1) && n3 < n_max) out[n3 * step + col] = v;
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) put(2 * r + (sub >> 1), d[r]);
#pragma unroll
    for (int k = 0; k < NB; ++k) put(8 + 2 * k + (sub >> 1), e[k]);
  }
  struct Dot {
    double s;
  };
  using Part = Dot;
  __device__ __forceinline__ void dot(Dot& s, const double* a, int step, int n_max, int lane) const {
    const int sub = lane >> 4, col = lane & 15;
#pragma unroll
    for (int r = 0; r < 4; ++r) s.s = fma(a[min(2 * r + (sub >> 1), n_max - 1) * step + col], d[r], s.s);
#pragma unroll
    for (int k = 0; k < NB; ++k) s.s = fma(a[min(8 + 2 * k + (sub >> 1), n_max - 1) * step + col], e[k], s.s);
  }
  static __device__ __forceinline__ void put(const Part& s, int lane, double* red) {
    const double v = s.s + __shfl_xor(s.s, 32, kWave);
    if (lane < 32) red[lane] = v;  // [p][TA]
  }
};

// The components of one wave: codes C = 2 M + (parity of L), each standing for every degree L of
// that parity with |M| <= L <= LMAX.
template <class T, int LMAX, int NMAX, int... CS>
struct SymProg {
  using Acc = SymAcc<T, NMAX>;
  static constexpr int TA = Acc::TA, LM = (LMAX + 1) * (LMAX + 1), NC = sizeof...(CS);
  static constexpr int kC[NC] = {CS...};
  static constexpr int par(int i) { return kC[i] & 1; }
  static constexpr int comp(int i) { return (kC[i] - par(i)) / 2; }
  static constexpr int iabs(int m) { return m < 0 ? -m : m; }
  static constexpr int lmin(int i) { return iabs(comp(i)) + ((iabs(comp(i)) + par(i)) & 1); }
  static constexpr int nl(int i) { return lmin(i) > LMAX ? 0 : (LMAX - lmin(i)) / 2 + 1; }
  static constexpr int base(int i) {
    int b = 0;
    for (int k = 0; k < i; ++k) b += nl(k);
    return b;
  }
  static constexpr int NA = base(NC);
  static constexpr bool holds(int i, int L) { return L % 2 == par(i) && L >= iabs(comp(i)) && L <= LMAX; }
  static constexpr int slot(int i, int L) { return base(i) + (L - lmin(i)) / 2; }
  // whether some component of the wave has degree L
  static constexpr bool has(int L) {
    for (int i = 0; i < NC; ++i)
      if (holds(i, L)) return true;
    return false;
  }
  static constexpr bool couples(int l1, int l2, int L) {
    return L >= l2 - l1 && L <= l1 + l2 && L <= LMAX && (l1 + l2 + L) % 2 == 0;
  }
  static constexpr bool uses(int l1, int l2) {
    for (int L = 0; L <= LMAX; ++L)
      if (couples(l1, l2, L) && has(L)) return true;
    return false;
  }
  static constexpr bool uses_comp(int l1, int l2, int i) {
    for (int L = 0; L <= LMAX; ++L)
      if (couples(l1, l2, L) && holds(i, L)) return true;
    return false;
  }

  Acc acc[NA];

  // All pairs of one type (this split's share of them).
  template <int L1, int L2>
  __device__ __forceinline__ void type(const SymArgs<T>& g, const T* As, int lane, int split) {
    constexpr int t = L2 * (L2 + 1) / 2 + L1;
    constexpr int N1 = 2 * L1 + 1, N2 = 2 * L2 + 1;
    const int ng = sld(g.off + kSymNg + t);
    const int lo = ng * split / g.nsplit, hi = ng * (split + 1) / g.nsplit;
    if (lo >= hi) return;
    const int* pt = g.pairs + sld(g.off + kSymPairs + t);
    const T* rows[LMAX + 1];
    typename Acc::Coef c[LMAX + 1];
    unsigned lb = Acc::lane_bytes(lane);
    static_for<0, LMAX + 1>([&](auto L) {
      if constexpr (couples(L1, L2, L) && has(L)) {
        rows[L] = g.coef + sld(g.off + t * 5 + L);
        c[L] = Acc::load(rows[L], lo, lb);
      }
    });
    T a[N1], b[N2], P[NC][5];
    auto products = [&]() {
      static_for<0, NC>([&](auto i) {
        if constexpr (uses_comp(L1, L2, i)) SymP<L1, L2, comp(i)>::template p<LMAX, T>(a, b, P[i]);
      });
    };
    auto steps = [&](const typename Acc::Coef(&cc)[LMAX + 1]) {
      static_for<0, NC>([&](auto i) {
        static_for<0, LMAX + 1>([&](auto L) {
          if constexpr (couples(L1, L2, L) && holds(i, L)) acc[slot(i, L)].step(cc[L], P[i][L]);
        });
      });
    };
    if constexpr (Acc::kPairs == 1) {
      // one pair per step, wave-uniform: the outer (larger-degree) label's block stays in
      // registers while the inner one runs.  The next pair's inner block is read while the
      // matrix instructions run, coefficients and indices two pairs ahead into two sets of
      // registers (the tables are padded).
      int pk = sld(pt + lo), nx = sld(pt + lo + 1);
      const T* al = As + lane;
#pragma unroll
      for (int m = 0; m < N2; ++m) b[m] = al[((pk >> 16) + m) * TA];
#pragma unroll
      for (int m = 0; m < N1; ++m) a[m] = al[((pk & 0xffff) + m) * TA];
      typename Acc::Coef d[LMAX + 1];
      static_for<0, LMAX + 1>([&](auto L) {
        if constexpr (couples(L1, L2, L) && has(L)) d[L] = Acc::load(rows[L], lo + 1, lb);
      });
      auto pair = [&](int p, typename Acc::Coef(&cc)[LMAX + 1]) {
        const int nn = sld(pt + p + 2);
        // opaque, so that the loads keep the scalar base (a vector pointer per table would be
        // advanced by vector instructions)
        asm volatile("" : "+v"(lb));
        products();
#pragma unroll
        for (int m = 0; m < N1; ++m) a[m] = al[((nx & 0xffff) + m) * TA];
        steps(cc);
        static_for<0, LMAX + 1>([&](auto L) {
          if constexpr (couples(L1, L2, L) && has(L)) cc[L] = Acc::load(rows[L], p + 2, lb);
        });
        if ((nx >> 16) != (pk >> 16)) {
#pragma unroll
          for (int m = 0; m < N2; ++m) b[m] = al[((nx >> 16) + m) * TA];
        }
        pk = nx;
        nx = nn;
      };
      int p = lo;
      for (; p + 1 < hi; p += 2) {
        pair(p, c);
        pair(p + 1, d);
      }
      if (p < hi) pair(p, c);
    } else {
      // four pairs side by side: lane = (pair of the group, atom)
      const T* al = As + (lane & (TA - 1));
      const int sub = lane / TA;
      int pk = pt[4 * lo + sub];
      auto blocks = [&](int w) {
#pragma unroll
        for (int m = 0; m < N1; ++m) a[m] = al[((w & 0xffff) + m) * TA];
#pragma unroll
        for (int m = 0; m < N2; ++m) b[m] = al[((w >> 16) + m) * TA];
      };
      blocks(pk);
      pk = pt[4 * (lo + 1) + sub];
      for (int p = lo; p < hi; ++p) {
        const int nx = pt[4 * (p + 2) + sub];
        products();
        blocks(pk);  // the next group's, read while the matrix instructions run
        steps(c);
        static_for<0, LMAX + 1>([&](auto L) {
          if constexpr (couples(L1, L2, L) && has(L)) c[L] = Acc::load(rows[L], p + 1, lb);
        });
        pk = nx;
      }
    }
  }

  // s += the components of degree L >= FROM times A
  template <int FROM>
  __device__ __forceinline__ void dots(const SymArgs<T>& g, const T* As, int lane, typename Acc::Dot& s) const {
    static_for<0, NC>([&](auto i) {
      static_for<FROM, LMAX + 1>([&](auto L) {
        if constexpr (holds(i, L))
          acc[slot(i, L)].dot(s, As + (L * L + L + comp(i)) * TA, LM * TA, g.n_max, lane);
      });
    });
  }

  // Second order: the pairs are single blocks (n', L).
  __device__ __forceinline__ void second_order(const SymArgs<T>& g, const T* As, int lane) {
    static_for<0, LMAX + 1>([&](auto L) {
      if constexpr (has(L)) {
        const T* rows = g.coef + sld(g.off + kSymB2 + L);
        const T* al = As + (lane & (TA - 1)) + (L * L + L) * TA;
        const int sub = lane / TA;
#pragma unroll 4
        for (int p = 0; p < (g.n_max + Acc::kPairs - 1) / Acc::kPairs; ++p) {
          const int n = p * Acc::kPairs + sub;
          const T* an = al + (n < g.n_max ? n : 0) * LM * TA;
          const typename Acc::Coef c = Acc::load(rows, p, Acc::lane_bytes(lane));
          static_for<0, NC>([&](auto i) {
            if constexpr (holds(i, L)) acc[slot(i, L)].step(c, an[comp(i) * TA]);
          });
        }
      }
    });
  }

  // The energies of the second order and of the third-order functions with a block of degree 0,
  // float32: per label pair of one degree, sum_M A_n1 A_n2 times (the pair's second-order
  // coefficient plus sum_n3 c A_n3,00), added in float64 two pairs at a time.  The pairs are shared
  // among the waves and done first, while registers are free.  Bound by vector instruction issue (30 a
  // pair): 0.2 of 5.4 ms for 821,266 atoms at (10, 4), 10 of 230 us for 29,150; 0.1 ms more with the
  // pairs dealt round-robin, behind two more table reads, at the end.
  static __device__ __forceinline__ void low_energy(const SymArgs<T>& g, const T* As, int lane, int share, int shares,
                                                    double (&e)[2]) {
    // (entries of a last group beyond hi are read, the tables are padded, and not added)
    constexpr int W = sym_low(NMAX), G = 2;
    const T* al = As + lane;
    const int K = g.n_max, np = K * (K + 1) / 2;  // pairs of a degree
    const int lo = np * share / shares, hi = np * (share + 1) / shares;
    // (before the pairs of (l, l) lie l (l + 1) / 2 types of two degrees and l of one)
    auto pairs_of = [&](int l) { return g.pairs + l * (l + 1) / 2 * K * K + l * np; };
    int pk[LMAX + 1][G];
    static_for<0, LMAX + 1>([&](auto l) {
#pragma unroll
      for (int k = 0; k < G; ++k) pk[l][k] = sld(pairs_of(l) + lo + k);
    });
    T A0[NMAX];
#pragma unroll
    for (int n = 0; n < NMAX; ++n) A0[n] = al[(n < K ? n : 0) * LM * TA];
    static_for<0, LMAX + 1>([&](auto l) {
      for (int p = lo; p < hi; p += G) {
        T I[G], q[G][2];
        const T* row = g.low + (l * np + p) * W;
#pragma unroll
        for (int k = 0; k < G; ++k) {
          const T *a = al + (pk[l][k] & 0xffff) * TA, *b = al + (pk[l][k] >> 16) * TA;
          I[k] = a[0] * b[0];
#pragma unroll
          for (int m = 1; m < 2 * l + 1; ++m) I[k] = fma(a[m * TA], b[m * TA], I[k]);
          I[k] = p + k < hi ? I[k] : T(0);
          q[k][0] = sld(row + k * W);
          q[k][1] = sld(row + k * W + 1);
        }
#pragma unroll
        for (int k = 0; k < G; ++k) pk[l][k] = sld(pairs_of(l) + p + G + k);
#pragma unroll
        for (int n = 0; n < NMAX; ++n) {
#pragma unroll
          for (int k = 0; k < G; ++k) {  // (coefficients beyond n_max are zero)
            q[k][0] = fma(sld(row + k * W + 2 + 2 * n), A0[n], q[k][0]);
            q[k][1] = fma(sld(row + k * W + 3 + 2 * n), A0[n], q[k][1]);
          }
        }
        T v0 = q[0][0] * I[0], v1 = q[0][1] * I[0];
#pragma unroll
        for (int k = 1; k < G; ++k) {
          v0 = fma(q[k][0], I[k], v0);
          v1 = fma(q[k][1], I[k], v1);
        }
        e[0] += (double)v0;
        e[1] += (double)v1;
      }
    });
  }

  // The derivatives of the second- and third-order sums into acc; returns the wave's share of the
  // sums themselves.
  __device__ __forceinline__ typename Acc::Part sums(const SymArgs<T>& g, const T* As, int lane, int wv, int split) {
    typename Acc::Dot s{};
    if constexpr (sizeof(T) == 4) {
      double low[2] = {0.0, 0.0};
      low_energy(g, As, lane, split * kSymWaves + wv, g.nsplit * kSymWaves, low);
#pragma unroll
      for (int k = 0; k < NA; ++k) acc[k].zero();
      // without blocks of degree 0: a third of A . D; the large terms, those with one, come last
      static_for<1, LMAX + 1>([&](auto l2) {
        static_for<1, l2 + 1>([&](auto l1) {
          if constexpr (uses(l1, l2)) type<l1, l2>(g, As, lane, split);
        });
      });
      dots<1>(g, As, lane, s);
      typename Acc::Part e = Acc::part(s, lane, 1.0 / 3.0);
      e.e[0] += low[0];
      e.e[1] += low[1];
      static_for<0, LMAX + 1>([&](auto l2) {
        if constexpr (uses(0, l2)) type<0, l2>(g, As, lane, split);
      });
      if (split == 0) second_order(g, As, lane);
      return e;
    } else {
#pragma unroll
      for (int k = 0; k < NA; ++k) acc[k].zero();
      static_for<0, LMAX + 1>([&](auto l2) {
        static_for<0, l2 + 1>([&](auto l1) {
          if constexpr (uses(l1, l2)) type<l1, l2>(g, As, lane, split);
        });
      });
      // third order / 3 + second order / 2 = (both - third order / 3) / 2
      dots<0>(g, As, lane, s);
      s.s *= -1.0 / 3.0;
      if (split == 0) second_order(g, As, lane);
      dots<0>(g, As, lane, s);
      s.s *= 0.5;
      return s;
    }
  }

  // The wave's part of a block: FUSED (one split): the combined derivative into the tile;
  // otherwise both derivatives to the slab and the sums to epart.
  template <bool FUSED>
  static __device__ __forceinline__ void run(const SymArgs<T>& g, T* As, double* red, int wv, int lane, int split,
                                             int slab_tile) {
    SymProg w;
    const typename Acc::Part s = w.sums(g, As, lane, wv, split);
    if constexpr (!FUSED) {
      T* out = g.slab + ((size_t)slab_tile * LM) * (Acc::R * TA);
      static_for<0, NC>([&](auto i) {
        static_for<0, LMAX + 1>([&](auto L) {
          if constexpr (holds(i, L)) w.acc[slot(i, L)].store(out + (size_t)(L * L + L + comp(i)) * (Acc::R * TA), lane);
        });
      });
    }
    // the first-order part joins once per tile (its derivative is added with the projection)
    double e1[2] = {0.0, 0.0};
    if (wv == 0 && lane < TA && split == 0) {
      for (int n = 0; n < g.n_max; ++n) {
        const double x = (double)As[n * LM * TA + lane];
        e1[0] = fma((double)g.b1[2 * n], x, e1[0]);
        e1[1] = fma((double)g.b1[2 * n + 1], x, e1[1]);
      }
    }
    __syncthreads();  // every wave is done with the tile: red lies over it
    Acc::put(s, lane, red + wv * 2 * TA);
    __syncthreads();
    T* fps = reinterpret_cast<T*>(red + kSymWaves * 2 * TA);
    if (wv == 0 && lane < TA) {
#pragma unroll
      for (int p = 0; p < 2; ++p)
        for (int k = 0; k < kSymWaves; ++k) e1[p] += red[(k * 2 + p) * TA + lane];
      if constexpr (FUSED) {
        const int q = slab_tile * TA + lane;  // slab_tile: the tile itself
        const double root = sqrt(fabs(e1[1]) + g.eps * g.eps), f2 = root - g.eps;
        fps[lane] = T(0.5 / root);
        if (g.slope && q < g.n_act) g.slope[q] = T(0.5 / root);
        if (q < g.n_act) g.e_site[g.active[q]] = e1[0] + (e1[1] < 0.0 ? -f2 : f2) + g.e_anch[q];
      } else {
#pragma unroll
        for (int p = 0; p < 2; ++p) g.epart[((size_t)slab_tile * 2 + p) * TA + lane] = e1[p];
      }
    }
    if constexpr (FUSED) {
      __syncthreads();
      T fp[Acc::kFp];
      Acc::slopes(fps, lane, fp);
      const T f = wv == 0 && lane < TA ? fps[lane] : T(0);
      __syncthreads();  // red and fps are read: the tile takes the combined derivative
      if (wv == 0 && lane < TA) As[g.n_max * LM * TA + lane] = f;  // behind the tile
      static_for<0, NC>([&](auto i) {
        static_for<0, LMAX + 1>([&](auto L) {
          if constexpr (holds(i, L))
            w.acc[slot(i, L)].combine(As + (L * L + L + comp(i)) * TA, LM * TA, g.n_max, fp, lane);
        });
      });
    }
  }
};

// The waves' components.  A wave's share of the matrix instructions (the number of pairs over
// its components) is within 20% of the others', and waves w and w + 4, which share a SIMD,
// together within 8%.
template <class T, int LMAX, int NMAX, bool FUSED>
__device__ __forceinline__ void sym_waves(const SymArgs<T>& g, T* As, double* red, int wv, int lane, int split,
                                          int slab_tile) {
#define APX_SYM(...) SymProg<T, LMAX, NMAX, __VA_ARGS__>::template run<FUSED>(g, As, red, wv, lane, split, slab_tile)
  constexpr auto even = [](int m) { return 2 * m; };
  constexpr auto odd = [](int m) { return 2 * m + 1; };
  if constexpr (LMAX == 4) {
    switch (wv) {
      case 0: APX_SYM(even(0), odd(-3)); break;
      case 1: APX_SYM(even(1), even(3)); break;
      case 2: APX_SYM(even(-1), even(-3)); break;
      case 3: APX_SYM(even(2), even(4)); break;
      case 4: APX_SYM(odd(0), odd(2)); break;
      case 5: APX_SYM(odd(1), odd(-2)); break;
      case 6: APX_SYM(odd(-1), odd(3)); break;
      default: APX_SYM(even(-2), even(-4)); break;
    }
  } else {
    switch (wv) {
      case 0: APX_SYM(even(0)); break;
      case 1: APX_SYM(even(1), even(-1)); break;
      case 2: APX_SYM(even(2), even(-2)); break;
      case 3: APX_SYM(odd(0)); break;
      case 4: APX_SYM(odd(1)); break;
      case 5: APX_SYM(odd(-1)); break;
      case 6: APX_SYM(odd(2), odd(-2)); break;
      default: APX_SYM(odd(3), odd(-3)); break;
    }
  }
#undef APX_SYM
}

// The radial mixing Wp[l][n][k] in LDS as [l][k][n], rows of NMAX, zero beyond n_max.
template <class T, int LMAX, int NMAX>
__device__ __forceinline__ void stage_mixing(const T* Wp, int K, T* ws) {
  for (int e = threadIdx.x; e < (LMAX + 1) * NMAX * NMAX; e += blockDim.x) {
    const int l = e / (NMAX * NMAX), r = e - l * NMAX * NMAX, kk = r / NMAX, nn = r - kk * NMAX;
    ws[e] = nn < K && kk < K ? Wp[((size_t)l * K + nn) * K + kk] : T(0);
  }
}

__device__ __forceinline__ int degree_of(int lm) {
  int l = 0;
  while ((l + 1) * (l + 1) <= lm) ++l;
  return l;
}

// sum_n Wp[l][n][k] d[n], the row w of (l, k)
template <class T, int NMAX>
__device__ __forceinline__ T project(const T* w, const T (&d)[NMAX]) {
  T v = T(0);
#pragma unroll
  for (int n = 0; n < NMAX; ++n) v = fma(w[n], d[n], v);
  return v;
}

// One tile of atoms and one of nsplit shares of its label pairs per block.  Bound by vector
// and matrix instruction issue (float32 matrix instructions share the vector unit's
// multipliers on gfx950: interleaved independent instructions of the two kinds take the sum of
// their times).  With one share (FUSED) the block finishes its tile: embedding, the two
// derivatives combined in registers, the projection in LDS.
template <class T, int LMAX, int NMAX, bool FUSED>
__global__ void __launch_bounds__(kSymWaves * 64, 4) k_ace_sym(SymArgs<T> g) {
  using Acc = SymAcc<T, NMAX>;
  constexpr int TA = Acc::TA, LM = (LMAX + 1) * (LMAX + 1);
  constexpr int V = 16 / (int)sizeof(T), CH = kSymWaves * 64 / TA;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  extern __shared__ double smem_raw[];
  __shared__ T ws[FUSED ? (LMAX + 1) * NMAX * NMAX : 1];
  T* As = reinterpret_cast<T*>(smem_raw);  // [a][TA]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int split = blockIdx.y, K = g.n_max, na = K * LM;
  const int tile = blockIdx.x;
  const int t = tid & (TA - 1), ch = tid / TA;
  const int q = tile * TA + t;
  const T* row = g.A + (size_t)q * g.stride;
  if constexpr (FUSED) stage_mixing<T, LMAX, NMAX>(g.Wp, K, ws);
  // 16 bytes of one atom's row per lane, lanes over atoms: the LDS stores are conflict-free,
  // and a row's cache lines are used up by the next loads
  for (int a0 = ch * V; a0 < na; a0 += CH * V) {
    vec v;
#pragma unroll
    for (int k = 0; k < V; ++k) v[k] = T(0);
    if (q < g.n_act) v = *reinterpret_cast<const vec*>(row + a0);
#pragma unroll
    for (int k = 0; k < V; ++k)
      if (a0 + k < na) As[(a0 + k) * TA + t] = v[k];
  }
  __syncthreads();
  sym_waves<T, LMAX, NMAX, FUSED>(g, As, smem_raw, wv, lane, split,
                                  FUSED ? tile : split * (int)gridDim.x + (int)blockIdx.x);
  if constexpr (FUSED) {
    __syncthreads();
    // projection in place: column lm's n_max rows give way to its n_max projections
    for (int lm = ch; lm < LM; lm += CH) {
      T d[NMAX];
#pragma unroll
      for (int n = 0; n < NMAX; ++n) d[n] = n < K ? As[(n * LM + lm) * TA + t] : T(0);
      if (lm == 0) {
        const T f = As[na * TA + t];
#pragma unroll
        for (int n = 0; n < NMAX; ++n)
          if (n < K) d[n] += fma(f, g.b1[2 * n + 1], g.b1[2 * n]);
      }
      const T* wl = ws + degree_of(lm) * NMAX * NMAX;
      for (int kk = 0; kk < K; ++kk) As[(kk * LM + lm) * TA + t] = project<T, NMAX>(wl + kk * NMAX, d);
    }
    __syncthreads();
    for (int o = ch * V; o < na; o += CH * V) {
      vec v;
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const int lm = (o + k) / K, kk = o + k - lm * K;
        v[k] = o + k < na ? As[(kk * LM + lm) * TA + t] : T(0);
      }
      if (q < g.n_act) *reinterpret_cast<vec*>(g.B + (size_t)q * g.stride + o) = v;
    }
  }
}

// The end of a tile whose pairs were shared by several blocks, sixteen atoms per block (one
// column lm per sixteen threads): per atom the two sums and, for each column, both derivatives
// summed over the shares, then as above; the rows are gathered in LDS and written out whole.
constexpr int kFinThreads = 512;
template <class T, int LMAX, int NMAX>
__global__ void __launch_bounds__(kFinThreads) k_ace_sym_finish(SymArgs<T> g) {
  using Acc = SymAcc<T, NMAX>;
  constexpr int TA = Acc::TA, LM = (LMAX + 1) * (LMAX + 1), R = Acc::R, NA = 16;
  static_assert(kFinThreads / NA >= LM, "a column per group of threads");
  __shared__ T ws[(LMAX + 1) * NMAX * NMAX];
  __shared__ alignas(16) T rows[NA * ((NMAX * LM + 3) / 4 * 4)];
  const int K = g.n_max;
  stage_mixing<T, LMAX, NMAX>(g.Wp, K, ws);
  const int r = threadIdx.x & (NA - 1), lm = threadIdx.x / NA;
  const int ntile = gridDim.x, t = NA * blockIdx.y + r;
  const int q0 = (int)blockIdx.x * TA + NA * (int)blockIdx.y, q = q0 + r;
  double phi[2] = {0.0, 0.0};
  for (int s = 0; s < g.nsplit; ++s)
#pragma unroll
    for (int p = 0; p < 2; ++p) phi[p] += g.epart[(((size_t)s * ntile + blockIdx.x) * 2 + p) * TA + t];
  T D1[NMAX], D2[NMAX];
#pragma unroll
  for (int n = 0; n < NMAX; ++n) D1[n] = D2[n] = T(0);
  if (lm < LM) {
#pragma unroll 2
    for (int s = 0; s < g.nsplit; ++s) {
      const T* in = g.slab + (((size_t)s * ntile + blockIdx.x) * LM + lm) * (R * TA) + t;
#pragma unroll
      for (int n = 0; n < NMAX; ++n) {
        D1[n] += in[(2 * n) * TA];
        D2[n] += in[(2 * n + 1) * TA];
      }
    }
  }
  const double root = sqrt(fabs(phi[1]) + g.eps * g.eps), f2 = root - g.eps;
  const T fp = T(0.5 / root);
  if (lm == 0 && g.slope && q < g.n_act) g.slope[q] = fp;
  if (lm == 0 && q < g.n_act) g.e_site[g.active[q]] = phi[0] + (phi[1] < 0.0 ? -f2 : f2) + g.e_anch[q];
  __syncthreads();
  if (lm < LM) {
#pragma unroll
    for (int n = 0; n < NMAX; ++n) {
      D1[n] = fma(fp, D2[n], D1[n]);
      if (lm == 0 && n < K) D1[n] += fma(fp, g.b1[2 * n + 1], g.b1[2 * n]);
    }
    const T* wl = ws + degree_of(lm) * NMAX * NMAX;
    for (int kk = 0; kk < K; ++kk) rows[r * g.stride + lm * K + kk] = project<T, NMAX>(wl + kk * NMAX, D1);
  }
  __syncthreads();
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int V = 16 / (int)sizeof(T);
  const int left = g.n_act - q0;
  const int total = (left < NA ? left : NA) * g.stride;
  vec* out = reinterpret_cast<vec*>(g.B + (size_t)q0 * g.stride);
  for (int o = threadIdx.x; o * V < total; o += kFinThreads) out[o] = reinterpret_cast<const vec*>(rows)[o];
}

namespace {

template <class T>
struct SymPlan {
  int tiles, split;    // tiles of the call, shares of a tile's pairs
  size_t slab, epart;  // bytes (one share needs neither)
};

// Bytes of one share's derivatives.
template <class T>
size_t share_slab(const apx_ace_model* m) {
  return sizeof(T) * (m->l_max + 1) * (m->l_max + 1) * 2 * sym_nmax(m->n_max) * sym_tile<T>();
}

// Shares of a tile's pairs: enough blocks for two per compute unit.  A share costs the block's
// staging and the sum over shares at the end; it pays while compute units idle.  Measured in
// float32 at (10, 4), products + end in us by shares 1/2/4/8: 8 tiles 164/94/60/44, 63 tiles
// 165/106/75/75, 125 tiles 166/113/99/129, 255 tiles 177/156/185/271, 375 tiles 235/239/260/403,
// 938 tiles 503/548/651/958; sixteen shares were no better than eight at 1 tile and worse beyond.
// In float64: 32 tiles 84/54/40/38, 125 tiles 87/64/57/73, 250 tiles 88/82/96/118, 500 tiles
// 131/148/165/217.
template <class T>
SymPlan<T> sym_plan(const apx_ace_model* m, int n_act) {
  constexpr int TA = sym_tile<T>();
  SymPlan<T> p;
  p.tiles = (n_act + TA - 1) / TA;
  p.split = std::max(1, std::min(kSymMaxSplit, kSymBlocks / std::max(1, p.tiles)));
  const size_t shares = p.split > 1 ? (size_t)p.split * p.tiles : 0;
  p.slab = shares * share_slab<T>(m);
  p.epart = shares * sizeof(double) * 2 * TA;
  return p;
}

template <class T, int LMAX, int NMAX>
apx_status sym_launch(apx_ctx* ctx, const apx_ace_model* m, const T* A, T* B, T* slope, int n_act,
                      const double* e_anch, const int* active, double* e_site, void* scratch) {
  using Acc = SymAcc<T, NMAX>;
  constexpr int TA = Acc::TA;
  const SymTables<T>& tb = sym_tables<T>(m);
  const SymPlan<T> pl = sym_plan<T>(m, n_act);
  SymArgs<T> g;
  g.A = A;
  g.B = B;
  g.slope = slope;
  g.coef = tb.coef;
  g.b1 = tb.b1;
  g.low = tb.low;
  g.pairs = tb.pairs;
  g.off = tb.off;
  g.slab = static_cast<T*>(scratch);
  g.epart = reinterpret_cast<double*>(static_cast<char*>(scratch) + pl.slab);
  g.n_act = n_act;
  g.stride = sym_stride(m->na);
  g.n_max = m->n_max;
  g.nsplit = pl.split;
  g.Wp = tb.Wp;
  g.e_anch = e_anch;
  g.active = active;
  g.e_site = e_site;
  g.eps = m->eps;
  // the tile and the slopes behind it; the sums' reduction and the slopes lie over the tile
  auto lds_for = [](int na) {
    return std::max(sizeof(T) * ((size_t)na + 1) * TA, sizeof(double) * kSymWaves * 2 * TA + sizeof(T) * TA);
  };
  const size_t lds = lds_for(m->na), most = lds_for(NMAX * (LMAX + 1) * (LMAX + 1));
  auto launch = [&](auto kern, int nt, int split) -> apx_status {
    // (the most of the instantiation: the attribute is the process's, and another thread's model may be smaller)
    APX_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most));
    ProfScope ps(ctx, "ace.products");
    kern<<<dim3(nt, split), kSymWaves * 64, lds, ctx->stream>>>(g);
    APX_LAUNCH_CHECK(ctx);
    return APX_OK;
  };
  if (pl.split == 1) return launch(k_ace_sym<T, LMAX, NMAX, true>, pl.tiles, 1);
  const apx_status s = launch(k_ace_sym<T, LMAX, NMAX, false>, pl.tiles, pl.split);
  if (s != APX_OK) return s;
  ProfScope ps(ctx, "ace.project");
  k_ace_sym_finish<T, LMAX, NMAX><<<dim3(pl.tiles, TA / 16), kFinThreads, 0, ctx->stream>>>(g);
  APX_LAUNCH_CHECK(ctx);
  return APX_OK;
}

}  // namespace

template <class T>
size_t sym_scratch(const apx_ace_model* m, int n_act) {
  const SymPlan<T> p = sym_plan<T>(m, n_act);
  return p.slab + p.epart;
}

size_t sym_scratch_most(const apx_ace_model* m, int n_act) {
  auto most = [&](auto t) {
    using T = decltype(t);
    constexpr int TA = sym_tile<T>();
    const size_t tiles = ((size_t)n_act + TA - 1) / TA;
    return std::min<size_t>(kSymMaxSplit * tiles, kSymBlocks) * (share_slab<T>(m) + sizeof(double) * 2 * TA);
  };
  return std::max(most(float{}), most(double{}));
}

template <class T>
apx_status sym_products(apx_ctx* ctx, const apx_ace_model* m, const T* A, T* B, T* slope, int n_act,
                        const double* e_anch, const int* active, double* e_site, void* scratch) {
  const int nm = sym_nmax(m->n_max);
#define APX_SYM_CASE(LM_, NM_) \
  if (m->l_max == LM_ && nm == NM_)                                                                      \
    return sym_launch<T, LM_, NM_>(ctx, m, A, B, slope, n_act, e_anch, active, e_site, scratch);
  APX_SYM_CASE(3, 8)
  APX_SYM_CASE(3, 10)
  APX_SYM_CASE(3, 12)
  APX_SYM_CASE(4, 8)
  APX_SYM_CASE(4, 10)
  APX_SYM_CASE(4, 12)
#undef APX_SYM_CASE
  return fail(ctx, APX_EINVAL, "unsupported ACE model size");
}

template size_t sym_scratch<float>(const apx_ace_model*, int);
template size_t sym_scratch<double>(const apx_ace_model*, int);
template apx_status sym_products<float>(apx_ctx*, const apx_ace_model*, const float*, float*, float*, int,
                                        const double*, const int*, double*, void*);
template apx_status sym_products<double>(apx_ctx*, const apx_ace_model*, const double*, double*, double*, int,
                                         const double*, const int*, double*, void*);

}  // namespace apx
