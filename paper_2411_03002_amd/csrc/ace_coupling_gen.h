// Generated by gen_coupling.py -- do not edit.  Real Gaunt coupling of two harmonic blocks
// (degrees l1 <= l2), one component M at a time, scaled by 1 / kSymScale[l1][l2][L].
#pragma once
#include <hip/hip_runtime.h>
namespace apx {
constexpr double kSymScale[5][5][5] = {
    {{0.28209479177387803, 1, 1, 1, 1}, {1, 0.28209479177387808, 1, 1, 1}, {1, 1, 0.2820947917738782, 1, 1}, {1, 1, 1, 0.2820947917738782, 1}, {1, 1, 1, 1, 0.28209479177387781}},
    {{1, 1, 1, 1, 1}, {0.28209479177387803, 1, 0.2185096861184159, 1, 1}, {1, 0.21850968611841587, 1, 0.23359668032760758, 1}, {1, 1, 0.18467439092237189, 1, 0.23841361350444787}, {1, 1, 1, 0.23841361350444787, 1}},
    {{1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, {0.2820947917738782, 1, 0.18022375157286874, 1, 0.23841361350444834}, {1, 0.18467439092237187, 1, 0.14867700967939756, 1}, {1, 1, 0.16858388283618389, 1, 0.14046334619025072}},
    {{1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, {0.2820947917738782, 1, 0.1880631945159188, 1, 0.099322584599279881}, {1, 0.23032943298089015, 1, 0.099322584599279853, 1}},
    {{1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, {0.28209479177387786, 1, 0.19036461502711166, 1, 0.1190989127526999}},
};
constexpr int kGauntTerms[5][5][5] = {
    {{1, 0, 0, 0, 0}, {0, 3, 0, 0, 0}, {0, 0, 5, 0, 0}, {0, 0, 0, 7, 0}, {0, 0, 0, 0, 9}},
    {{0, 3, 0, 0, 0}, {3, 0, 11, 0, 0}, {0, 11, 0, 21, 0}, {0, 0, 21, 0, 31}, {0, 0, 0, 31, 0}},
    {{0, 0, 5, 0, 0}, {0, 11, 0, 21, 0}, {5, 0, 25, 0, 37}, {0, 21, 0, 41, 0}, {0, 0, 37, 0, 61}},
    {{0, 0, 0, 7, 0}, {0, 0, 21, 0, 31}, {0, 21, 0, 41, 0}, {7, 0, 41, 0, 67}, {0, 31, 0, 67, 0}},
    {{0, 0, 0, 0, 9}, {0, 0, 0, 31, 0}, {0, 0, 37, 0, 61}, {0, 31, 0, 67, 0}, {9, 0, 61, 0, 97}},
};
template <int L1, int L2, int M> struct SymP;
template <> struct SymP<0, 0, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      P[0] = t;
    }
  }
};
template <> struct SymP<0, 1, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      P[1] = t;
    }
  }
};
template <> struct SymP<0, 1, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      P[1] = t;
    }
  }
};
template <> struct SymP<0, 1, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      P[1] = t;
    }
  }
};
template <> struct SymP<0, 2, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      P[2] = t;
    }
  }
};
template <> struct SymP<0, 2, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      P[2] = t;
    }
  }
};
template <> struct SymP<0, 2, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      P[2] = t;
    }
  }
};
template <> struct SymP<0, 2, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      P[2] = t;
    }
  }
};
template <> struct SymP<0, 2, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      P[2] = t;
    }
  }
};
template <> struct SymP<0, 3, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 3, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 3, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 3, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 3, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 3, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[5];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 3, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[6];
      P[3] = t;
    }
  }
};
template <> struct SymP<0, 4, -4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[0];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[1];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[2];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[3];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[4];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[5];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[6];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[7];
      P[4] = t;
    }
  }
};
template <> struct SymP<0, 4, 4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[8];
      P[4] = t;
    }
  }
};
template <> struct SymP<1, 1, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[2], b[0], t);
      P[2] = t;
    }
  }
};
template <> struct SymP<1, 1, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[1], b[0], t);
      P[2] = t;
    }
  }
};
template <> struct SymP<1, 1, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[2], b[2], t);
      P[0] = t;
      P[2] = T(-0.57735026918962584) * t;
    }
    {
      T t = a[1] * b[1];
      P[0] = P[0] + t;
      P[2] = fma(T(1.154700538379251), t, P[2]);
    }
  }
};
template <> struct SymP<1, 1, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[1] * b[2];
      t = fma(a[2], b[1], t);
      P[2] = t;
    }
  }
};
template <> struct SymP<1, 1, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(-a[2], b[2], t);
      P[2] = -t;
    }
  }
};
template <> struct SymP<1, 2, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      t = fma(a[2], b[0], t);
      P[3] = T(0.96824583655185315) * t;
    }
  }
};
template <> struct SymP<1, 2, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      t = fma(a[1], b[0], t);
      t = fma(a[2], b[1], t);
      P[3] = T(0.79056941504209466) * t;
    }
  }
};
template <> struct SymP<1, 2, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      P[1] = T(-0.57735026918962584) * t;
      P[3] = T(0.86602540378443804) * t;
    }
    {
      T t = a[0] * b[4];
      t = fma(-a[2], b[0], t);
      P[1] = P[1] - t;
      P[3] = fma(T(0.24999999999999928), t, P[3]);
    }
    {
      T t = a[1] * b[1];
      P[1] = P[1] + t;
      P[3] = P[3] + t;
    }
  }
};
template <> struct SymP<1, 2, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[2], b[3], t);
      P[1] = t;
      P[3] = T(-0.61237243569579436) * t;
    }
    {
      T t = a[1] * b[2];
      P[1] = fma(T(1.1547005383792512), t, P[1]);
      P[3] = fma(T(1.0606601717798201), t, P[3]);
    }
  }
};
template <> struct SymP<1, 2, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[2], b[4], t);
      P[1] = t;
      P[3] = T(-0.24999999999999986) * t;
    }
    {
      T t = a[1] * b[3];
      P[1] = P[1] + t;
      P[3] = P[3] + t;
    }
    {
      T t = a[2] * b[2];
      P[1] = fma(T(-0.57735026918962584), t, P[1]);
      P[3] = fma(T(0.86602540378443804), t, P[3]);
    }
  }
};
template <> struct SymP<1, 2, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(-a[1], b[4], t);
      t = fma(-a[2], b[3], t);
      P[3] = T(-0.79056941504209466) * t;
    }
  }
};
template <> struct SymP<1, 2, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(-a[2], b[4], t);
      P[3] = T(-0.96824583655185392) * t;
    }
  }
};
template <> struct SymP<1, 3, -4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[6];
      t = fma(a[2], b[0], t);
      P[4] = T(0.96609178307929611) * t;
    }
  }
};
template <> struct SymP<1, 3, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[5];
      t = fma(a[2], b[1], t);
      P[4] = T(0.83666002653407578) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[0];
      P[4] = fma(T(0.68313005106397384), t, P[4]);
    }
  }
};
template <> struct SymP<1, 3, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      t = fma(a[2], b[2], t);
      P[2] = T(-0.31622776601683789) * t;
      if constexpr (LMAX >= 4) P[4] = T(0.70710678118654835) * t;
    }
    {
      T t = a[0] * b[6];
      t = fma(-a[2], b[0], t);
      P[2] = fma(T(-1.2247448713915892), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.18257418583505539), t, P[4]);
    }
    {
      T t = a[1] * b[1];
      P[2] = P[2] + t;
      if constexpr (LMAX >= 4) P[4] = fma(T(0.89442719099991697), t, P[4]);
    }
  }
};
template <> struct SymP<1, 3, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      P[2] = T(-0.7745966692414834) * t;
      if constexpr (LMAX >= 4) P[4] = T(0.81649658092772581) * t;
    }
    {
      T t = a[0] * b[5];
      t = fma(-a[2], b[1], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(0.31622776601683783), t, P[4]);
    }
    {
      T t = a[1] * b[2];
      P[2] = fma(T(1.2649110640673522), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = P[4] + t;
    }
  }
};
template <> struct SymP<1, 3, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[2], b[4], t);
      P[2] = T(1.0954451150103319) * t;
      if constexpr (LMAX >= 4) P[4] = T(-0.63245553203367699) * t;
    }
    {
      T t = a[1] * b[3];
      P[2] = fma(T(1.341640786499873), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.0327955589886459), t, P[4]);
    }
  }
};
template <> struct SymP<1, 3, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[2], b[5], t);
      P[2] = t;
      if constexpr (LMAX >= 4) P[4] = T(-0.31622776601683822) * t;
    }
    {
      T t = a[1] * b[4];
      P[2] = fma(T(1.2649110640673522), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = P[4] + t;
    }
    {
      T t = a[2] * b[3];
      P[2] = fma(T(-0.7745966692414834), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.81649658092772581), t, P[4]);
    }
  }
};
template <> struct SymP<1, 3, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[2], b[6], t);
      P[2] = T(1.2247448713915883) * t;
      if constexpr (LMAX >= 4) P[4] = T(-0.18257418583505561) * t;
    }
    {
      T t = a[0] * b[2];
      t = fma(-a[2], b[4], t);
      P[2] = fma(T(0.31622776601683716), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.70710678118654846), t, P[4]);
    }
    {
      T t = a[1] * b[5];
      P[2] = P[2] + t;
      if constexpr (LMAX >= 4) P[4] = fma(T(0.89442719099991697), t, P[4]);
    }
  }
};
template <> struct SymP<1, 3, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[1];
      t = fma(-a[2], b[5], t);
      P[4] = T(-0.83666002653407623) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[6];
      P[4] = fma(T(0.68313005106397384), t, P[4]);
    }
  }
};
template <> struct SymP<1, 3, 4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[0];
      t = fma(-a[2], b[6], t);
      P[4] = T(-0.96609178307929744) * t;
    }
  }
};
template <> struct SymP<1, 4, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[6];
      t = fma(a[2], b[2], t);
      P[3] = T(-0.18257418583505552) * t;
    }
    {
      T t = a[0] * b[8];
      t = fma(-a[2], b[0], t);
      P[3] = fma(T(-0.96609178307929744), t, P[3]);
    }
    {
      T t = a[1] * b[1];
      P[3] = fma(T(0.68313005106397384), t, P[3]);
    }
  }
};
template <> struct SymP<1, 4, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[5];
      t = fma(a[2], b[3], t);
      P[3] = T(-0.31622776601683822) * t;
    }
    {
      T t = a[0] * b[7];
      t = fma(-a[2], b[1], t);
      P[3] = fma(T(-0.83666002653407623), t, P[3]);
    }
    {
      T t = a[1] * b[2];
      P[3] = fma(T(0.89442719099991697), t, P[3]);
    }
  }
};
template <> struct SymP<1, 4, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      P[3] = T(-0.63245553203367699) * t;
    }
    {
      T t = a[0] * b[6];
      t = fma(-a[2], b[2], t);
      P[3] = fma(T(-0.70710678118654846), t, P[3]);
    }
    {
      T t = a[1] * b[3];
      P[3] = P[3] + t;
    }
  }
};
template <> struct SymP<1, 4, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      t = fma(a[2], b[5], t);
      P[3] = T(0.81649658092772581) * t;
    }
    {
      T t = a[1] * b[4];
      P[3] = fma(T(1.0327955589886459), t, P[3]);
    }
  }
};
template <> struct SymP<1, 4, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[2], b[6], t);
      P[3] = T(0.70710678118654835) * t;
    }
    {
      T t = a[1] * b[5];
      P[3] = P[3] + t;
    }
    {
      T t = a[2] * b[4];
      P[3] = fma(T(-0.63245553203367699), t, P[3]);
    }
  }
};
template <> struct SymP<1, 4, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[2], b[7], t);
      P[3] = T(0.83666002653407578) * t;
    }
    {
      T t = a[0] * b[3];
      t = fma(-a[2], b[5], t);
      P[3] = fma(T(0.31622776601683783), t, P[3]);
    }
    {
      T t = a[1] * b[6];
      P[3] = fma(T(0.89442719099991674), t, P[3]);
    }
  }
};
template <> struct SymP<1, 4, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[2], b[8], t);
      P[3] = T(0.96609178307929611) * t;
    }
    {
      T t = a[0] * b[2];
      t = fma(-a[2], b[6], t);
      P[3] = fma(T(0.18257418583505547), t, P[3]);
    }
    {
      T t = a[1] * b[7];
      P[3] = fma(T(0.68313005106397384), t, P[3]);
    }
  }
};
template <> struct SymP<2, 2, -4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[4];
      t = fma(a[4], b[0], t);
      P[4] = t;
    }
  }
};
template <> struct SymP<2, 2, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[3];
      t = fma(a[1], b[4], t);
      t = fma(a[3], b[0], t);
      t = fma(a[4], b[1], t);
      P[4] = T(0.70710678118654691) * t;
    }
  }
};
template <> struct SymP<2, 2, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[2], b[0], t);
      P[2] = -t;
      if constexpr (LMAX >= 4) P[4] = T(0.65465367070797664) * t;
    }
    {
      T t = a[1] * b[3];
      t = fma(a[3], b[1], t);
      P[2] = fma(T(0.86602540378443849), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.75592894601845395), t, P[4]);
    }
  }
};
template <> struct SymP<2, 2, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      t = fma(-a[1], b[4], t);
      t = fma(a[3], b[0], t);
      t = fma(-a[4], b[1], t);
      P[2] = T(0.86602540378443849) * t;
      if constexpr (LMAX >= 4) P[4] = T(-0.26726124191242406) * t;
    }
    {
      T t = a[1] * b[2];
      t = fma(a[2], b[1], t);
      P[2] = fma(T(0.50000000000000011), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.92582009977254953), t, P[4]);
    }
  }
};
template <> struct SymP<2, 2, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[4], b[4], t);
      P[0] = t;
      P[2] = -t;
      if constexpr (LMAX >= 4) P[4] = T(0.16903085094570297) * t;
    }
    {
      T t = a[1] * b[1];
      t = fma(a[3], b[3], t);
      P[0] = P[0] + t;
      P[2] = fma(T(0.50000000000000011), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.67612340378281399), t, P[4]);
    }
    {
      T t = a[2] * b[2];
      P[0] = P[0] + t;
      P[2] = P[2] + t;
      if constexpr (LMAX >= 4) P[4] = fma(T(1.0141851056742193), t, P[4]);
    }
  }
};
template <> struct SymP<2, 2, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[1], b[0], t);
      t = fma(a[3], b[4], t);
      t = fma(a[4], b[3], t);
      P[2] = T(0.86602540378443849) * t;
      if constexpr (LMAX >= 4) P[4] = T(-0.26726124191242406) * t;
    }
    {
      T t = a[2] * b[3];
      t = fma(a[3], b[2], t);
      P[2] = fma(T(0.50000000000000011), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.92582009977254953), t, P[4]);
    }
  }
};
template <> struct SymP<2, 2, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[1] * b[1];
      t = fma(-a[3], b[3], t);
      P[2] = T(-0.86602540378443871) * t;
      if constexpr (LMAX >= 4) P[4] = T(-0.7559289460184544) * t;
    }
    {
      T t = a[2] * b[4];
      t = fma(a[4], b[2], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(0.65465367070797675), t, P[4]);
    }
  }
};
template <> struct SymP<2, 2, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[1];
      t = fma(a[1], b[0], t);
      t = fma(-a[3], b[4], t);
      t = fma(-a[4], b[3], t);
      P[4] = T(-0.70710678118654691) * t;
    }
  }
};
template <> struct SymP<2, 2, 4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[0];
      t = fma(-a[4], b[4], t);
      P[4] = -t;
    }
  }
};
template <> struct SymP<2, 3, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      t = fma(a[4], b[2], t);
      P[3] = T(-0.63245553203367577) * t;
    }
    {
      T t = a[1] * b[5];
      t = fma(a[3], b[1], t);
      P[3] = P[3] + t;
    }
    {
      T t = a[2] * b[0];
      P[3] = fma(T(-1.4142135623730954), t, P[3]);
    }
  }
};
template <> struct SymP<2, 3, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      P[3] = T(-1.2649110640673522) * t;
    }
    {
      T t = a[1] * b[4];
      t = fma(a[3], b[2], t);
      P[3] = fma(T(0.77459666924148407), t, P[3]);
    }
    {
      T t = a[1] * b[6];
      t = fma(-a[3], b[0], t);
      P[3] = P[3] - t;
    }
  }
};
template <> struct SymP<2, 3, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      t = fma(-a[4], b[2], t);
      P[1] = T(-0.31622776601683794) * t;
      P[3] = T(0.97979589711327175) * t;
    }
    {
      T t = a[0] * b[6];
      t = fma(-a[4], b[0], t);
      P[1] = fma(T(-1.2247448713915894), t, P[1]);
      P[3] = fma(T(0.63245553203367566), t, P[3]);
    }
    {
      T t = a[1] * b[3];
      P[1] = fma(T(-0.77459666924148352), t, P[1]);
      P[3] = fma(T(0.39999999999999869), t, P[3]);
    }
    {
      T t = a[1] * b[5];
      t = fma(-a[3], b[1], t);
      P[1] = P[1] - t;
      P[3] = fma(T(-0.7745966692414844), t, P[3]);
    }
    {
      T t = a[2] * b[2];
      P[1] = fma(T(1.0954451150103321), t, P[1]);
      P[3] = fma(T(0.84852813742385624), t, P[3]);
    }
  }
};
template <> struct SymP<2, 3, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[4], b[5], t);
      P[1] = t;
      P[3] = T(-1.2649110640673522) * t;
    }
    {
      T t = a[1] * b[2];
      t = fma(a[3], b[4], t);
      P[1] = fma(T(1.2649110640673524), t, P[1]);
      P[3] = fma(T(0.39999999999999869), t, P[3]);
    }
    {
      T t = a[2] * b[3];
      P[1] = fma(T(1.3416407864998732), t, P[1]);
      P[3] = fma(T(1.1313708498984774), t, P[3]);
    }
  }
};
template <> struct SymP<2, 3, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[4], b[6], t);
      P[1] = T(1.2247448713915894) * t;
      P[3] = T(-0.63245553203367555) * t;
    }
    {
      T t = a[0] * b[2];
      t = fma(a[4], b[4], t);
      P[1] = fma(T(-0.31622776601683794), t, P[1]);
      P[3] = fma(T(0.97979589711327175), t, P[3]);
    }
    {
      T t = a[1] * b[1];
      t = fma(a[3], b[5], t);
      P[1] = P[1] + t;
      P[3] = fma(T(0.77459666924148407), t, P[3]);
    }
    {
      T t = a[2] * b[4];
      P[1] = fma(T(1.0954451150103321), t, P[1]);
      P[3] = fma(T(0.84852813742385624), t, P[3]);
    }
    {
      T t = a[3] * b[3];
      P[1] = fma(T(-0.77459666924148352), t, P[1]);
      P[3] = fma(T(0.39999999999999869), t, P[3]);
    }
  }
};
template <> struct SymP<2, 3, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[1] * b[0];
      t = fma(a[3], b[6], t);
      P[3] = t;
    }
    {
      T t = a[1] * b[2];
      t = fma(-a[3], b[4], t);
      P[3] = fma(T(-0.7745966692414844), t, P[3]);
    }
    {
      T t = a[4] * b[3];
      P[3] = fma(T(-1.2649110640673511), t, P[3]);
    }
  }
};
template <> struct SymP<2, 3, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(-a[4], b[4], t);
      P[3] = T(0.63245553203367577) * t;
    }
    {
      T t = a[1] * b[1];
      t = fma(-a[3], b[5], t);
      P[3] = P[3] - t;
    }
    {
      T t = a[2] * b[6];
      P[3] = fma(T(-1.4142135623730954), t, P[3]);
    }
  }
};
template <> struct SymP<2, 4, -4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[6];
      t = fma(a[4], b[2], t);
      P[4] = T(-0.53452248382484924) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[7];
      t = fma(a[3], b[1], t);
      P[4] = P[4] + t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[0];
      P[4] = fma(T(-1.6329931618554532), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[5];
      t = fma(a[4], b[3], t);
      P[4] = T(-0.80178372573727341) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[6];
      t = fma(a[3], b[2], t);
      P[4] = fma(T(0.94491118252306838), t, P[4]);
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[8];
      t = fma(-a[3], b[0], t);
      P[4] = P[4] - t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[1];
      P[4] = fma(T(-0.40824829046386252), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      P[2] = T(0.23904572186687828) * t;
      if constexpr (LMAX >= 4) P[4] = T(-1.3552618543578778) * t;
    }
    {
      T t = a[0] * b[8];
      t = fma(-a[4], b[0], t);
      P[2] = fma(T(-1.4142135623730963), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.5345224838248479), t, P[4]);
    }
    {
      T t = a[1] * b[5];
      t = fma(a[3], b[3], t);
      P[2] = fma(T(-0.37796447300922736), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.64285714285714224), t, P[4]);
    }
    {
      T t = a[1] * b[7];
      t = fma(-a[3], b[1], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.94491118252306883), t, P[4]);
    }
    {
      T t = a[2] * b[2];
      P[2] = fma(T(0.92582009977255131), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.46656947481584238), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[5];
      t = fma(-a[4], b[3], t);
      P[2] = T(-0.37796447300922725) * t;
      if constexpr (LMAX >= 4) P[4] = T(1.0101525445522106) * t;
    }
    {
      T t = a[0] * b[7];
      t = fma(-a[4], b[1], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(0.8017837257372733), t, P[4]);
    }
    {
      T t = a[1] * b[4];
      P[2] = fma(T(-0.95618288746751645), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.3194382824999708), t, P[4]);
    }
    {
      T t = a[1] * b[6];
      t = fma(-a[3], b[2], t);
      P[2] = fma(T(-1.0690449676496983), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.64285714285714346), t, P[4]);
    }
    {
      T t = a[2] * b[3];
      P[2] = fma(T(1.3093073414159533), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.99146013398366739), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[4], b[6], t);
      P[2] = T(0.92582009977255153) * t;
      if constexpr (LMAX >= 4) P[4] = T(-1.3552618543578778) * t;
    }
    {
      T t = a[1] * b[3];
      t = fma(a[3], b[5], t);
      P[2] = fma(T(1.3093073414159526), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.31943828249997047), t, P[4]);
    }
    {
      T t = a[2] * b[4];
      P[2] = fma(T(1.4342743312012729), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.1664236870396105), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[4], b[7], t);
      P[2] = t;
      if constexpr (LMAX >= 4) P[4] = T(-0.80178372573727341) * t;
    }
    {
      T t = a[0] * b[3];
      t = fma(a[4], b[5], t);
      P[2] = fma(T(-0.37796447300922725), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.0101525445522106), t, P[4]);
    }
    {
      T t = a[1] * b[2];
      t = fma(a[3], b[6], t);
      P[2] = fma(T(1.0690449676496978), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.64285714285714191), t, P[4]);
    }
    {
      T t = a[2] * b[5];
      P[2] = fma(T(1.3093073414159528), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.99146013398366684), t, P[4]);
    }
    {
      T t = a[3] * b[4];
      P[2] = fma(T(-0.95618288746751623), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.31943828249997058), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[4], b[8], t);
      P[2] = T(1.4142135623730931) * t;
      if constexpr (LMAX >= 4) P[4] = T(-0.53452248382484924) * t;
    }
    {
      T t = a[1] * b[1];
      t = fma(a[3], b[7], t);
      P[2] = P[2] + t;
      if constexpr (LMAX >= 4) P[4] = fma(T(0.94491118252306838), t, P[4]);
    }
    {
      T t = a[1] * b[3];
      t = fma(-a[3], b[5], t);
      P[2] = fma(T(0.37796447300922653), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.64285714285714368), t, P[4]);
    }
    {
      T t = a[2] * b[6];
      P[2] = fma(T(0.92582009977255131), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.46656947481584315), t, P[4]);
    }
    {
      T t = a[4] * b[4];
      P[2] = fma(T(0.23904572186687897), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-1.3552618543578783), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[3];
      t = fma(-a[4], b[5], t);
      P[4] = T(0.80178372573727352) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[0];
      t = fma(a[3], b[8], t);
      P[4] = P[4] + t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[2];
      t = fma(-a[3], b[6], t);
      P[4] = fma(T(-0.94491118252306927), t, P[4]);
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[7];
      P[4] = fma(T(-0.40824829046386252), t, P[4]);
    }
  }
};
template <> struct SymP<2, 4, 4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[2];
      t = fma(-a[4], b[6], t);
      P[4] = T(0.53452248382484835) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[1];
      t = fma(-a[3], b[7], t);
      P[4] = P[4] - t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[8];
      P[4] = fma(T(-1.6329931618554523), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, -4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[4];
      t = fma(a[2], b[6], t);
      t = fma(a[4], b[0], t);
      t = fma(a[6], b[2], t);
      P[4] = T(-1.1832159566199238) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[5];
      t = fma(a[5], b[1], t);
      P[4] = fma(T(1.5275252316519459), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[3];
      t = fma(a[3], b[0], t);
      P[4] = T(-2.0493901531919199) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[4];
      t = fma(a[2], b[5], t);
      t = fma(a[4], b[1], t);
      t = fma(a[5], b[2], t);
      P[4] = fma(T(0.68313005106397406), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      t = fma(-a[2], b[6], t);
      t = fma(a[4], b[0], t);
      t = fma(-a[6], b[2], t);
      P[2] = T(-0.49999999999999978) * t;
      if constexpr (LMAX >= 4) P[4] = T(1.3416407864998749) * t;
    }
    {
      T t = a[1] * b[3];
      t = fma(a[3], b[1], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.44721359549995848), t, P[4]);
    }
    {
      T t = a[2] * b[4];
      t = fma(a[4], b[2], t);
      P[2] = fma(T(0.77459666924148318), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.1547005383792521), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[5];
      t = fma(-a[1], b[6], t);
      t = fma(a[5], b[0], t);
      t = fma(-a[6], b[1], t);
      P[2] = T(0.79056941504209444) * t;
      if constexpr (LMAX >= 4) P[4] = -t;
    }
    {
      T t = a[1] * b[4];
      t = fma(-a[2], b[5], t);
      t = fma(a[4], b[1], t);
      t = fma(-a[5], b[2], t);
      P[2] = fma(T(0.6123724356957948), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.0327955589886442), t, P[4]);
    }
    {
      T t = a[2] * b[3];
      t = fma(a[3], b[2], t);
      P[2] = fma(T(0.31622776601683661), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = P[4] + t;
    }
  }
};
template <> struct SymP<3, 3, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[6], b[6], t);
      P[0] = t;
      P[2] = T(-1.1180339887498947) * t;
      if constexpr (LMAX >= 4) P[4] = T(0.77459666924148385) * t;
    }
    {
      T t = a[1] * b[1];
      t = fma(a[5], b[5], t);
      P[0] = P[0] + t;
      if constexpr (LMAX >= 4) P[4] = fma(T(-1.8073922282301289), t, P[4]);
    }
    {
      T t = a[2] * b[2];
      t = fma(a[4], b[4], t);
      P[0] = P[0] + t;
      P[2] = fma(T(0.67082039324993603), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.25819888974715854), t, P[4]);
    }
    {
      T t = a[3] * b[3];
      P[0] = P[0] + t;
      P[2] = fma(T(0.89442719099991652), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.5491933384829684), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[1], b[0], t);
      t = fma(a[5], b[6], t);
      t = fma(a[6], b[5], t);
      P[2] = T(0.79056941504209499) * t;
      if constexpr (LMAX >= 4) P[4] = -t;
    }
    {
      T t = a[1] * b[2];
      t = fma(a[2], b[1], t);
      t = fma(a[4], b[5], t);
      t = fma(a[5], b[4], t);
      P[2] = fma(T(0.6123724356957948), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.0327955589886442), t, P[4]);
    }
    {
      T t = a[3] * b[4];
      t = fma(a[4], b[3], t);
      P[2] = fma(T(0.31622776601683644), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = P[4] + t;
    }
  }
};
template <> struct SymP<3, 3, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[2], b[0], t);
      t = fma(a[4], b[6], t);
      t = fma(a[6], b[4], t);
      P[2] = T(-0.49999999999999978) * t;
      if constexpr (LMAX >= 4) P[4] = T(1.3416407864998747) * t;
    }
    {
      T t = a[2] * b[2];
      t = fma(-a[4], b[4], t);
      P[2] = fma(T(-0.77459666924148352), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-1.154700538379251), t, P[4]);
    }
    {
      T t = a[3] * b[5];
      t = fma(a[5], b[3], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.44721359549995643), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[2];
      t = fma(a[2], b[1], t);
      t = fma(-a[4], b[5], t);
      t = fma(-a[5], b[4], t);
      P[4] = T(-0.68313005106397418) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[3] * b[6];
      t = fma(a[6], b[3], t);
      P[4] = fma(T(-2.0493901531919199), t, P[4]);
    }
  }
};
template <> struct SymP<3, 3, 4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[2];
      t = fma(a[2], b[0], t);
      t = fma(-a[4], b[6], t);
      t = fma(-a[6], b[4], t);
      P[4] = T(1.1832159566199223) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[1];
      t = fma(-a[5], b[5], t);
      P[4] = fma(T(-1.5275252316519476), t, P[4]);
    }
  }
};
template <> struct SymP<3, 4, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[4];
      P[3] = T(0.77459666924148418) * t;
    }
    {
      T t = a[1] * b[5];
      t = fma(a[5], b[3], t);
      P[3] = P[3] - t;
    }
    {
      T t = a[2] * b[6];
      t = fma(a[4], b[2], t);
      P[3] = fma(T(1.3416407864998754), t, P[3]);
    }
    {
      T t = a[2] * b[8];
      t = fma(-a[4], b[0], t);
      P[3] = fma(T(1.1832159566199236), t, P[3]);
    }
    {
      T t = a[3] * b[1];
      P[3] = fma(T(-2.0493901531919203), t, P[3]);
    }
  }
};
template <> struct SymP<3, 4, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[5];
      t = fma(-a[6], b[3], t);
      P[3] = -t;
    }
    {
      T t = a[1] * b[4];
      P[3] = fma(T(-1.8073922282301291), t, P[3]);
    }
    {
      T t = a[1] * b[8];
      t = fma(-a[5], b[0], t);
      P[3] = fma(T(-1.527525231651949), t, P[3]);
    }
    {
      T t = a[2] * b[5];
      t = fma(a[4], b[3], t);
      P[3] = fma(T(1.0327955589886439), t, P[3]);
    }
    {
      T t = a[2] * b[7];
      t = fma(-a[4], b[1], t);
      P[3] = fma(T(-0.68313005106397406), t, P[3]);
    }
    {
      T t = a[3] * b[2];
      P[3] = fma(T(-0.44721359549995854), t, P[3]);
    }
  }
};
template <> struct SymP<3, 4, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[6];
      t = fma(-a[6], b[2], t);
      P[1] = T(-0.18898223650461382) * t;
      P[3] = T(1.3416407864998749) * t;
    }
    {
      T t = a[0] * b[8];
      t = fma(-a[6], b[0], t);
      P[1] = P[1] - t;
      P[3] = fma(T(1.1832159566199234), t, P[3]);
    }
    {
      T t = a[1] * b[5];
      t = fma(-a[5], b[3], t);
      P[1] = fma(T(-0.32732683535398882), t, P[1]);
      P[3] = fma(T(1.0327955589886439), t, P[3]);
    }
    {
      T t = a[1] * b[7];
      t = fma(-a[5], b[1], t);
      P[1] = fma(T(-0.86602540378443915), t, P[1]);
      P[3] = fma(T(-0.68313005106397406), t, P[3]);
    }
    {
      T t = a[2] * b[4];
      P[1] = fma(T(-0.65465367070797809), t, P[1]);
      P[3] = fma(T(0.25819888974715882), t, P[3]);
    }
    {
      T t = a[2] * b[6];
      t = fma(-a[4], b[2], t);
      P[1] = fma(T(-0.73192505471140068), t, P[1]);
      P[3] = fma(T(-1.1547005383792512), t, P[3]);
    }
    {
      T t = a[3] * b[3];
      P[1] = fma(T(0.84515425472851613), t, P[1]);
      P[3] = P[3] + t;
    }
  }
};
template <> struct SymP<3, 4, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[6], b[7], t);
      P[1] = T(0.70710678118654802) * t;
      P[3] = T(-2.0493901531919207) * t;
    }
    {
      T t = a[1] * b[2];
      t = fma(a[5], b[6], t);
      P[1] = fma(T(0.92582009977255242), t, P[1]);
      P[3] = fma(T(-0.44721359549995854), t, P[3]);
    }
    {
      T t = a[2] * b[3];
      t = fma(a[4], b[5], t);
      P[1] = fma(T(1.0350983390135311), t, P[1]);
      P[3] = P[3] + t;
    }
    {
      T t = a[3] * b[4];
      P[1] = fma(T(1.0690449676496989), t, P[1]);
      P[3] = fma(T(1.5491933384829686), t, P[3]);
    }
  }
};
template <> struct SymP<3, 4, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[6], b[8], t);
      P[1] = t;
      P[3] = T(-1.1832159566199243) * t;
    }
    {
      T t = a[0] * b[2];
      t = fma(a[6], b[6], t);
      P[1] = fma(T(-0.1889822365046136), t, P[1]);
      P[3] = fma(T(1.3416407864998745), t, P[3]);
    }
    {
      T t = a[1] * b[1];
      t = fma(a[5], b[7], t);
      P[1] = fma(T(0.86602540378443915), t, P[1]);
      P[3] = fma(T(0.68313005106397384), t, P[3]);
    }
    {
      T t = a[1] * b[3];
      t = fma(a[5], b[5], t);
      P[1] = fma(T(-0.32732683535398882), t, P[1]);
      P[3] = fma(T(1.0327955589886439), t, P[3]);
    }
    {
      T t = a[2] * b[2];
      t = fma(a[4], b[6], t);
      P[1] = fma(T(0.73192505471140057), t, P[1]);
      P[3] = fma(T(1.1547005383792517), t, P[3]);
    }
    {
      T t = a[3] * b[5];
      P[1] = fma(T(0.84515425472851613), t, P[1]);
      P[3] = P[3] + t;
    }
    {
      T t = a[4] * b[4];
      P[1] = fma(T(-0.65465367070797809), t, P[1]);
      P[3] = fma(T(0.25819888974715921), t, P[3]);
    }
  }
};
template <> struct SymP<3, 4, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[3];
      t = fma(a[6], b[5], t);
      P[3] = -t;
    }
    {
      T t = a[1] * b[0];
      t = fma(a[5], b[8], t);
      P[3] = fma(T(1.5275252316519459), t, P[3]);
    }
    {
      T t = a[2] * b[1];
      t = fma(a[4], b[7], t);
      P[3] = fma(T(0.68313005106397429), t, P[3]);
    }
    {
      T t = a[2] * b[3];
      t = fma(-a[4], b[5], t);
      P[3] = fma(T(-1.0327955589886453), t, P[3]);
    }
    {
      T t = a[3] * b[6];
      P[3] = fma(T(-0.44721359549995648), t, P[3]);
    }
    {
      T t = a[5] * b[4];
      P[3] = fma(T(-1.8073922282301278), t, P[3]);
    }
  }
};
template <> struct SymP<3, 4, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[1] * b[3];
      t = fma(-a[5], b[5], t);
      P[3] = t;
    }
    {
      T t = a[2] * b[0];
      t = fma(a[4], b[8], t);
      P[3] = fma(T(-1.1832159566199241), t, P[3]);
    }
    {
      T t = a[2] * b[2];
      t = fma(-a[4], b[6], t);
      P[3] = fma(T(-1.3416407864998747), t, P[3]);
    }
    {
      T t = a[3] * b[7];
      P[3] = fma(T(-2.0493901531919203), t, P[3]);
    }
    {
      T t = a[6] * b[4];
      P[3] = fma(T(0.77459666924148418), t, P[3]);
    }
  }
};
template <> struct SymP<4, 4, -4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[4];
      t = fma(a[4], b[0], t);
      P[4] = T(0.8944271909999173) * t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[5];
      t = fma(a[3], b[7], t);
      t = fma(a[5], b[1], t);
      t = fma(a[7], b[3], t);
      P[4] = P[4] - t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[6];
      t = fma(a[6], b[2], t);
      P[4] = fma(T(1.1338934190276815), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, -3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[5];
      t = fma(-a[3], b[8], t);
      t = fma(a[5], b[0], t);
      t = fma(-a[8], b[3], t);
      P[4] = -t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[4];
      t = fma(a[4], b[1], t);
      P[4] = fma(T(-1.3416407864998741), t, P[4]);
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[5];
      t = fma(a[3], b[6], t);
      t = fma(a[5], b[2], t);
      t = fma(a[6], b[3], t);
      P[4] = fma(T(0.37796447300922736), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, -2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[6];
      t = fma(-a[2], b[8], t);
      t = fma(a[6], b[0], t);
      t = fma(-a[8], b[2], t);
      P[2] = T(-0.39440531887330799) * t;
      if constexpr (LMAX >= 4) P[4] = T(1.1338934190276817) * t;
    }
    {
      T t = a[1] * b[5];
      t = fma(-a[3], b[7], t);
      t = fma(a[5], b[1], t);
      t = fma(-a[7], b[3], t);
      P[2] = fma(T(-0.59160797830996159), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.37796447300922675), t, P[4]);
    }
    {
      T t = a[2] * b[4];
      t = fma(a[4], b[2], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.7027642214999329), t, P[4]);
    }
    {
      T t = a[3] * b[5];
      t = fma(a[5], b[3], t);
      P[2] = fma(T(0.74535599249992968), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.85714285714285698), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, -1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[7];
      t = fma(-a[1], b[8], t);
      t = fma(a[7], b[0], t);
      t = fma(-a[8], b[1], t);
      P[2] = T(0.73786478737262184) * t;
      if constexpr (LMAX >= 4) P[4] = -t;
    }
    {
      T t = a[1] * b[6];
      t = fma(-a[2], b[7], t);
      t = fma(a[6], b[1], t);
      t = fma(-a[7], b[2], t);
      P[2] = fma(T(0.69721668877839649), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.37796447300922703), t, P[4]);
    }
    {
      T t = a[2] * b[5];
      t = fma(-a[3], b[6], t);
      t = fma(a[5], b[2], t);
      t = fma(-a[6], b[3], t);
      P[2] = fma(T(0.47434164902525616), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.85714285714285698), t, P[4]);
    }
    {
      T t = a[3] * b[4];
      t = fma(a[4], b[3], t);
      P[2] = fma(T(0.23570226039551537), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.57498890849994344), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, 0> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[0];
      t = fma(a[8], b[8], t);
      P[0] = t;
      P[2] = T(-1.2049281521534192) * t;
      if constexpr (LMAX >= 4) P[4] = T(0.89442719099991641) * t;
    }
    {
      T t = a[1] * b[1];
      t = fma(a[7], b[7], t);
      P[0] = P[0] + t;
      P[2] = fma(T(-0.30123203803835424), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-1.3416407864998734), t, P[4]);
    }
    {
      T t = a[2] * b[2];
      t = fma(a[6], b[6], t);
      P[0] = P[0] + t;
      P[2] = fma(T(0.34426518632954733), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.70276422149993201), t, P[4]);
    }
    {
      T t = a[3] * b[3];
      t = fma(a[5], b[5], t);
      P[0] = P[0] + t;
      P[2] = fma(T(0.73156352095028987), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.57498890849994466), t, P[4]);
    }
    {
      T t = a[4] * b[4];
      P[0] = P[0] + t;
      P[2] = fma(T(0.8606629658238717), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(1.1499778169998935), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, 1> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[1];
      t = fma(a[1], b[0], t);
      t = fma(a[7], b[8], t);
      t = fma(a[8], b[7], t);
      P[2] = T(0.73786478737262184) * t;
      if constexpr (LMAX >= 4) P[4] = -t;
    }
    {
      T t = a[1] * b[2];
      t = fma(a[2], b[1], t);
      t = fma(a[6], b[7], t);
      t = fma(a[7], b[6], t);
      P[2] = fma(T(0.69721668877839682), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.37796447300922692), t, P[4]);
    }
    {
      T t = a[2] * b[3];
      t = fma(a[3], b[2], t);
      t = fma(a[5], b[6], t);
      t = fma(a[6], b[5], t);
      P[2] = fma(T(0.47434164902525616), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.85714285714285698), t, P[4]);
    }
    {
      T t = a[4] * b[5];
      t = fma(a[5], b[4], t);
      P[2] = fma(T(0.23570226039551523), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.57498890849994322), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, 2> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    {
      T t = a[0] * b[2];
      t = fma(a[2], b[0], t);
      t = fma(a[6], b[8], t);
      t = fma(a[8], b[6], t);
      P[2] = T(-0.39440531887330799) * t;
      if constexpr (LMAX >= 4) P[4] = T(1.1338934190276815) * t;
    }
    {
      T t = a[1] * b[3];
      t = fma(a[3], b[1], t);
      t = fma(a[5], b[7], t);
      t = fma(a[7], b[5], t);
      P[2] = fma(T(-0.59160797830996137), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(0.37796447300922675), t, P[4]);
    }
    {
      T t = a[3] * b[3];
      t = fma(-a[5], b[5], t);
      P[2] = fma(T(-0.74535599249992979), t, P[2]);
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.85714285714285932), t, P[4]);
    }
    {
      T t = a[4] * b[6];
      t = fma(a[6], b[4], t);
      P[2] = P[2] - t;
      if constexpr (LMAX >= 4) P[4] = fma(T(-0.70276422149993145), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, 3> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[0] * b[3];
      t = fma(a[3], b[0], t);
      t = fma(a[5], b[8], t);
      t = fma(a[8], b[5], t);
      P[4] = -t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[3];
      t = fma(a[3], b[2], t);
      t = fma(-a[5], b[6], t);
      t = fma(-a[6], b[5], t);
      P[4] = fma(T(-0.37796447300922698), t, P[4]);
    }
    if constexpr (LMAX >= 4) {
      T t = a[4] * b[7];
      t = fma(a[7], b[4], t);
      P[4] = fma(T(-1.3416407864998743), t, P[4]);
    }
  }
};
template <> struct SymP<4, 4, 4> {
  template <int LMAX, class T>
  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {
    if constexpr (LMAX >= 4) {
      T t = a[1] * b[3];
      t = fma(a[3], b[1], t);
      t = fma(-a[5], b[7], t);
      t = fma(-a[7], b[5], t);
      P[4] = t;
    }
    if constexpr (LMAX >= 4) {
      T t = a[2] * b[2];
      t = fma(-a[6], b[6], t);
      P[4] = fma(T(-1.1338934190276817), t, P[4]);
    }
    if constexpr (LMAX >= 4) {
      T t = a[4] * b[8];
      t = fma(a[8], b[4], t);
      P[4] = fma(T(0.8944271909999143), t, P[4]);
    }
  }
};
}  // namespace apx
