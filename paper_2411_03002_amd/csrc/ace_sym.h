// Product basis of the atomic cluster expansion: host interface of the symmetric kernels.
#pragma once

#include "ace_model.h"

namespace apx {

// Atoms per tile of the product kernels: one per lane in float32; in float64 sixteen, with
// four label pairs side by side in a wave.
template <class T>
constexpr int sym_tile() { return sizeof(T) == 4 ? 64 : 16; }

// Row stride of the atomic base (and of its projected adjoint) in elements: 16-byte groups.
inline int sym_stride(int na) { return (na + 3) & ~3; }

// Device scratch of sym_products beyond the atomic base, in bytes.
template <class T>
size_t sym_scratch(const apx_ace_model* m, int n_act);
// The most that a call of at most n_act atoms takes, in either type.
size_t sym_scratch_most(const apx_ace_model* m, int n_act);

// For the atoms active[0..n_act) with the atomic base A [n_act][sym_stride(na)]:
// e_site[active[q]] = E_q (random part plus e_anch[q]); slope[q] = F_eps'(phi2) (null: not
// wanted); B [n_act][sym_stride(na)] (may be A) the projected adjoint
// B'[lm * n_max + k] = sum_n Wp[l][n][k] dE/dA_nlm.
template <class T>
apx_status sym_products(apx_ctx* ctx, const apx_ace_model* m, const T* A, T* B, T* slope, int n_act,
                        const double* e_anch, const int* active, double* e_site, void* scratch);

// dc1, dc2 [n_basis]: the gradients of sum_q w E_q with respect to the coefficients (w null: 1),
// from the atomic base and the slopes of sym_products (ace_grad.hip).
size_t ace_grad_scratch(const apx_ace_model* m, int n_act);
template <class T>
apx_status ace_grad(apx_ctx* ctx, const apx_ace_model* m, const T* A, const T* slope, const double* w,
                    const int* active, int n_act, double* dc1, double* dc2, void* scratch);

}  // namespace apx
