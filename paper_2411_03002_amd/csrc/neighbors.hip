// Cell-list neighbour build: full Verlet list in neighbour-major ELL layout, rows in
// ascending neighbour index.
#include <climits>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "device_util.h"

namespace apx {

constexpr int kNbCap = 128;     // largest row capacity (max_nb)
constexpr int kRowCap = 192;    // entries of a row kept while it is found
constexpr int kCellWaves = 4;   // waves per block; a block serves atoms of one cell
constexpr int kCandCap = 1024;  // candidates staged in LDS (more are read from global memory)

// Orders the LDS accesses of one wave (the LDS executes a wave's accesses in issue order;
// this keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One step of a bitonic network across the wave: partner lane = lane ^ J; lanes with `low` keep the
// smaller key.  The exchanges stay in the vector unit: quad permutations (1, 2), a half-row mirror and
// a quad reversal (4), a row rotation by eight (8), row and half-wave swaps (16, 32).  Through the LDS
// permutation instead, the 21 steps of a 64-key sort were a chain of 21 LDS round trips.  The minimum
// and the maximum read the partner's lane themselves (the compiler makes two moves of it); s_nop 1 is
// the two wait states between a vector write and its read through another lane.
template <int J>
__device__ __forceinline__ int bitonic_step(int v, bool low) {
  int lo, hi;
  if constexpr (J >= 16) {
    const auto r = J == 16 ? __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false)
                           : __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    lo = min((int)r[0], (int)r[1]);
    hi = max((int)r[0], (int)r[1]);
  } else if constexpr (J == 4) {
    const int m = __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false);
    asm volatile("s_nop 1\n\tv_min_i32_dpp %0, %2, %3 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_i32_dpp %1, %2, %3 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf"
        : "=&v"(lo), "=&v"(hi) : "v"(m), "v"(v));
  } else if constexpr (J == 8) {
    asm volatile("s_nop 1\n\tv_min_i32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_max_i32_dpp %1, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf"
        : "=&v"(lo), "=&v"(hi) : "v"(v));
  } else if constexpr (J == 2) {
    asm volatile("s_nop 1\n\tv_min_i32_dpp %0, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_i32_dpp %1, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
        : "=&v"(lo), "=&v"(hi) : "v"(v));
  } else {
    asm volatile("s_nop 1\n\tv_min_i32_dpp %0, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_i32_dpp %1, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
        : "=&v"(lo), "=&v"(hi) : "v"(v));
  }
  return low ? lo : hi;
}

// The steps J, J / 2, ... 1 of the stage that sorts blocks of K keys, element e = lane + 64 h.
template <int K, int J, int H>
__device__ __forceinline__ void bitonic_stage(int (&v)[H], int lane) {
  if constexpr (J == 64) {  // partners are the lane's own two elements (K = 128: ascending)
    const int a = min(v[0], v[1]), b = max(v[0], v[1]);
    v[0] = a;
    v[1] = b;
  } else {
#pragma unroll
    for (int h = 0; h < H; ++h) v[h] = bitonic_step<J>(v[h], ((lane & J) == 0) == (((lane + 64 * h) & K) == 0));
  }
  if constexpr (J > 1) bitonic_stage<K, J / 2, H>(v, lane);
}

// Sorts 64 H keys ascending.
template <int H>
__device__ __forceinline__ void wave_sort(int (&v)[H], int lane) {
  bitonic_stage<2, 1>(v, lane);
  bitonic_stage<4, 2>(v, lane);
  bitonic_stage<8, 4>(v, lane);
  bitonic_stage<16, 8>(v, lane);
  bitonic_stage<32, 16>(v, lane);
  bitonic_stage<64, 32>(v, lane);
  if constexpr (H == 2) bitonic_stage<128, 64>(v, lane);
}

// Candidate e lies in stencil cell s with pref[s] <= e < pref[s + 1] (pref has 32 entries, those past
// the 27th hold the number of candidates).
__device__ __forceinline__ int candidate(const int* cell_atoms, const int* start, const int* pref, int e) {
  int s = 0;
#pragma unroll
  for (int h = 16; h > 0; h >>= 1) s += s + h < 32 && pref[s + h] <= e ? h : 0;
  return cell_atoms[start[s] + (e - pref[s])];
}

// Appends the lanes' j with `ok` to the wave's row at cnt, in lane order; entries past kRowCap are
// only counted.
__device__ __forceinline__ void append(bool ok, int j, int* row, int& cnt) {
  const unsigned long long m = __ballot(ok);
  if (ok) {
    const int p = cnt + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    if (p < kRowCap) row[p] = j;
  }
  cnt += __popcll(m);
}

struct BuildDev {
  double rl2, edge[3];
  float in2, out2;      // float32 squared distances below / from which a pair is surely inside / outside
  float lx[3], ilx[3];  // period and its inverse where an axis has too few cells (0: no image is needed)
};

// One block per cell, or per 1 / parts of a cell's atoms where the cells alone are few.  The candidates
// (atoms of the up to 27 neighbouring cells, fewer for grids with fewer than 3 cells along a periodic
// axis) are staged in LDS as float32 offsets from the cell's centre at their nearest image; each wave
// takes atoms of the cell in turn and tests 64 candidates at a time, appends the accepted indices to its
// LDS row by ballot, sorts the row across the wave and writes it out.
//
// Bound by vector instructions.  Six of seven candidates lie outside the list radius, so the test is
// done in float32: with the squares staged beside the offsets a squared distance (less the atom's own
// square) is three multiply-adds, some ten instructions per 64 candidates with the append (in float64
// with the image found per pair some 45).  It is off by less than 5e-6 of the cell's edge squared; a row
// with a candidate within twice that of the list radius squared is tested again in float64, with the
// operation order of the other kernels, so the rows are those of the float64 test.
// A cell with an atom outside the reach of its grid cell (an unwrapped position), or with more candidates
// than are staged, is tested in float64 from global memory throughout.
// Measured (us, with the read-back of the row length), before / now: rows of 54 entries, 860 atoms 67 / 33,
// 130,466 atoms 174 / 110, 440,320 atoms 509 / 290, 4,102,125 atoms 4,030 / 2,264; 258 vector and 195 scalar
// instructions per atom.
__global__ void __launch_bounds__(kCellWaves * 64) k_build(const double* __restrict__ pos, int n, Grid g, BuildDev bd,
                                                            const int* __restrict__ cell_start,
                                                            const int* __restrict__ cell_atoms, int parts, int max_nb,
                                                            int* __restrict__ count, int* __restrict__ idx,
                                                            int* __restrict__ flags) {
  __shared__ float4 cand[kCandCap];  // offset from the centre, its square
  __shared__ int cand_j[kCandCap];
  __shared__ int rows[kCellWaves][kRowCap];
  __shared__ int sc_start[27], sc_pref[32], sc_wrap[27];
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const int c = b / parts, part = b - c * parts;
  const int b0 = cell_start[c], own = cell_start[c + 1] - b0;
  if (part * kCellWaves >= own) return;  // uniform over the block
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ci[3] = {c % g.nc[0], (c / g.nc[0]) % g.nc[1], c / (g.nc[0] * g.nc[1])};
  if (wv == 0) {
    // stencil cell `lane` (< 27): offsets -1..1 per axis, restricted as for the grid
    int sz = 0, st = 0, wrap = 0;  // (wrap: two bits per axis, 1 for the image below, 2 for the image above)
    if (lane < 27) {
      const int o[3] = {lane % 3 - 1, (lane / 3) % 3 - 1, lane / 9 - 1};
      bool ok = true;
      int cc[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const bool below = ci[d] > 0, above = ci[d] < g.nc[d] - 1;
        const bool both = g.per[d] && g.nc[d] >= 3;
        // (a periodic axis of two cells has the other one at offset 1 only, one of a single cell none)
        ok = ok && (o[d] >= 0 || both || (!g.per[d] && below)) &&
             (o[d] <= 0 || both || (g.per[d] ? g.nc[d] == 2 : above));
        cc[d] = ci[d] + o[d];
        if (g.per[d]) {
          wrap |= (cc[d] < 0 ? 1 : (cc[d] >= g.nc[d] ? 2 : 0)) << (2 * d);
          cc[d] = cc[d] < 0 ? g.nc[d] - 1 : (cc[d] >= g.nc[d] ? 0 : cc[d]);
        }
      }
      if (ok) {
        const int id = cc[0] + g.nc[0] * (cc[1] + g.nc[1] * cc[2]);
        st = cell_start[id];
        sz = cell_start[id + 1] - st;
      }
    }
    int incl = sz;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      const int u = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += u;
    }
    if (lane < 27) {
      sc_start[lane] = st;
      sc_wrap[lane] = wrap;
    }
    if (lane < 32) sc_pref[lane] = incl - sz;  // (lanes past 26 add nothing: the total)
  }
  __syncthreads();
  const int M = __builtin_amdgcn_readfirstlane(sc_pref[27]);
  const int self = __builtin_amdgcn_readfirstlane(sc_pref[13]);  // the cell's own atoms among the candidates
  bool near = M <= kCandCap && bd.out2 < 1e30f;  // (float32 squares stay finite)
  if (near) {
    if (tid < 216) {  // eight threads per stencil cell
      const int s = tid >> 3, first = sc_start[s], at = sc_pref[s], size = sc_pref[s + 1] - at, im = sc_wrap[s];
      double c0[3], reach[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double edge = bd.edge[d];
        const int m = (im >> (2 * d)) & 3;
        c0[d] = g.lo[d] + (ci[d] + 0.5) * edge + (m == 1 ? g.L[d] : (m == 2 ? -g.L[d] : 0.0));
        reach[d] = 1.501 * edge;
      }
      for (int q = tid & 7; q < size; q += 8) {
        const int j = cell_atoms[first + q];
        float r[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double x = pos[(size_t)d * n + j] - c0[d];
          near = near && fabs(x) <= reach[d];
          r[d] = (float)x;
        }
        cand[at + q] = make_float4(r[0], r[1], r[2], r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
        cand_j[at + q] = j;
      }
    } else {  // the last 64 candidates are filled up with ones that no row takes
      for (int e = M + tid - 216; e < ((M + 63) & ~63); e += kCellWaves * 64 - 216)
        cand[e] = make_float4(0.f, 0.f, 0.f, 2e30f);
    }
  }
  near = __syncthreads_and(near);
  int* row = rows[wv];
  int longest = 0;
  const bool image = bd.lx[0] > 0.f || bd.lx[1] > 0.f || bd.lx[2] > 0.f;
  for (int a = part * kCellWaves + wv; a < own; a += parts * kCellWaves) {
    int cnt = 0;
    bool exact = !near;
    const int me = self + a;
    if (near) {
      const float4 ri = cand[me];
      unsigned long long border = 0;
      const float mx = -2.f * ri.x, my = -2.f * ri.y, mz = -2.f * ri.z;
      const float in = bd.in2 - ri.w, out = bd.out2 - ri.w;
      auto sweep = [&](auto image_c) {
        for (int s0 = 0; s0 < M && cnt <= kRowCap - 64; s0 += 64) {
          const int e = s0 + lane;
          const float4 rj = cand[e];
          float r2;  // (less the atom's square)
          bool ok;
          if constexpr (decltype(image_c)::value) {
            float dx = rj.x - ri.x, dy = rj.y - ri.y, dz = rj.z - ri.z;
            dx -= rintf(dx * bd.ilx[0]) * bd.lx[0];
            dy -= rintf(dy * bd.ilx[1]) * bd.lx[1];
            dz -= rintf(dz * bd.ilx[2]) * bd.lx[2];
            r2 = dx * dx + dy * dy + dz * dz - ri.w;
            ok = r2 < out && e < M;
          } else {
            r2 = __builtin_fmaf(mx, rj.x, __builtin_fmaf(my, rj.y, __builtin_fmaf(mz, rj.z, rj.w)));
            ok = r2 < out;
          }
          const unsigned long long m = __ballot(ok);
          border |= m & ~__ballot(r2 < in);
          // (the row has room for all 64: see the loop's condition)
          if (ok) row[__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, cnt))] = e;
          cnt += __popcll(m);
        }
      };
      if (image)
        sweep(std::true_type{});
      else
        sweep(std::false_type{});
      // the row holds the atom itself; past 128 entries it may not be complete
      exact = border != 0 || cnt > 128;
    }
    const int i = __builtin_amdgcn_readfirstlane(near ? cand_j[me] : cell_atoms[b0 + a]);
    if (exact) {
      // float64: the entries of the row, or all candidates where the row does not hold them all
      const bool all = !near || cnt > 128;
      const int total = all ? M : cnt;
      const double xi = pos[i], yi = pos[(size_t)n + i], zi = pos[2 * (size_t)n + i];
      cnt = 0;
      for (int s0 = 0; s0 < total; s0 += 64) {
        wave_lds_sync();
        const int e = s0 + lane;
        int j = i;
        if (e < total) j = all ? candidate(cell_atoms, sc_start, sc_pref, e) : cand_j[row[e]];
        wave_lds_sync();  // (an entry is read before its place is written)
        const double dx = min_image(pos[j] - xi, g.L[0], 0.5 * g.L[0], g.per[0]);
        const double dy = min_image(pos[(size_t)n + j] - yi, g.L[1], 0.5 * g.L[1], g.per[1]);
        const double dz = min_image(pos[2 * (size_t)n + j] - zi, g.L[2], 0.5 * g.L[2], g.per[2]);
        append(j != i && sq_dist_exact(dx, dy, dz) < bd.rl2, j, row, cnt);
      }
    }
    wave_lds_sync();
    auto key = [&](int e) {
      if (e >= cnt) return INT_MAX;
      const int v = row[e];
      return exact ? v : (v == me ? INT_MAX : cand_j[v]);
    };
    int v[2] = {key(lane), INT_MAX};
    if (cnt <= 64) {
      int v0[1] = {v[0]};
      wave_sort(v0, lane);
      v[0] = v0[0];
    } else {
      v[1] = key(lane + 64);
      wave_sort(v, lane);
    }
    if (!exact) cnt -= 1;
    const int kept = cnt < max_nb ? cnt : max_nb;
    if (lane < kept) idx[(size_t)lane * n + i] = v[0];
    if (lane + 64 < kept) idx[(size_t)(lane + 64) * n + i] = v[1];
    if (lane == 0) count[i] = cnt;
    longest = cnt > longest ? cnt : longest;
    wave_lds_sync();
  }
  // the longest row and the capacity flag: one atomic per wave (longest is wave-uniform)
  if (lane == 0 && longest > 0) {
    if (longest > max_nb) atomicOr(&flags[0], 4);
    sparse_atomic_max(&flags[1], longest);
  }
}

// Blocks that fill the card, and the most that share a cell: below this many cells each is split, so that
// a few large cells do not leave the card idle.
constexpr long long kFillBlocks = 1024, kMaxParts = 8;

BuildDev build_dev(const Grid& g, double r_list) {
  BuildDev bd;
  double edge = 0.0;
  for (int d = 0; d < 3; ++d) {
    bd.edge[d] = g.L[d] / g.nc[d];
    edge = std::fmax(edge, bd.edge[d]);
    // offsets of a cell's atoms and its candidates differ by at most two edges: the nearest image to the
    // centre is the nearest to the atom from five cells on
    const bool image = g.per[d] && g.nc[d] < 5;
    bd.lx[d] = image ? (float)g.L[d] : 0.f;
    bd.ilx[d] = image ? (float)(1.0 / g.L[d]) : 0.f;
  }
  const double slack = 1e-5 * edge * edge;
  bd.rl2 = r_list * r_list;
  bd.in2 = (float)(bd.rl2 - slack);
  bd.out2 = (float)(bd.rl2 + slack);
  return bd;
}

}  // namespace apx

using namespace apx;

extern "C" apx_status apx_build_neighbors(apx_ctx* ctx, const apx_atoms* atoms, double r_list,
                                          apx_nlist* nl, int32_t* needed) {
  if (!ctx) return APX_EINVAL;
  apx_status s = check_atoms(ctx, atoms);
  if (s != APX_OK) return s;
  if (!nl || !needed) return fail(ctx, APX_EINVAL, "nl and needed are required");
  if (nl->n != atoms->n) return fail(ctx, APX_EINVAL, "nlist size %lld != atoms %lld", (long long)nl->n, (long long)atoms->n);
  if (nl->max_nb < 1 || nl->max_nb > kNbCap) return fail(ctx, APX_EINVAL, "max_nb must be in 1..%d", kNbCap);
  if (atoms->n > 0 && (!nl->count || !nl->idx)) return fail(ctx, APX_EINVAL, "nlist arrays are NULL");
  if (!(r_list > 0.0)) return fail(ctx, APX_EINVAL, "r_list must be positive");
  for (int d = 0; d < 3; ++d)
    if (atoms->periodic[d] && !(r_list < 0.5 * (atoms->hi[d] - atoms->lo[d])))
      return fail(ctx, APX_EINVAL, "r_list %.4f must be below half the periodic box (axis %d)", r_list, d);
  nl->r_list = r_list;
  const int n = (int)atoms->n;
  if (n == 0) {
    *needed = 0;
    return APX_OK;
  }
  Grid g = make_grid(atoms, r_list);
  {
    ProfScope ps(ctx, "nbr.bin");
    s = bin_atoms(ctx, atoms, g);
  }
  if (s != APX_OK) return s;
  ProfScope ps(ctx, "nbr.build");
  const long long ncell = g.ncell();
  if (ncell > INT_MAX) return fail(ctx, APX_EINVAL, "too many cells (%lld)", ncell);
  const int parts = ncell >= kFillBlocks ? 1 : (int)(kFillBlocks / ncell < kMaxParts ? kFillBlocks / ncell : kMaxParts);
  k_build<<<(unsigned)(ncell * parts), kCellWaves * 64, 0, ctx->stream>>>(
      atoms->pos, n, g, build_dev(g, r_list), ctx->cell_start.as<int>(), ctx->cell_atoms.as<int>(), parts, nl->max_nb,
      nl->count, nl->idx, ctx->flags.as<int>());
  APX_LAUNCH_CHECK(ctx);
  int fl[2];
  s = read_ints(ctx, ctx->flags.as<int>(), fl, 2);
  if (s != APX_OK) return s;
  *needed = fl[1];
  if (fl[0] & 1) return fail(ctx, APX_EINVAL, "a coordinate lies outside the box along a non-periodic axis");
  if (fl[0] & 2) return fail(ctx, APX_ENONFINITE, "non-finite position");
  if (fl[0] & 4) return fail(ctx, APX_ECAPACITY, "neighbour row of %d entries exceeds max_nb %d", fl[1], nl->max_nb);
  return APX_OK;
}
