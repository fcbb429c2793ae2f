// Host-side construction of the ACE tables (basis catalogue, label pairs, coefficient slots) and
// their upload; the coefficients are laid out for the product kernels on the device.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdlib>
#include <utility>

#include "ace_coupling_gen.h"
#include "ace_model.h"

namespace apx {
namespace {

bool coupled(int l1, int l2, int l3) { return ((l1 + l2 + l3) % 2 == 0) && l3 >= std::abs(l1 - l2) && l3 <= l1 + l2; }

// The basis in the order of the definition: B1 (n), B2 (n1 <= n2, l), B3 over labels
// p = n (l_max + 1) + l, p1 <= p2 <= p3.
struct Catalogue {
  long long n_basis = 0;
  std::vector<int> index3;  // basis index of the triple p1 <= p2 <= p3, [p1][p2][p3]
  int npairs = 0, ntrip = 0;
  long long coupling_terms = 0, triple_width = 0;
};

int index2(int n_max, int l_max, int a, int b, int l) {  // a <= b
  return n_max + (l_max + 1) * (a * n_max - a * (a - 1) / 2 + b - a) + l;
}

Catalogue build_catalogue(int n_max, int l_max) {
  Catalogue c;
  const int LL = l_max + 1, P = n_max * LL;
  long long v = n_max + (long long)LL * n_max * (n_max + 1) / 2;
  c.index3.assign((size_t)P * P * P, -1);
  // the counts of apx_ace_model_stats, of an evaluation that takes every function once with the label
  // first in degree-major order (l, then n) as the third block: the pairs of the other two, and per
  // pair the degrees met (the kernels take all pairs and degrees, see ace_sym.hip)
  std::vector<unsigned char> met((size_t)P * P, 0);
  auto key = [&](int p) { return (p % LL) * n_max + p / LL; };
  for (int p1 = 0; p1 < P; ++p1)
    for (int p2 = p1; p2 < P; ++p2)
      for (int p3 = p2; p3 < P; ++p3) {
        if (!coupled(p1 % LL, p2 % LL, p3 % LL)) continue;
        c.index3[((size_t)p1 * P + p2) * P + p3] = (int)v++;
        std::array<int, 3> k = {key(p1), key(p2), key(p3)};
        std::sort(k.begin(), k.end());
        const int L = k[0] / n_max;
        unsigned char& m = met[(size_t)k[1] * P + k[2]];
        if (!m) ++c.npairs;
        if (!((m >> L) & 1)) c.coupling_terms += kGauntTerms[k[1] / n_max][k[2] / n_max][L];
        m |= (unsigned char)(1u << L);
        c.triple_width += 2 * L + 1;
        ++c.ntrip;
      }
  c.n_basis = v;
  return c;
}

// The label pairs (n1, n2) of type (l1, l2).
std::vector<std::pair<int, int>> label_pairs(int n_max, int l1, int l2) {
  std::vector<std::pair<int, int>> nn;
  for (int n2 = 0; n2 < n_max; ++n2)
    for (int n1 = l1 == l2 ? n2 : 0; n1 < n_max; ++n1) nn.push_back({n1, n2});
  return nn;
}

int triple_index(const Catalogue& c, int P, int a, int b, int r) {
  std::array<int, 3> q = {a, b, r};
  std::sort(q.begin(), q.end());
  return c.index3[((size_t)q[0] * P + q[1]) * P + q[2]];
}

// Tables of the product kernels for groups of `width` pairs (1: float32, 4: float64): the
// offsets, the pairs, and per coefficient slot the basis index and its factor (the number of
// times the output block occurs in the function times the scale of the generated coupling).
// A group of one pair is a row of 2 NMAX values; of four pairs the operand layout of the float64
// instructions: 16 rows x 4 pairs with the row fastest, then 4 rows x 4 pairs each.
struct SymHost {
  std::vector<int> off, pairs, slot;
  std::vector<double> factor;
  int low = 0;  // first slot of the rows of pairs of one degree
  int b1 = 0;   // and of the first-order pairs
};

SymHost build_sym(const Catalogue& c, int n_max, int l_max, int width) {
  SymHost s;
  s.off.assign(kSymOff, 0);
  const int LL = l_max + 1, P = n_max * LL, LM = LL * LL, R = 2 * sym_nmax(n_max);
  auto put = [&](int v, int o, double f) {
    s.slot.push_back(v < 0 ? -1 : 2 * v + (o & 1));
    s.factor.push_back(f);
  };
  // value(row o, member k) of one group, appended in the group's layout
  auto group = [&](auto&& value) {
    auto one = [&](int o, int k) {
      const std::pair<int, double> e = value(o, k);
      put(e.first, o, e.second);
    };
    if (width == 1) {
      for (int o = 0; o < R; ++o) one(o, 0);
      return;
    }
    for (int k = 0; k < 4; ++k)
      for (int o = 0; o < 16; ++o) one(o, k);
    for (int b = 16; b < R; b += 4)
      for (int k = 0; k < 4; ++k)
        for (int o = b; o < b + 4; ++o) one(o, k);
  };
  for (int l2 = 0; l2 < LL; ++l2)
    for (int l1 = 0; l1 <= l2; ++l1) {
      const int t = l2 * (l2 + 1) / 2 + l1;
      const auto nn = label_pairs(n_max, l1, l2);
      const int ng = ((int)nn.size() + width - 1) / width;
      s.off[kSymPairs + t] = (int)s.pairs.size();
      s.off[kSymNg + t] = ng;
      for (int p = 0; p < ng * width; ++p) {
        const auto q = p < (int)nn.size() ? nn[p] : std::make_pair(0, 0);
        s.pairs.push_back((q.first * LM + l1 * l1) | ((q.second * LM + l2 * l2) << 16));
      }
      for (int L = 0; L < LL; ++L) {
        if (!coupled(l1, l2, L)) continue;
        s.off[t * 5 + L] = (int)s.slot.size();
        for (int g = 0; g < ng; ++g)
          group([&](int o, int k) -> std::pair<int, double> {
            const int p = g * width + k, n3 = o >> 1;
            if (p >= (int)nn.size() || n3 >= n_max) return {-1, 0.0};
            const int r = n3 * LL + L, a = nn[p].first * LL + l1, b = nn[p].second * LL + l2;
            return {triple_index(c, P, a, b, r), (1 + (a == r) + (b == r)) * kSymScale[l1][l2][L]};
          });
      }
    }
  for (int L = 0; L < LL; ++L) {
    s.off[kSymB2 + L] = (int)s.slot.size();
    for (int g = 0; g * width < n_max; ++g)
      group([&](int o, int k) -> std::pair<int, double> {
        const int n = g * width + k, n3 = o >> 1;
        if (n >= n_max || n3 >= n_max) return {-1, 0.0};
        return {index2(n_max, l_max, std::min(n, n3), std::max(n, n3), L), n == n3 ? 2.0 : 1.0};
      });
  }
  if (width == 1) {
    while (s.slot.size() % 4) put(-1, 0, 0.0);
    s.low = (int)s.slot.size();
    for (int l = 0; l < LL; ++l)
      for (const auto& q : label_pairs(n_max, l, l))
        for (int o = 0; o < sym_low(sym_nmax(n_max)); ++o) {
          const int n1 = q.first, n2 = q.second, n3 = o / 2 - 1;  // (n1 >= n2)
          if (o < 2) put(index2(n_max, l_max, n2, n1, l), o, 1.0);
          else if (n3 >= n_max || (l == 0 && n3 > n2)) put(-1, 0, 0.0);
          else put(triple_index(c, P, n1 * LL + l, n2 * LL + l, n3 * LL), o, kSymScale[l][l][0]);
        }
  }
  // the kernels read up to two groups, or four pairs and two rows of low, ahead
  for (int k = 0; k < std::max(2 * width * R, 2 * sym_low(sym_nmax(n_max))); ++k) put(-1, 0, 0.0);
  for (int k = 0; k < std::max(3 * width, 4); ++k) s.pairs.push_back(0);
  s.b1 = (int)s.slot.size();
  for (int n = 0; n < n_max; ++n)
    for (int p = 0; p < 2; ++p) put(n, p, 1.0);
  return s;
}

// Tables of the coefficient gradients: items of sixteen pairs, dealt to the waves in order, the
// longest first.  Every function has one slot per coefficient: the block of the smallest degree
// is the row, and among blocks of equal degree the smallest radial index.
struct GradHost {
  std::vector<int> pairs, items, at;
  std::vector<double> scale;
};

GradHost build_grad(const Catalogue& c, int n_max, int l_max) {
  GradHost h;
  const int LL = l_max + 1, P = n_max * LL, R = 2 * sym_nmax(n_max);
  struct Item {
    int type, pair, slot, cost;
  };
  std::vector<Item> items;
  auto rows = [&](auto&& value, double scale) {
    for (int o = 0; o < R; ++o)
      for (int col = 0; col < 16; ++col) {
        const int v = o >> 1 < n_max ? value(o >> 1, col) : -1;
        h.at.push_back(v < 0 ? -1 : 2 * v + (o & 1));
        h.scale.push_back(scale);
      }
  };
  for (int l2 = 0; l2 < LL; ++l2)
    for (int l1 = 0; l1 <= l2; ++l1) {
      if (l2 - l1 > l1) continue;
      const auto nn = label_pairs(n_max, l1, l2);
      for (int p0 = 0; p0 < (int)nn.size(); p0 += 16) {
        Item it{l2 * (l2 + 1) / 2 + l1, (int)h.pairs.size(), (int)h.at.size(), 0};
        for (int k = 0; k < 16; ++k) {
          const auto q = p0 + k < (int)nn.size() ? nn[p0 + k] : std::make_pair(0, 0);
          h.pairs.push_back(q.first | (q.second << 16));
        }
        for (int L = l2 - l1; L <= l1; L += 2) {
          it.cost += 2 * L + 1;
          rows([&](int n3, int col) {
            if (p0 + col >= (int)nn.size()) return -1;
            const int n1 = nn[p0 + col].first, n2 = nn[p0 + col].second;
            if ((L == l1 && n3 > n1) || (L == l2 && n3 > n2)) return -1;
            return triple_index(c, P, n1 * LL + l1, n2 * LL + l2, n3 * LL + L);
          }, kSymScale[l1][l2][L]);
        }
        items.push_back(it);
      }
    }
  for (int L = 0; L < LL; ++L) {
    items.push_back({15 + L, 0, (int)h.at.size(), 2 * L + 1});
    rows([&](int n3, int col) {
      if (L == 0 && col == n_max) return n3;
      return col < n_max && n3 <= col ? index2(n_max, l_max, n3, col, L) : -1;
    }, 1.0);
  }
  std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b) { return a.cost > b.cost; });
  for (const Item& i : items) h.items.insert(h.items.end(), {i.type, i.pair, i.slot});
  return h;
}

template <class T>
__global__ void k_layout_coeffs(int n, const int* __restrict__ slot, const double* __restrict__ factor,
                                const double* __restrict__ c, long long n_basis, T* __restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int s = slot[k];
  out[k] = s < 0 ? T(0) : (T)(factor[k] * c[(s & 1) * n_basis + (s >> 1)]);
}

// Copies c1 and c2 to the device and writes both precisions' rows.
apx_status layout_coeffs(apx_ctx* ctx, apx_ace_model* m, const double* c1, const double* c2) {
  double* c = m->c.as<double>();
  const size_t b = sizeof(double) * (size_t)m->n_basis;
  // On the default stream: the copies, and so the rows, wait for the evaluations queued there, which end
  // with the rows they began with, also where the context's stream is another by now.
  APX_HIP(ctx, hipMemcpyAsync(c, c1, b, hipMemcpyHostToDevice, nullptr));
  APX_HIP(ctx, hipMemcpyAsync(c + m->n_basis, c2, b, hipMemcpyHostToDevice, nullptr));
  if (ctx->stream) APX_HIP(ctx, hipStreamSynchronize(nullptr));
  k_layout_coeffs<<<blocks_for(m->s64.n, 256), 256, 0, ctx->stream>>>(m->s64.n, m->s64.slot, m->s64.factor, c,
                                                                     m->n_basis, m->coef64.as<double>());
  k_layout_coeffs<<<blocks_for(m->s32.n, 256), 256, 0, ctx->stream>>>(m->s32.n, m->s32.slot, m->s32.factor, c,
                                                                     m->n_basis, m->coef32.as<float>());
  APX_LAUNCH_CHECK(ctx);
  APX_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return APX_OK;
}

template <class T>
hipError_t upload(DevBuf& buf, const std::vector<T>& h) {
  const hipError_t e = buf.ensure(h.size() * sizeof(T));
  return e == hipSuccess ? hipMemcpy(buf.p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) : e;
}

// Builds and uploads every table of the model.
apx_status model_tables(apx_ctx* ctx, apx_ace_model* m, const Catalogue& c, const apx_ace_desc* d) {
  std::vector<int> ints;
  std::vector<double> dbl;
  auto add = [](auto& to, const auto& from) {
    const size_t at = to.size();
    to.insert(to.end(), from.begin(), from.end());
    return at;
  };
  for (int l = 0; l <= m->l_max; ++l) {
    const double nl = std::sqrt((2.0 * l + 1.0) / (4.0 * M_PI));
    for (int k = 0; k < m->n_max * m->n_max; ++k) dbl.push_back(d->W[(size_t)l * m->n_max * m->n_max + k] * nl / m->s_a);
  }
  const std::vector<float> wp32(dbl.begin(), dbl.end());
  const SymHost h64 = build_sym(c, m->n_max, m->l_max, 4), h32 = build_sym(c, m->n_max, m->l_max, 1);
  const GradHost g = build_grad(c, m->n_max, m->l_max);
  struct At {
    size_t off, pairs, slot, factor;
  };
  auto place = [&](const SymHost& h) { return At{add(ints, h.off), add(ints, h.pairs), add(ints, h.slot), add(dbl, h.factor)}; };
  const At a64 = place(h64), a32 = place(h32);
  const size_t gp = add(ints, g.pairs), gi = add(ints, g.items), ga = add(ints, g.at), gs = add(dbl, g.scale);
  if (m->ints.ensure(ints.size() * sizeof(int)) != hipSuccess || m->doubles.ensure(dbl.size() * sizeof(double)) != hipSuccess ||
      m->wp32.ensure(wp32.size() * sizeof(float)) != hipSuccess ||
      m->c.ensure(2 * sizeof(double) * (size_t)m->n_basis) != hipSuccess ||
      m->coef64.ensure(h64.slot.size() * sizeof(double)) != hipSuccess ||
      m->coef32.ensure(h32.slot.size() * sizeof(float)) != hipSuccess)
    return fail(ctx, APX_ENOMEM, "ACE table allocation failed");
  if (upload(m->ints, ints) != hipSuccess || upload(m->doubles, dbl) != hipSuccess || upload(m->wp32, wp32) != hipSuccess)
    return fail(ctx, APX_EDEVICE, "ACE table upload failed");
  const int* ib = m->ints.as<int>();
  const double* db = m->doubles.as<double>();
  auto set = [&](auto& t, const SymHost& h, const At& a, auto* wp, auto* coef) {
    t.Wp = wp;
    t.coef = coef;
    t.b1 = coef + h.b1;
    t.low = coef + h.low;
    t.off = ib + a.off;
    t.pairs = ib + a.pairs;
    t.slot = ib + a.slot;
    t.factor = db + a.factor;
    t.n = (int)h.slot.size();
  };
  set(m->s64, h64, a64, db, m->coef64.as<double>());
  set(m->s32, h32, a32, m->wp32.as<float>(), m->coef32.as<float>());
  m->grad = GradTables{ib + gp, ib + gi, ib + ga, db + gs, (int)g.items.size() / 3, (int)g.at.size()};
  return layout_coeffs(ctx, m, d->c1, d->c2);
}

}  // namespace
}  // namespace apx

using namespace apx;

extern "C" int64_t apx_ace_num_basis(int32_t n_max, int32_t l_max) {
  if (n_max < 1 || n_max > 12 || (l_max != 3 && l_max != 4)) return -1;
  try {
    return build_catalogue(n_max, l_max).n_basis;
  } catch (...) {
    return -1;
  }
}

extern "C" apx_status apx_ace_model_create(apx_ctx* ctx, const apx_ace_desc* d, apx_ace_model** out) {
  if (!ctx) return APX_EINVAL;
  if (!d || !out) return fail(ctx, APX_EINVAL, "desc and out are required");
  *out = nullptr;
  if (d->n_max < 1 || d->n_max > 12) return fail(ctx, APX_EINVAL, "n_max must be in 1..12");
  if (d->l_max != 3 && d->l_max != 4) return fail(ctx, APX_EINVAL, "l_max must be 3 or 4");
  if (!d->W || !d->c1 || !d->c2) return fail(ctx, APX_EINVAL, "W, c1 and c2 are required");
  if (d->anchored && d->anchor.kind != APX_EAM_CLOSED)
    return fail(ctx, APX_EINVAL, "the EAM anchor of an ACE model must use the closed form");
  if (!(d->r_cut > 0.0) || !(d->h > 0.0) || !(d->s_a > 0.0) || !(d->eps > 0.0))
    return fail(ctx, APX_EINVAL, "r_cut, h, s_a and eps must be positive");
  apx_ace_model* m = nullptr;
  apx_status s;
  try {
    const Catalogue c = build_catalogue(d->n_max, d->l_max);
    m = new apx_ace_model();
    m->device = ctx->device;
    m->n_max = d->n_max;
    m->l_max = d->l_max;
    m->na = d->n_max * (d->l_max + 1) * (d->l_max + 1);
    m->n_basis = c.n_basis;
    m->npairs = c.npairs;
    m->ntrip = c.ntrip;
    m->coupling_terms = c.coupling_terms;
    m->triple_width = c.triple_width;
    m->r_cut = d->r_cut;
    m->h = d->h;
    m->s_a = d->s_a;
    m->eps = d->eps;
    m->anchored = d->anchored ? 1 : 0;
    m->anchor = d->anchor;
    s = model_tables(ctx, m, c, d);
  } catch (...) {
    s = fail(ctx, APX_ENOMEM, "ACE tables");
  }
  if (s != APX_OK) {
    delete m;
    return s;
  }
  *out = m;
  return APX_OK;
}

extern "C" apx_status apx_ace_model_set_coeffs(apx_ctx* ctx, apx_ace_model* m, const double* c1, const double* c2) {
  if (!ctx) return APX_EINVAL;
  if (!m || !c1 || !c2) return fail(ctx, APX_EINVAL, "model, c1 and c2 are required");
  return layout_coeffs(ctx, m, c1, c2);
}

extern "C" apx_status apx_ace_model_stats(const apx_ace_model* m, int64_t* out6) {
  if (!m || !out6) return APX_EINVAL;
  out6[0] = m->npairs;
  out6[1] = m->ntrip;
  out6[2] = m->coupling_terms;
  out6[3] = m->triple_width;
  out6[4] = m->n_basis;
  out6[5] = m->na;
  return APX_OK;
}

extern "C" void apx_ace_model_destroy(apx_ace_model* m) {
  if (!m) return;
  (void)hipSetDevice(m->device);
  delete m;
}
