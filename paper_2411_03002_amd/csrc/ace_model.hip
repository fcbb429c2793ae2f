// Host-side construction of the ACE coupling tables (basis catalogue, pair and triple
// lists, per-wave work split) and their upload to the device.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <map>
#include <tuple>
#include <utility>

#include "ace_coupling_gen.h"
#include "ace_model.h"
#include "ace_sym_gen.h"

namespace apx {
namespace {

template <int LMAX, int L1, int L2>
constexpr int couple_terms() {
  return Couple<LMAX, L1, L2>::kTerms;
}

template <int LMAX>
int terms_of(int l1, int l2) {
  static const int tab4[5][5] = {
      {couple_terms<4, 0, 0>(), couple_terms<4, 0, 1>(), couple_terms<4, 0, 2>(), couple_terms<4, 0, 3>(), couple_terms<4, 0, 4>()},
      {couple_terms<4, 1, 0>(), couple_terms<4, 1, 1>(), couple_terms<4, 1, 2>(), couple_terms<4, 1, 3>(), couple_terms<4, 1, 4>()},
      {couple_terms<4, 2, 0>(), couple_terms<4, 2, 1>(), couple_terms<4, 2, 2>(), couple_terms<4, 2, 3>(), couple_terms<4, 2, 4>()},
      {couple_terms<4, 3, 0>(), couple_terms<4, 3, 1>(), couple_terms<4, 3, 2>(), couple_terms<4, 3, 3>(), couple_terms<4, 3, 4>()},
      {couple_terms<4, 4, 0>(), couple_terms<4, 4, 1>(), couple_terms<4, 4, 2>(), couple_terms<4, 4, 3>(), couple_terms<4, 4, 4>()}};
  static const int tab3[4][4] = {
      {couple_terms<3, 0, 0>(), couple_terms<3, 0, 1>(), couple_terms<3, 0, 2>(), couple_terms<3, 0, 3>()},
      {couple_terms<3, 1, 0>(), couple_terms<3, 1, 1>(), couple_terms<3, 1, 2>(), couple_terms<3, 1, 3>()},
      {couple_terms<3, 2, 0>(), couple_terms<3, 2, 1>(), couple_terms<3, 2, 2>(), couple_terms<3, 2, 3>()},
      {couple_terms<3, 3, 0>(), couple_terms<3, 3, 1>(), couple_terms<3, 3, 2>(), couple_terms<3, 3, 3>()}};
  return LMAX == 4 ? tab4[l1][l2] : tab3[l1][l2];
}

bool coupled(int l1, int l2, int l3) { return ((l1 + l2 + l3) % 2 == 0) && l3 >= std::abs(l1 - l2) && l3 <= l1 + l2; }

// Coupling terms of (l1, l2) -> L alone (the per-degree functions Couple3).
template <int LMAX, int L1, int L2, int L>
constexpr int terms3() {
  if constexpr ((L1 + L2 + L) % 2 == 0 && L >= (L1 > L2 ? L1 - L2 : L2 - L1) && L <= L1 + L2 && L <= LMAX)
    return Couple3<LMAX, L1, L2, L>::kTerms;
  else
    return 0;
}
template <int LMAX, int L1, int L2, int... Ls>
int terms3_L(int L, std::integer_sequence<int, Ls...>) {
  int r = 0;
  ((r = (L == Ls ? terms3<LMAX, L1, L2, Ls>() : r)), ...);
  return r;
}
template <int LMAX, int L1, int... L2s>
int terms3_l2(int l2, int L, std::integer_sequence<int, L2s...>) {
  int r = 0;
  ((r = (l2 == L2s ? terms3_L<LMAX, L1, L2s>(L, std::make_integer_sequence<int, LMAX + 1>{}) : r)), ...);
  return r;
}
template <int LMAX, int... L1s>
int terms3_l1(int l1, int l2, int L, std::integer_sequence<int, L1s...>) {
  int r = 0;
  ((r = (l1 == L1s ? terms3_l2<LMAX, L1s>(l2, L, std::make_integer_sequence<int, LMAX + 1>{}) : r)), ...);
  return r;
}
int terms3_of(int l_max, int l1, int l2, int L) {
  return l_max == 4 ? terms3_l1<4>(l1, l2, L, std::make_integer_sequence<int, 5>{})
                    : terms3_l1<3>(l1, l2, L, std::make_integer_sequence<int, 4>{});
}

struct Catalogue {
  long long n_basis = 0;
  std::vector<int> pairs, t_v, b1_off, b1_v, b2_off, b2_v;
  std::vector<int> index3;  // basis index of the triple p1 <= p2 <= p3, [p1][p2][p3]
  int ntrip = 0;
  long long coupling_terms = 0, triple_width = 0;
};

Catalogue build_catalogue(int n_max, int l_max) {
  Catalogue c;
  const int LL = l_max + 1;
  const int P = n_max * LL;
  auto off = [&](int p) { int n = p / LL, l = p % LL; return n * LL * LL + l * l; };
  long long v = 0;
  for (int n = 0; n < n_max; ++n) {
    c.b1_off.push_back(n * LL * LL);
    c.b1_v.push_back((int)v++);
  }
  for (int n1 = 0; n1 < n_max; ++n1)
    for (int n2 = n1; n2 < n_max; ++n2)
      for (int l = 0; l < LL; ++l) {
        c.b2_off.push_back(n1 * LL * LL + l * l);
        c.b2_off.push_back(n2 * LL * LL + l * l);
        c.b2_off.push_back(l);
        c.b2_v.push_back((int)v++);
      }
  // B3: the basis indices follow the enumeration p1 <= p2 <= p3 of labels p = n (l_max+1) + l
  // (the basis definition).  The real Gaunt product of three blocks is symmetric in them,
  // so each triple may be evaluated as any of its labels coupled to the pair of the other
  // two.  Here the third block is the label that comes first in degree-major order
  // (l, then n) and the pair holds the other two: a pair (q2 <= q3) then meets third
  // blocks of degree L < l(q2) for every n, and of degree l(q2) for n <= n(q2).  Each pair
  // and degree thus has a run of third blocks n = 0, 1, ... of full or near-full length,
  // which makes fewer (pair, degree) combinations than the enumeration order would.
  struct PairTmp {
    int rec[kPairRec];
    std::vector<int> v;  // basis indices of its triples, in segment order
    double cost;
  };
  auto lkey = [LL](int p) { return std::make_pair(p % LL, p / LL); };
  c.index3.assign((size_t)P * P * P, -1);
  std::map<std::pair<int, int>, std::vector<std::vector<std::pair<int, int>>>> groups;  // (n3, v) by L
  for (int p1 = 0; p1 < P; ++p1)
    for (int p2 = p1; p2 < P; ++p2)
      for (int p3 = p2; p3 < P; ++p3) {
        if (!coupled(p1 % LL, p2 % LL, p3 % LL)) continue;
        c.index3[(p1 * P + p2) * P + p3] = (int)v;
        std::array<int, 3> s3 = {p1, p2, p3};
        std::sort(s3.begin(), s3.end(), [&](int a, int b) { return lkey(a) < lkey(b); });
        auto& g = groups[{s3[1], s3[2]}];
        if (g.empty()) g.resize(LL);
        g[s3[0] % LL].push_back({s3[0] / LL, (int)v++});
      }
  std::vector<PairTmp> tmp;
  for (auto& kv : groups) {
    const int q2 = kv.first.first, q3 = kv.first.second;
    const int l1 = q2 % LL, l2 = q3 % LL;
    auto& byL = kv.second;
    PairTmp pt{};
    pt.rec[0] = off(q2);
    pt.rec[1] = off(q3);
    pt.rec[2] = l1 * LL + l2;
    pt.rec[3] = q2 / LL;
    pt.rec[15] = q3 / LL;
    pt.cost = 8.0;
    int t = 0;
    for (int L = 0; L < LL; ++L) {
      std::sort(byL[L].begin(), byL[L].end());
      pt.rec[4 + L] = t;
      pt.rec[10 + L] = byL[L].empty() ? 0 : byL[L][0].first * LL * LL + L * L;
      if (!byL[L].empty()) {
        const int nterm = terms3_of(l_max, l1, l2, L);
        c.coupling_terms += nterm;
        pt.cost += nterm;
      }
      for (size_t e = 0; e < byL[L].size(); ++e) {
        // third blocks of one degree are consecutive in n: offsets step by (l_max+1)^2
        if (byL[L][e].first != byL[L][0].first + (int)e) throw 1;
        pt.v.push_back(byL[L][e].second);
        pt.cost += 2 * L + 1 + 2;
        c.triple_width += 2 * L + 1;
        ++t;
      }
    }
    for (int L = LL; L <= 5; ++L) pt.rec[4 + L] = t;
    tmp.push_back(pt);
  }
  c.n_basis = v;
  // group the pairs by coupling type so that a wave stays in one specialisation for
  // long runs of pairs (instruction-cache locality); within a type order them by the
  // label of larger degree, then the other label
  auto key = [LL](const PairTmp& a) {
    const int l1 = a.rec[2] / LL, l2 = a.rec[2] % LL;
    const int run = l1 >= l2 ? a.rec[3] : a.rec[15];
    const int oth = l1 >= l2 ? a.rec[15] : a.rec[3];
    return std::make_tuple(a.rec[2], run, oth);
  };
  std::stable_sort(tmp.begin(), tmp.end(), [&](const PairTmp& a, const PairTmp& b) { return key(a) < key(b); });
  std::vector<double> cost;
  int base = 0;
  for (auto& pt : tmp) {
    for (int L = 0; L <= 5; ++L) pt.rec[4 + L] += base;
    base += (int)pt.v.size();
    c.pairs.insert(c.pairs.end(), pt.rec, pt.rec + kPairRec);
    c.t_v.insert(c.t_v.end(), pt.v.begin(), pt.v.end());
    cost.push_back(pt.cost);
  }
  c.ntrip = base;
  return c;
}

// Tables of the symmetric product kernels for groups of `width` pairs (1: float32, 4: float64):
// the offsets, the pairs, and per coefficient slot the basis index and its factor (the number of
// times the output block occurs in the function times the scale of the generated coupling).
// A group of one pair is a row of 2 NMAX values; of four pairs the operand layout of the float64
// instructions: 16 rows x 4 pairs with the row fastest, then 4 rows x 4 pairs each.
struct SymHost {
  std::vector<int> off, pairs, v;
  std::vector<double> m;
};

SymHost build_sym(const Catalogue& c, int n_max, int l_max, int width) {
  SymHost s;
  s.off.assign(kSymOff, 0);
  const int LL = l_max + 1, P = n_max * LL, LM = LL * LL, R = 2 * sym_nmax(n_max);
  // value(row o, member k) of one group, appended in the group's layout
  auto group = [&](auto&& value) {
    auto put = [&](int o, int k) {
      const std::pair<int, double> e = value(o, k);
      s.v.push_back(e.first < 0 ? -1 : 2 * e.first + (o & 1));
      s.m.push_back(e.second);
    };
    if (width == 1) {
      for (int o = 0; o < R; ++o) put(o, 0);
      return;
    }
    for (int k = 0; k < 4; ++k)
      for (int o = 0; o < 16; ++o) put(o, k);
    for (int b = 16; b < R; b += 4)
      for (int k = 0; k < 4; ++k)
        for (int o = b; o < b + 4; ++o) put(o, k);
  };
  for (int l2 = 0; l2 < LL; ++l2)
    for (int l1 = 0; l1 <= l2; ++l1) {
      const int t = l2 * (l2 + 1) / 2 + l1;
      std::vector<std::pair<int, int>> nn;
      for (int n2 = 0; n2 < n_max; ++n2)
        for (int n1 = l1 == l2 ? n2 : 0; n1 < n_max; ++n1) nn.push_back({n1, n2});
      const int ng = ((int)nn.size() + width - 1) / width;
      s.off[kSymPairs + t] = (int)s.pairs.size();
      s.off[kSymNg + t] = ng;
      for (int p = 0; p < ng * width; ++p) {
        const auto q = p < (int)nn.size() ? nn[p] : std::make_pair(0, 0);
        s.pairs.push_back((q.first * LM + l1 * l1) | ((q.second * LM + l2 * l2) << 16));
      }
      for (int L = 0; L < LL; ++L) {
        if (!coupled(l1, l2, L)) continue;
        s.off[t * 5 + L] = (int)s.v.size();
        for (int g = 0; g < ng; ++g)
          group([&](int o, int k) -> std::pair<int, double> {
            const int p = g * width + k, n3 = o >> 1;
            if (p >= (int)nn.size() || n3 >= n_max) return {-1, 0.0};
            const int r = n3 * LL + L;
            std::array<int, 3> q = {r, nn[p].first * LL + l1, nn[p].second * LL + l2};
            const int times = 1 + (q[1] == r) + (q[2] == r);
            std::sort(q.begin(), q.end());
            return {c.index3[(q[0] * P + q[1]) * P + q[2]], times * kSymScale[l1][l2][L]};
          });
      }
    }
  for (int L = 0; L < LL; ++L) {
    s.off[kSymB2 + L] = (int)s.v.size();
    for (int g = 0; g * width < n_max; ++g)
      group([&](int o, int k) -> std::pair<int, double> {
        const int n = g * width + k, n3 = o >> 1;
        if (n >= n_max || n3 >= n_max) return {-1, 0.0};
        const int a = std::min(n, n3), b = std::max(n, n3);
        // second-order functions follow the n_max first-order ones in the order (n1, n2, l)
        const int v = n_max + LL * (a * n_max - a * (a - 1) / 2 + b - a) + L;
        return {v, a == b ? 2.0 : 1.0};
      });
  }
  // the kernels read up to two groups ahead
  for (int k = 0; k < 2 * width * R; ++k) {
    s.v.push_back(-1);
    s.m.push_back(0.0);
  }
  for (int k = 0; k < 3 * width; ++k) s.pairs.push_back(0);
  return s;
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

template <class T>
static void fill_reals(std::vector<T>& out, const apx_ace_model* m, const Catalogue& c, const double* c1,
                       const double* c2, size_t* offs) {
  const int LL = m->l_max + 1, nm = m->n_max;
  // order: Wp, (c1, c2) per triple + one padding pair, b1_c1, b1_c2, b2_c1, b2_c2
  out.clear();
  offs[0] = out.size();
  for (int l = 0; l < LL; ++l) {
    const double nl = std::sqrt((2.0 * l + 1.0) / (4.0 * M_PI));
    for (int n = 0; n < nm; ++n)
      for (int k = 0; k < nm; ++k) out.push_back((T)(m->W[((size_t)l * nm + n) * nm + k] * nl / m->s_a));
  }
  while (out.size() % 4) out.push_back((T)0);
  // the triples' coefficients with kTcPad zero pairs on either side: a kernel reads the
  // n_max coefficients around a run at once, whatever part of them the run uses
  for (int k = 0; k < 2 * kTcPad; ++k) out.push_back((T)0);
  offs[1] = out.size();
  for (int v : c.t_v) {
    out.push_back((T)c1[v]);
    out.push_back((T)c2[v]);
  }
  for (int k = 0; k < 2 * kTcPad; ++k) out.push_back((T)0);
  offs[2] = out.size();
  offs[3] = out.size();
  for (int v : c.b1_v) out.push_back((T)c1[v]);
  offs[4] = out.size();
  for (int v : c.b1_v) out.push_back((T)c2[v]);
  offs[5] = out.size();
  for (int v : c.b2_v) out.push_back((T)c1[v]);
  offs[6] = out.size();
  for (int v : c.b2_v) out.push_back((T)c2[v]);
  offs[7] = out.size();
}

// Coefficient rows of the symmetric product kernels, then the first-order pairs [n_max][2].
template <class T>
static void fill_sym(std::vector<T>& out, const std::vector<int>& v, const std::vector<double>& mul, int n_max,
                     const double* c1, const double* c2) {
  out.resize(v.size() + 2 * (size_t)n_max);
  for (size_t k = 0; k < v.size(); ++k)
    out[k] = v[k] < 0 ? T(0) : (T)(mul[k] * (v[k] & 1 ? c2 : c1)[v[k] >> 1]);
  for (int n = 0; n < n_max; ++n) {
    out[v.size() + 2 * n] = (T)c1[n];
    out[v.size() + 2 * n + 1] = (T)c2[n];
  }
}

template <class T>
static hipError_t upload(DevBuf& buf, const std::vector<T>& h) {
  hipError_t e = buf.ensure(h.size() * sizeof(T));
  return e == hipSuccess ? hipMemcpy(buf.p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) : e;
}

// Uploads one precision's tables of the symmetric product kernels.
template <class T>
static apx_status sym_upload(apx_ctx* ctx, const Catalogue& c, const apx_ace_model* m, int width, const T* Wp,
                             const double* c1, const double* c2, std::vector<int>& v, std::vector<double>& mul,
                             DevBuf& bi, DevBuf& br, SymTables<T>& t) {
  SymHost s = build_sym(c, m->n_max, m->l_max, width);
  std::vector<int> ints = s.off;
  ints.insert(ints.end(), s.pairs.begin(), s.pairs.end());
  std::vector<T> reals;
  fill_sym(reals, s.v, s.m, m->n_max, c1, c2);
  if (upload(bi, ints) != hipSuccess || upload(br, reals) != hipSuccess)
    return fail(ctx, APX_ENOMEM, "ACE table allocation failed");
  t.Wp = Wp;
  t.coef = br.template as<T>();
  t.b1 = t.coef + s.v.size();
  t.off = bi.as<int>();
  t.pairs = t.off + kSymOff;
  v = std::move(s.v);
  mul = std::move(s.m);
  return APX_OK;
}

template <class T>
static void set_tables(AceTables<T>& t, const T* base, const size_t* offs, const int* ib, const size_t* ioffs) {
  t.Wp = base + offs[0];
  t.tc = reinterpret_cast<const Coef2<T>*>(base + offs[1]);
  t.b1_c1 = base + offs[3];
  t.b1_c2 = base + offs[4];
  t.b2_c1 = base + offs[5];
  t.b2_c2 = base + offs[6];
  t.pairs = ib + ioffs[0];
  t.t_v = ib + ioffs[1];
  t.b1_off = ib + ioffs[2];
  t.b1_v = ib + ioffs[3];
  t.b2_off = ib + ioffs[4];
  t.b2_v = ib + ioffs[5];
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
  Catalogue c;
  try {
    c = build_catalogue(d->n_max, d->l_max);
  } catch (...) {
    return fail(ctx, APX_EINVAL, "inconsistent coupling catalogue");
  }
  apx_ace_model* m = new apx_ace_model();
  m->device = ctx->device;
  m->n_max = d->n_max;
  m->l_max = d->l_max;
  m->na = d->n_max * (d->l_max + 1) * (d->l_max + 1);
  m->n_basis = c.n_basis;
  m->npairs = (int)(c.pairs.size() / kPairRec);
  m->ntrip = c.ntrip;
  m->nb1 = (int)c.b1_v.size();
  m->nb2 = (int)c.b2_v.size();
  m->coupling_terms = c.coupling_terms;
  m->triple_width = c.triple_width;
  m->r_cut = d->r_cut;
  m->h = d->h;
  m->s_a = d->s_a;
  m->eps = d->eps;
  m->anchored = d->anchored ? 1 : 0;
  m->anchor = d->anchor;
  m->W.assign(d->W, d->W + (size_t)(d->l_max + 1) * d->n_max * d->n_max);
  m->t_v = c.t_v;
  m->b1_v = c.b1_v;
  m->b2_v = c.b2_v;
  // integer tables
  std::vector<int> ib;
  size_t ioffs[6];
  const std::vector<int>* parts[6] = {&c.pairs, &c.t_v, &c.b1_off, &c.b1_v, &c.b2_off, &c.b2_v};
  for (int q = 0; q < 6; ++q) {
    ioffs[q] = ib.size();
    ib.insert(ib.end(), parts[q]->begin(), parts[q]->end());
  }
  std::vector<double> r64;
  std::vector<float> r32;
  size_t o64[8], o32[8];
  fill_reals(r64, m, c, d->c1, d->c2, o64);
  fill_reals(r32, m, c, d->c1, d->c2, o32);
  if (m->ints.ensure(ib.size() * sizeof(int)) != hipSuccess || m->reals64.ensure(r64.size() * sizeof(double)) != hipSuccess ||
      m->reals32.ensure(r32.size() * sizeof(float)) != hipSuccess) {
    delete m;
    return fail(ctx, APX_ENOMEM, "ACE table allocation failed");
  }
  hipError_t e1 = hipMemcpy(m->ints.p, ib.data(), ib.size() * sizeof(int), hipMemcpyHostToDevice);
  hipError_t e2 = hipMemcpy(m->reals64.p, r64.data(), r64.size() * sizeof(double), hipMemcpyHostToDevice);
  hipError_t e3 = hipMemcpy(m->reals32.p, r32.data(), r32.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e1 != hipSuccess || e2 != hipSuccess || e3 != hipSuccess) {
    delete m;
    return fail(ctx, APX_EDEVICE, "ACE table upload failed");
  }
  set_tables(m->t64, m->reals64.as<double>(), o64, m->ints.as<int>(), ioffs);
  set_tables(m->t32, m->reals32.as<float>(), o32, m->ints.as<int>(), ioffs);
  m->t64.npairs = m->npairs;
  m->t32.npairs = m->npairs;
  apx_status st = sym_upload<float>(ctx, c, m, 1, m->t32.Wp, d->c1, d->c2, m->sym_v32, m->sym_m32, m->sym_i32,
                                    m->sym_r32, m->s32);
  if (st == APX_OK)
    st = sym_upload<double>(ctx, c, m, 4, m->t64.Wp, d->c1, d->c2, m->sym_v64, m->sym_m64, m->sym_i64, m->sym_r64,
                            m->s64);
  if (st != APX_OK) {
    delete m;
    return st;
  }
  *out = m;
  return APX_OK;
}

extern "C" apx_status apx_ace_model_set_coeffs(apx_ctx* ctx, apx_ace_model* m, const double* c1, const double* c2) {
  if (!ctx) return APX_EINVAL;
  if (!m || !c1 || !c2) return fail(ctx, APX_EINVAL, "model, c1 and c2 are required");
  Catalogue c;
  c.t_v = m->t_v;
  c.b1_v = m->b1_v;
  c.b2_v = m->b2_v;
  std::vector<double> r64;
  std::vector<float> r32;
  size_t o64[8], o32[8];
  fill_reals(r64, m, c, c1, c2, o64);
  fill_reals(r32, m, c, c1, c2, o32);
  if (r64.size() * sizeof(double) > m->reals64.bytes || r32.size() * sizeof(float) > m->reals32.bytes)
    return fail(ctx, APX_EINVAL, "coefficient table size changed");
  APX_HIP(ctx, hipStreamSynchronize(ctx->stream));
  APX_HIP(ctx, hipMemcpy(m->reals64.p, r64.data(), r64.size() * sizeof(double), hipMemcpyHostToDevice));
  APX_HIP(ctx, hipMemcpy(m->reals32.p, r32.data(), r32.size() * sizeof(float), hipMemcpyHostToDevice));
  std::vector<float> y32;
  std::vector<double> y64;
  fill_sym(y32, m->sym_v32, m->sym_m32, m->n_max, c1, c2);
  fill_sym(y64, m->sym_v64, m->sym_m64, m->n_max, c1, c2);
  APX_HIP(ctx, hipMemcpy(m->sym_r32.p, y32.data(), y32.size() * sizeof(float), hipMemcpyHostToDevice));
  APX_HIP(ctx, hipMemcpy(m->sym_r64.p, y64.data(), y64.size() * sizeof(double), hipMemcpyHostToDevice));
  return APX_OK;
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
