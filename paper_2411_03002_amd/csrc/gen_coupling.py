"""Generates ace_coupling_gen.h: unrolled real-Gaunt coupling code for the ACE kernels.

Real spherical harmonics are Y_lm = sqrt((2l+1)/(4 pi)) S_lm(u) with S_lm the real
regular solid harmonics built by the standard recursion
    S_00 = 1
    S_{l+1,l+1}    = c_l (x S_ll - (1-d_l0) y S_l,-l)
    S_{l+1,-(l+1)} = c_l (y S_ll + (1-d_l0) x S_l,-l),   c_l = sqrt(2^d_l0 (2l+1)/(2l+2))
    S_{l+1,m}      = ((2l+1) z S_lm - sqrt((l+m)(l-m)) r^2 S_{l-1,m}) / sqrt((l+m+1)(l-m+1))
(the same recursion the device code evaluates).  The Gaunt coefficient
G(l1 l2 L; m1 m2 M) = integral of Y_l1m1 Y_l2m2 Y_LM over the unit sphere is obtained
exactly by expanding the product into monomials and integrating each with
    integral x^a y^b z^c dOmega = 2 G((a+1)/2) G((b+1)/2) G((c+1)/2) / G((a+b+c+3)/2)
for even a, b, c (zero otherwise), G the gamma function.

For degrees l1 <= l2 and a component M the generated function forms, for every coupled degree
L <= l_max (l1 + l2 + L even, L >= |M|), the scaled product
    P[L] = (1 / s(l1, l2, L)) sum_{m1 m2} G(l1 l2 L; m1 m2 M) a[m1] b[m2]
(m indices offset by l).  Products whose coefficients agree up to a sign in every L are summed
first (a product of real harmonics meets M = |m1 + m2| and M = |m1 - m2| in two or four such
products), and each sum enters the degrees by one multiply-add.  The scale s(l1, l2, L), the
coefficient most of these sums share, is folded into the tabulated expansion coefficients
(kSymScale), which saves their multiplication.  kGauntTerms[l1][l2][L] counts the nonzero
coefficients.  Run: python gen_coupling.py (writes the header next to this file).
"""

from __future__ import annotations

import math
import os
from collections import Counter, defaultdict

LMAX_ALL = 4


def padd(p, q, s=1.0):
    out = defaultdict(float, p)
    for k, v in q.items():
        out[k] += s * v
    return dict(out)


def pmul_mono(p, mono, s=1.0):
    return {(a + mono[0], b + mono[1], c + mono[2]): s * v for (a, b, c), v in p.items()}


def pmul(p, q):
    out = defaultdict(float)
    for k1, v1 in p.items():
        for k2, v2 in q.items():
            out[(k1[0] + k2[0], k1[1] + k2[1], k1[2] + k2[2])] += v1 * v2
    return dict(out)


def solid_harmonics(lmax):
    S = {(0, 0): {(0, 0, 0): 1.0}}
    r2 = {(2, 0, 0): 1.0, (0, 2, 0): 1.0, (0, 0, 2): 1.0}
    for l in range(lmax):
        d0 = 1 if l == 0 else 0
        c = math.sqrt((2.0 if d0 else 1.0) * (2 * l + 1) / (2 * l + 2))
        sll, slml = S[(l, l)], S[(l, -l)]
        top = pmul_mono(sll, (1, 0, 0), c)
        bot = pmul_mono(sll, (0, 1, 0), c)
        if not d0:
            top = padd(top, pmul_mono(slml, (0, 1, 0), c), -1.0)
            bot = padd(bot, pmul_mono(slml, (1, 0, 0), c), 1.0)
        S[(l + 1, l + 1)] = top
        S[(l + 1, -(l + 1))] = bot
        for m in range(-l, l + 1):
            t = pmul_mono(S[(l, m)], (0, 0, 1), 2 * l + 1)
            if abs(m) <= l - 1:
                t = padd(t, pmul(r2, S[(l - 1, m)]), -math.sqrt((l + m) * (l - m)))
            den = math.sqrt((l + m + 1) * (l - m + 1))
            S[(l + 1, m)] = {k: v / den for k, v in t.items()}
    return S


def sphere_integral(a, b, c):
    if a % 2 or b % 2 or c % 2:
        return 0.0
    g = math.gamma
    return 2.0 * g((a + 1) / 2) * g((b + 1) / 2) * g((c + 1) / 2) / g((a + b + c + 3) / 2)


def gaunt_table(lmax):
    S = solid_harmonics(lmax)
    norm = [math.sqrt((2 * l + 1) / (4 * math.pi)) for l in range(lmax + 1)]
    G = {}
    for l1 in range(lmax + 1):
        for l2 in range(lmax + 1):
            for L in range(lmax + 1):
                if (l1 + l2 + L) % 2 or L < abs(l1 - l2) or L > l1 + l2:
                    continue
                for m1 in range(-l1, l1 + 1):
                    for m2 in range(-l2, l2 + 1):
                        p12 = pmul(S[(l1, m1)], S[(l2, m2)])
                        for M in range(-L, L + 1):
                            tot = 0.0
                            for k, v in pmul(p12, S[(L, M)]).items():
                                tot += v * sphere_integral(*k)
                            val = norm[l1] * norm[l2] * norm[L] * tot
                            if abs(val) > 1e-13:
                                G[(l1, m1, l2, m2, L, M)] = val
    return G


def sums_of(G, l1, l2, M):
    """[(signed products [(m1, m2, sign)], {L: coefficient})] of component M."""
    vec = {}
    for (a, m1, b, m2, L, MM), v in G.items():
        if a == l1 and b == l2 and MM == M:
            vec.setdefault((m1, m2), {})[L] = v
    out = []
    for (m1, m2), c in sorted(vec.items()):
        for prods, c0 in out:
            if c0.keys() != c.keys():
                continue
            for sg in (1, -1):
                if all(abs(c[L] - sg * c0[L]) < 1e-13 for L in c):
                    prods.append((m1, m2, sg))
                    break
            else:
                continue
            break
        else:
            out.append(([(m1, m2, 1)], c))
    return out


def emit():
    G = gaunt_table(LMAX_ALL)
    n = LMAX_ALL + 1
    scale = [[[1.0] * n for _ in range(n)] for _ in range(n)]
    for l1 in range(n):
        for l2 in range(l1, n):
            votes = {}
            for M in range(-LMAX_ALL, LMAX_ALL + 1):
                for prods, c in sums_of(G, l1, l2, M):
                    for L, v in c.items():
                        votes.setdefault(L, Counter())[round(abs(v), 12)] += 1
            for L, cnt in votes.items():
                scale[l1][l2][L] = max(cnt.items(), key=lambda kv: (kv[1], kv[0]))[0]
    # the exact value behind each rounded vote
    for l1 in range(n):
        for l2 in range(l1, n):
            for L in range(n):
                for (a, m1, b, m2, LL, M), v in G.items():
                    if a == l1 and b == l2 and LL == L and abs(abs(v) - scale[l1][l2][L]) < 1e-11:
                        scale[l1][l2][L] = abs(v)
                        break
    lines = [
        "// Generated by gen_coupling.py -- do not edit.  Real Gaunt coupling of two harmonic blocks",
        "// (degrees l1 <= l2), one component M at a time, scaled by 1 / kSymScale[l1][l2][L].",
        "#pragma once",
        "#include <hip/hip_runtime.h>",
        "namespace apx {",
        f"constexpr double kSymScale[{n}][{n}][{n}] = {{",
    ]
    for l1 in range(n):
        lines.append("    {" + ", ".join("{" + ", ".join(f"{x:.17g}" for x in scale[l1][l2]) + "}" for l2 in range(n)) + "},")
    lines.append("};")
    lines.append(f"constexpr int kGauntTerms[{n}][{n}][{n}] = {{")
    for l1 in range(n):
        cnt = [[sum(1 for k in G if k[0] == l1 and k[2] == l2 and k[4] == L) for L in range(n)] for l2 in range(n)]
        lines.append("    {" + ", ".join("{" + ", ".join(str(x) for x in c) + "}" for c in cnt) + "},")
    lines.append("};")
    lines.append("template <int L1, int L2, int M> struct SymP;")
    for l1 in range(n):
        for l2 in range(l1, n):
            for M in range(-LMAX_ALL, LMAX_ALL + 1):
                sums = sums_of(G, l1, l2, M)
                if not sums:
                    continue
                degs = sorted({L for _, c in sums for L in c})
                lines.append(f"template <> struct SymP<{l1}, {l2}, {M}> {{")
                lines.append("  template <int LMAX, class T>")
                lines.append("  __device__ __forceinline__ static void p(const T* a, const T* b, T* P) {")
                started = set()
                for prods, c in sums:
                    if min(c) > 3:
                        lines.append("    if constexpr (LMAX >= 4) {")
                        ind = "      "
                    else:
                        lines.append("    {")
                        ind = "      "
                    m1, m2, _ = prods[0]
                    lines.append(f"{ind}T t = a[{m1 + l1}] * b[{m2 + l2}];")
                    for m1, m2, sg in prods[1:]:
                        lines.append(f"{ind}t = fma({'-' if sg < 0 else ''}a[{m1 + l1}], b[{m2 + l2}], t);")
                    for L in sorted(c):
                        g = c[L] / scale[l1][l2][L]
                        unit = abs(abs(g) - 1.0) < 1e-12
                        guard = f"if constexpr (LMAX >= {L}) " if L > 3 and min(c) <= 3 else ""
                        if unit:
                            s = "" if g > 0 else "-"
                            rhs = f"{s}t" if L not in started else (f"P[{L}] {'+' if g > 0 else '-'} t")
                        else:
                            rhs = f"T({g:.17g}) * t" if L not in started else f"fma(T({g:.17g}), t, P[{L}])"
                        lines.append(f"{ind}{guard}P[{L}] = {rhs};")
                        started.add(L)
                    lines.append("    }")
                lines.append("  }")
                lines.append("};")
                assert started == set(degs)
    lines.append("}  // namespace apx")
    return "\n".join(lines) + "\n"


if __name__ == "__main__":
    here = os.path.dirname(os.path.abspath(__file__))
    with open(os.path.join(here, "ace_coupling_gen.h"), "w") as fh:
        fh.write(emit())
