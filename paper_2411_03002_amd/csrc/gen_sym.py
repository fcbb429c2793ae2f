"""Generates ace_sym_gen.h: real-Gaunt coupling of two harmonic blocks, one component at a time.

For degrees l1 <= l2 and a component M the generated function forms, for every coupled degree
L <= l_max (l1 + l2 + L even, L >= |M|), the scaled product
    P[L] = (1 / s(l1, l2, L)) sum_{m1 m2} G(l1 l2 L; m1 m2 M) a[m1] b[m2]
with the real Gaunt coefficients of gen_coupling.py (m indices offset by l).  Products whose
coefficients agree up to a sign in every L are summed first (a product of real harmonics meets
M = |m1 + m2| and M = |m1 - m2| in two or four such products), and each sum enters the degrees
by one multiply-add.  The scale s(l1, l2, L), the coefficient most of these sums share, is
folded into the tabulated expansion coefficients (kSymScale), which saves their multiplication.
Run: python gen_sym.py (writes the header next to this file).
"""

from __future__ import annotations

import os
from collections import Counter

from gen_coupling import LMAX_ALL, gaunt_table


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
        "// Generated by gen_sym.py -- do not edit.  Real Gaunt coupling of two harmonic blocks",
        "// (degrees l1 <= l2), one component M at a time, scaled by 1 / kSymScale[l1][l2][L].",
        "#pragma once",
        "#include <hip/hip_runtime.h>",
        "namespace apx {",
        f"constexpr double kSymScale[{n}][{n}][{n}] = {{",
    ]
    for l1 in range(n):
        lines.append("    {" + ", ".join("{" + ", ".join(f"{x:.17g}" for x in scale[l1][l2]) + "}" for l2 in range(n)) + "},")
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
    with open(os.path.join(here, "ace_sym_gen.h"), "w") as fh:
        fh.write(emit())
