#!/usr/bin/env python3
"""Generate hw_coeffs2d.h: the two-dimensional reconstruction operators of Step 5.1
(Zhao & Qiu, arXiv 2002.08816, Section 2.2) as straight-line device code.

Derivation (exact, sympy), in reference coordinates (xi, eta) in [-1/2, 1/2]^2 of the
target cell, neighbours at integer offsets (labels 1..9 of Figure 1):

* p0 (quartic, 15 monomials): the nine averages and the two first moments of the target
  cell are met exactly; the first moments of the four edge neighbours (labels 2, 4, 6, 8)
  in the unweighted least-squares sense.  Solved in null-space form: a particular
  solution of the exact rows plus the null-space component minimising the residual.
* p1..p4 (quadratics, 6 monomials): the averages of the 2x2 sub-stencils of Figure 2 and
  the two first moments of the target cell, interpolated.
* smoothness indicators (eq. 2dGHYZ, square cells): Gram matrices of the derivative
  integrals over the target cell, each multi-index counted once.

Emitted code
* lin2d_fold, lin2d_inner, lin2d_xparts_ng<NG> / lin2d_xface_ng<NG>: the linear path (Steps
  5.2 and 5.3) for one field.  lin2d_fold folds the stencil data into the four
  reflection-parity classes of the 3x3 stencil (even/odd under xi -> -xi and under eta ->
  -eta); since p0 commutes with both reflections, each parity part of a point value depends
  only on the folds of the same class, and the mirror images of a point follow by a
  butterfly: about a quarter of the dense map's multiplies.  lin2d_inner: values of p0 at
  the 3 x 3 interior Gauss points; lin2d_xparts: the parity parts of the left and right
  edges' Gauss points, lin2d_xface: one of the two edges from them.  p0 also commutes with
  the exchange of x and y: the bottom and top edges are the x edges of lin2d_transpose.
* p0_coeffs (from the folds) / pq_coeffs<n>: monomial coefficients of p0 and p_n, for the
  HWENO path (p0's edge values there are those of the linear path).
* beta_p0 / beta_pq: the smoothness indicators as sparse quadratic forms.
* edge monomial tables for evaluating the candidates at the edge Gauss points.

Input order of the 19 stencil values ("in"):
  0..8   averages of labels 1..9
  9..13  x first moments of labels 2, 4, 5, 6, 8
  14..18 y first moments of labels 2, 4, 5, 6, 8
Edge point order: left (-1/2, e_k), right (1/2, e_k), bottom (e_k, -1/2), top (e_k, 1/2)
with e_k the ascending Gauss nodes; interior (g_k, g_l) at index 3 l + k (3-point Gauss).

Run: python gen_coeffs2d.py > hw_coeffs2d.h
"""
import sys

import sympy as sp

HALF = sp.Rational(1, 2)


def cell_int(m, j):
    x = sp.Symbol("x")
    return sp.integrate(x ** m, (x, j - HALF, j + HALF))


def cell_int_w(m, j):
    x = sp.Symbol("x")
    return sp.integrate(x ** m * (x - j), (x, j - HALF, j + HALF))


def offset(label):
    return (label - 1) % 3 - 1, (label - 1) // 3 - 1


def monos(r):
    return [(p, t - p) for t in range(r + 1) for p in range(t, -1, -1)]


CROSS = (2, 4, 5, 6, 8)
IN_NAMES = ([f"u{k}" for k in range(1, 10)] + [f"v{k}" for k in CROSS] + [f"w{k}" for k in CROSS])


def in_index(kind, label):
    if kind == "u":
        return label - 1
    base = 9 if kind == "v" else 14
    return base + CROSS.index(label)


def moment_row(kind, label, mons):
    a, b = offset(label)
    row = []
    for p, q in mons:
        if kind == "u":
            row.append(cell_int(p, a) * cell_int(q, b))
        elif kind == "v":
            row.append(cell_int_w(p, a) * cell_int(q, b))
        else:
            row.append(cell_int(p, a) * cell_int_w(q, b))
    return row


def derive_p0():
    mons = monos(4)
    ex = [("u", k) for k in range(1, 10)] + [("v", 5), ("w", 5)]
    ls = [(kd, k) for k in (2, 4, 6, 8) for kd in ("v", "w")]
    E = sp.Matrix([moment_row(kd, k, mons) for kd, k in ex])
    B = sp.Matrix([moment_row(kd, k, mons) for kd, k in ls])
    # selector matrices from the 19 inputs
    SE = sp.zeros(len(ex), 19)
    for i, (kd, k) in enumerate(ex):
        SE[i, in_index(kd, k)] = 1
    SB = sp.zeros(len(ls), 19)
    for i, (kd, k) in enumerate(ls):
        SB[i, in_index(kd, k)] = 1
    # particular solution: minimum-norm-free choice via pivot columns of E
    N = E.nullspace()
    assert len(N) == 4
    N = sp.Matrix.hstack(*N)
    Ep = E.pinv()
    # c = Ep SE d + N z ;  minimise |B c - SB d|^2 over z
    BN = B * N
    z_map = -(BN.T * BN).inv() * BN.T * (B * Ep * SE - SB)
    C = Ep * SE + N * z_map
    C = C.applyfunc(sp.simplify)
    assert (E * C - SE).applyfunc(sp.simplify) == sp.zeros(len(ex), 19)
    return mons, C


SUB = {1: (1, 2, 4, 5), 2: (2, 3, 5, 6), 3: (4, 5, 7, 8), 4: (5, 6, 8, 9)}


def derive_pq(n):
    mons = monos(2)
    conds = [("u", k) for k in SUB[n]] + [("v", 5), ("w", 5)]
    A = sp.Matrix([moment_row(kd, k, mons) for kd, k in conds])
    S = sp.zeros(6, 19)
    for i, (kd, k) in enumerate(conds):
        S[i, in_index(kd, k)] = 1
    return mons, A.inv() * S


def int_sym(a):
    """Integral of x^a over [-1/2, 1/2]."""
    return sp.Integer(0) if a % 2 else 2 * HALF ** (a + 1) / (a + 1)


def dmono(p, l):
    """(coefficient, exponent) of d^l/dx^l x^p."""
    if l > p:
        return sp.Integer(0), 0
    c = sp.Integer(1)
    for t in range(l):
        c *= (p - t)
    return c, p - l


def gram(mons, r):
    G = sp.zeros(len(mons), len(mons))
    for L in range(1, r + 1):
        for l1 in range(L + 1):
            l2 = L - l1
            for s, (p, q) in enumerate(mons):
                cp, ep = dmono(p, l1)
                cq, eq = dmono(q, l2)
                if cp == 0 or cq == 0:
                    continue
                for t, (p2, q2) in enumerate(mons):
                    cp2, ep2 = dmono(p2, l1)
                    cq2, eq2 = dmono(q2, l2)
                    if cp2 == 0 or cq2 == 0:
                        continue
                    G[s, t] += cp * cq * cp2 * cq2 * int_sym(ep + ep2) * int_sym(eq + eq2)
    return G


def gauss_nodes(ng):
    if ng == 2:
        return [-sp.sqrt(3) / 6, sp.sqrt(3) / 6]
    return [-sp.sqrt(15) / 10, sp.Integer(0), sp.sqrt(15) / 10]


def cnum(v):
    f = float(sp.N(v, 40))
    return repr(f)


def emit_sum(terms, indent="  "):
    """terms: list of (coef, expr_string); returns an expression using fma chains."""
    terms = [(c, e) for c, e in terms if c != 0]
    if not terms:
        return "0.0"
    c0, e0 = terms[0]
    acc = e0 if c0 == 1 else f"{cnum(c0)} * {e0}"
    for c, e in terms[1:]:
        acc = f"fma({cnum(c)}, {e}, {acc})"
    return acc


# ------------------------------------------------------------------ parity folding
# class -> list of (name, {input_index: sign})
def folded_inputs():
    u = lambda k: in_index("u", k)
    v = lambda k: in_index("v", k)
    w = lambda k: in_index("w", k)
    return {
        "ee": [{u(5): 1}, {u(4): 1, u(6): 1}, {u(2): 1, u(8): 1}, {u(1): 1, u(3): 1, u(7): 1, u(9): 1},
               {v(6): 1, v(4): -1}, {w(8): 1, w(2): -1}],
        # (the sums v4 + v6, v2 + v8, w2 + w8, w4 + w6 enter no value of p0)
        "oe": [{u(6): 1, u(4): -1}, {u(3): 1, u(9): 1, u(1): -1, u(7): -1}, {v(5): 1}],
        "eo": [{u(8): 1, u(2): -1}, {u(7): 1, u(9): 1, u(1): -1, u(3): -1}, {w(5): 1}],
        "oo": [{u(1): 1, u(9): 1, u(3): -1, u(7): -1}, {v(8): 1, v(2): -1}, {w(6): 1, w(4): -1}],
    }


def parity_part_rows(row, cls_inputs):
    """Express the parity part of the linear functional `row` (over the 19 inputs) in
    terms of the folded inputs of one class.  The folded inputs of a class are mutually
    orthogonal sign patterns over disjoint supports, so the coefficient of folded input f
    is row . f / |f|^2."""
    out = []
    for f in cls_inputs:
        num = sum(row[i] * s for i, s in f.items())
        den = sum(s * s for s in f.values())
        out.append(sp.simplify(num / den))
    return out


def main():
    mons4, C0 = derive_p0()
    pq = {n: derive_pq(n) for n in (1, 2, 3, 4)}
    mons2 = pq[1][0]
    G4 = gram(mons4, 4)
    G2 = gram(mons2, 2)
    classes = folded_inputs()
    cls_sign = {"ee": (1, 1), "oe": (-1, 1), "eo": (1, -1), "oo": (-1, -1)}

    def value_row(C, mons, x, y):
        return [sp.simplify(sum(C[s, k] * x ** p * y ** q for s, (p, q) in enumerate(mons)))
                for k in range(19)]

    out = []
    w = out.append
    w("// Generated by gen_coeffs2d.py -- do not edit.")
    w("// Two-dimensional reconstruction operators of Step 5.1 (Section 2.2): the least-squares")
    w("// quartic p0 (Figure 1 stencil), the quadratics p1..p4 (Figure 2 sub-stencils) and the")
    w("// smoothness indicators of eq. 2dGHYZ for square cells.")
    w("#pragma once")
    w("namespace hw2 {")
    w("")
    w("// ---------------------------------------------------------------- linear path")
    w("// One field: reflection-parity folding of the 19 inputs, then the point values of p0 from the")
    w("// folds, with a butterfly per orbit of mirror-image points.")
    names = [f"{cls}{i}" for cls, fl in classes.items() for i in range(len(fl))]
    slot = {nm: f"f[{k}]" for k, nm in enumerate(names)}

    # the folding, with the four corners through their diagonal sums and differences (the
    # mixed part oo0 from differences along the edges, which are exact between close values).
    # On the transposed stencil every operation is the same up to commuting operands, except
    # oo0's: a reader of the transposed stencil takes lin2d_fold_oo0_T for it, and then its
    # folds equal lin2d_transpose of the untransposed folds to the bit
    fold = {
        "ee0": "in[4]", "ee1": "in[3] + in[5]", "ee2": "in[1] + in[7]", "ee3": "s0 + s1",
        "ee4": "in[12] - in[10]", "ee5": "in[18] - in[14]",
        "oe0": "in[5] - in[3]", "oe1": "d0 + d1", "oe2": "in[11]",
        "eo0": "in[7] - in[1]", "eo1": "d0 - d1", "eo2": "in[16]",
        "oo0": "(in[8] - in[2]) - (in[6] - in[0])", "oo1": "in[13] - in[9]", "oo2": "in[17] - in[15]"}
    corner = {"s0": "in[0] + in[8]", "s1": "in[2] + in[6]", "d0": "in[8] - in[0]", "d1": "in[2] - in[6]"}
    sym = [sp.Symbol(f"i{k}") for k in range(19)]
    def value(expr):
        import re as _re
        return sp.sympify(eval(_re.sub(r"in\[(\d+)\]", r"sym[\1]", expr),
                               {"sym": sym, **{k: value(v) for k, v in corner.items() if k in expr}}))
    for cls, fl in classes.items():
        for i, f in enumerate(fl):
            assert sp.expand(value(fold[f"{cls}{i}"]) - sum(sg * sym[k] for k, sg in f.items())) == 0
    w(f"constexpr int NFOLD = {len(names)};")
    w("__device__ __forceinline__ void lin2d_fold(const double* in, double* f) {")
    for nm, expr in corner.items():
        w(f"  const double {nm} = {expr};")
    for nm in names:
        w(f"  {slot[nm]} = {fold[nm]};")
    w("}")
    w("__device__ __forceinline__ double lin2d_fold_oo0_T(const double* in) { return (in[8] - in[6]) - (in[2] - in[0]); }")
    w("// the fold of the stencil with x and y exchanged")
    w("__device__ __forceinline__ void lin2d_transpose(const double* f, double* g) {")
    swap = {"ee1": "ee2", "ee4": "ee5", "oe0": "eo0", "oe1": "eo1", "oe2": "eo2", "oo1": "oo2"}
    swap.update({v: k for k, v in swap.items()})
    for nm in names:
        w(f"  {slot[nm].replace('f', 'g')} = {slot[swap.get(nm, nm)]};")
    w("}")
    w("")

    def emit_points(fname, pts_and_targets, orbits):
        """One straight-line function of the folded inputs: the parity parts at the
        representative points, and the requested point values by a butterfly over each
        orbit of mirror-image points (orbits: four targets (-,-), (+,-), (-,+), (+,+) of
        one representative each)."""
        w(f"__device__ __forceinline__ void {fname} {{")
        reps.clear()
        at = dict(pts_and_targets)
        done = set()
        for n, orb in enumerate(orbits):
            x, y = at[orb[3]]
            p = {cls: part(cls, x, y) for cls in cls_sign}
            w(f"  const double p{n} = {p['ee']} + {p['oo']}, m{n} = {p['ee']} - {p['oo']};")
            w(f"  const double q{n} = {p['oe']} + {p['eo']}, r{n} = {p['oe']} - {p['eo']};")
            for t, e in zip(orb, (f"p{n} - q{n}", f"m{n} + r{n}", f"m{n} - r{n}", f"p{n} + q{n}")):
                point(*at[t])   # (its self-check)
                w(f"  {t} = {e};")
                done.add(t)
        for target, (x, y) in pts_and_targets:
            if target not in done:
                w(f"  {target} = {point(x, y)};")
        w("}")
        w("")

    def emit_face(ng):
        """The x faces' points: parity parts at (1/2, |e_k|), then one face from its side's
        sign (side = -1 low, +1 high; its products are exact)."""
        nodes = gauss_nodes(ng)
        reps.clear()
        w(f"// parity parts of the x-face points ({'ee oe eo oo at the outer pair' + (', ee oe at the middle' if ng == 3 else '')})")
        w(f"__device__ __forceinline__ void lin2d_xparts_ng{ng}(const double* f, double* p) {{")
        e = nodes[-1]
        for k, cls in enumerate(cls_sign):
            w(f"  p[{k}] = {part_expr(cls, HALF, e)};")
        if ng == 3:
            w(f"  p[4] = {part_expr('ee', HALF, sp.Integer(0))};")
            w(f"  p[5] = {part_expr('oe', HALF, sp.Integer(0))};")
        w("}")
        w(f"__device__ __forceinline__ void lin2d_xface_ng{ng}(const double* p, double side, double* v) {{")
        w("  v[0] = fma(side, fma(-side, p[2], p[1]), fma(-side, p[3], p[0]));")
        if ng == 3:
            w("  v[1] = fma(side, p[5], p[4]);")
        w(f"  v[{ng - 1}] = fma(side, fma(side, p[2], p[1]), fma(side, p[3], p[0]));")
        w("}")
        w("")
        for x in (-HALF, HALF):
            for y in nodes:
                point(x, y, emit=False)

    reps = {}

    def part_expr(cls, x, y):
        row = value_row(C0, mons4, x, y)
        coefs = parity_part_rows(row, classes[cls])
        return emit_sum([(c, slot[f"{cls}{i}"]) for i, c in enumerate(coefs)])

    def part(cls, x, y, emit=True):
        key = (cls, x, y)
        if not emit or key in reps:
            return reps.get(key, "")
        name = f"P{cls}_{len(reps)}"
        w(f"  const double {name} = {part_expr(cls, x, y)};")
        reps[key] = name
        return name

    def point(x, y, emit=True):
        """expression for p0 at (x, y) from the parity parts at (|x|, |y|)."""
        ax, ay = abs(x), abs(y)
        sx = -1 if x < 0 else 1
        sy = -1 if y < 0 else 1
        terms = []
        for cls, (px, py) in cls_sign.items():
            if (px == -1 and ax == 0) or (py == -1 and ay == 0):
                continue   # odd part vanishes on the mirror line
            sgn = (sx if px == -1 else 1) * (sy if py == -1 else 1)
            terms.append((sgn, part(cls, ax, ay, emit)))
        # self-check: the parity parts add up to the dense row of p0 at (x, y)
        dense = value_row(C0, mons4, x, y)
        back = [sp.Integer(0)] * 19
        for cls, (px, py) in cls_sign.items():
            if (px == -1 and ax == 0) or (py == -1 and ay == 0):
                continue
            sgn = (sx if px == -1 else 1) * (sy if py == -1 else 1)
            coefs = parity_part_rows(value_row(C0, mons4, ax, ay), classes[cls])
            for f, c in zip(classes[cls], coefs):
                for idx, sg in f.items():
                    back[idx] += sgn * c * sg
        assert all(sp.simplify(a - b) == 0 for a, b in zip(dense, back)), (x, y)
        expr = ""
        for sgn, nm in terms:
            expr += (" + " if sgn > 0 else " - ") + nm
        expr = expr.strip()
        if expr.startswith("+ "):
            expr = expr[2:]
        elif expr.startswith("- "):
            expr = "-" + expr[2:]
        return expr

    inner_nodes = gauss_nodes(3)
    emit_points("lin2d_inner(const double* f, double* inner)",
                [(f"inner[{3 * l + k}]", (a, b)) for l, b in enumerate(inner_nodes)
                 for k, a in enumerate(inner_nodes)],
                [("inner[0]", "inner[2]", "inner[6]", "inner[8]")])
    for ng in (2, 3):
        emit_face(ng)

    # ---------------------------------------------------------------- HWENO path
    w("// ---------------------------------------------------------------- HWENO path")
    w("// Monomial order (p, q) for xi^p eta^q: by total degree, then descending p.")
    # a monomial coefficient of p0 depends on the folds of its own parity only
    order = {"ee": (0, 0), "oe": (1, 0), "eo": (0, 1), "oo": (1, 1)}
    fold_rows = []
    for s, (p, q) in enumerate(mons4):
        cls = next(k for k, v in order.items() if v == (p % 2, q % 2))
        row = [C0[s, k] for k in range(19)]
        coefs = parity_part_rows(row, classes[cls])
        back = [sp.Integer(0)] * 19
        for f, c in zip(classes[cls], coefs):
            for idx, sg in f.items():
                back[idx] += c * sg
        assert all(sp.simplify(a - b) == 0 for a, b in zip(row, back)), s
        fold_rows.append([(c, slot[f"{cls}{i}"]) for i, c in enumerate(coefs) if c != 0])
    w("// (p0 from the folded inputs)")
    w("__device__ __forceinline__ void p0_coeffs(const double* f, double* c) {")
    for s in range(15):
        w(f"  c[{s}] = {emit_sum(fold_rows[s])};")
    w("}")
    for n in (1, 2, 3, 4):
        mons, C = pq[n]
        w(f"__device__ __forceinline__ void p{n}_coeffs(const double* in, double* c) {{")
        for s in range(6):
            w(f"  c[{s}] = {emit_sum([(C[s, k], f'in[{k}]') for k in range(19)])};")
        w("}")

    def emit_quad(G, n, name):
        w(f"__device__ __forceinline__ double {name}(const double* c) {{")
        w("  double b = 0.0;")
        for s in range(n):
            terms = []
            if G[s, s] != 0:
                terms.append((G[s, s], f"c[{s}]"))
            for t in range(s + 1, n):
                if G[s, t] != 0:
                    terms.append((2 * G[s, t], f"c[{t}]"))
            if terms:
                w(f"  b = fma(c[{s}], {emit_sum(terms)}, b);")
        w("  return b;")
        w("}")

    emit_quad(G4, 15, "beta_p0")
    emit_quad(G2, 6, "beta_pq")
    for ng in (2, 3):
        nodes = gauss_nodes(ng)
        pts = ([(-HALF, e) for e in nodes] + [(HALF, e) for e in nodes]
               + [(e, -HALF) for e in nodes] + [(e, HALF) for e in nodes])
        w(f"// value of a quadratic (6 coefficients) at edge point i")
        w(f"__device__ __forceinline__ double edge_quad_ng{ng}(const double* c, int i) {{")
        w("  switch (i) {")
        for i, (x, y) in enumerate(pts):
            w(f"  case {i}: return {emit_sum([(x ** p * y ** q, f'c[{s}]') for s, (p, q) in enumerate(mons2)])};")
        w("  }")
        w("  return 0.0;")
        w("}")
    # ---------------------------------------------------------------- adjoint pieces
    w("// ---------------------------------------------------------------- adjoint path")
    w("// Transposes (accumulating into fold cotangents fb, or db[19]) of the linear point maps, of the candidate")
    w("// coefficient maps and of the edge evaluations; gradients of the indicators.")

    def acc_T(pairs, indent="  "):
        """fold cotangents fb[j] += sum coef * expr, for (expr, [(coef, 'f[j]'), ...])."""
        by = {}
        for expr, row in pairs:
            for c, tgt in row:
                if c != 0:
                    by.setdefault(tgt, []).append((c, expr))
        for tgt in sorted(by, key=lambda t: int(t[2:-1])):
            acc = "fb" + tgt[1:]
            tgt_b = acc
            for c, e in by[tgt]:
                acc = f"fma({cnum(c)}, {e}, {acc})"
            w(f"{indent}{tgt_b} = {acc};")

    def part_row(cls, x, y):
        row = value_row(C0, mons4, x, y)
        return [(c, slot[f"{cls}{i}"]) for i, c in enumerate(parity_part_rows(row, classes[cls]))]

    w("// db[19] += the transpose of lin2d_fold applied to fb")
    w("__device__ __forceinline__ void lin2d_fold_T(const double* fb, double* db) {")
    corner_T = {0: "s0 - d0", 8: "s0 + d0", 2: "s1 + d1", 6: "s1 - d1"}
    fi = {nm: slot[nm].replace("f[", "fb[") for nm in names}
    w(f"  const double s0 = {fi['ee3']} + {fi['oo0']}, s1 = {fi['ee3']} - {fi['oo0']};")
    w(f"  const double d0 = {fi['oe1']} + {fi['eo1']}, d1 = {fi['oe1']} - {fi['eo1']};")
    for k, e in corner_T.items():
        w(f"  db[{k}] += {e};")
    plain = {}
    for cls, fl in classes.items():
        for i, f in enumerate(fl):
            nm = f"{cls}{i}"
            if nm in ("ee3", "oo0", "oe1", "eo1"):
                continue
            for idx, sg in f.items():
                plain.setdefault(idx, []).append((sg, fi[nm]))
    for idx in sorted(plain):
        expr = " ".join(("+ " if sg > 0 else "- ") + e for sg, e in plain[idx])
        expr = expr[2:] if expr.startswith("+ ") else "-" + expr[2:]
        w(f"  db[{idx}] += {expr};")
    w("}")
    # self-check: the folds' transpose, corner by corner
    for k, want in ((0, (1, 1, -1, -1)), (8, (1, 1, 1, 1)), (2, (1, -1, 1, -1)), (6, (1, -1, -1, 1))):
        got = tuple(classes[c][i].get(k, 0) for c, i in (("ee", 3), ("oo", 0), ("oe", 1), ("eo", 1)))
        assert got == want, (k, got)
    w("")
    w("// fb += the transpose of lin2d_inner applied to ub[9]")
    w("__device__ __forceinline__ void lin2d_inner_T(const double* ub, double* fb) {")
    w("  const double pb = ub[0] + ub[8], qb = ub[8] - ub[0], mb = ub[2] + ub[6], rb = ub[2] - ub[6];")
    w("  const double ee0 = pb + mb, oo0 = pb - mb, oe0 = qb + rb, eo0 = qb - rb;")
    w("  const double ee1 = ub[1] + ub[7], eo1 = ub[7] - ub[1], ee2 = ub[3] + ub[5], oe2 = ub[5] - ub[3];")
    g, z = inner_nodes[-1], sp.Integer(0)
    acc_T([("ee0", part_row("ee", g, g)), ("oe0", part_row("oe", g, g)), ("eo0", part_row("eo", g, g)),
           ("oo0", part_row("oo", g, g)), ("ee1", part_row("ee", z, g)), ("eo1", part_row("eo", z, g)),
           ("ee2", part_row("ee", g, z)), ("oe2", part_row("oe", g, z)), ("ub[4]", part_row("ee", z, z))])
    w("}")
    w("")
    for ng in (2, 3):
        e = gauss_nodes(ng)[-1]
        w("// fb += the transpose of the x faces' values (low face lo, high face hi)")
        w(f"__device__ __forceinline__ void lin2d_xfaces_ng{ng}_T(const double* lo, const double* hi, double* fb) {{")
        L = ng - 1
        w(f"  const double a = lo[0] + hi[{L}], b = hi[{L}] - lo[0], c = lo[{L}] + hi[0], d = hi[0] - lo[{L}];")
        w("  const double p0 = a + c, p1 = b + d, p2 = b - d, p3 = a - c;")
        rows = [("p0", part_row("ee", HALF, e)), ("p1", part_row("oe", HALF, e)),
                ("p2", part_row("eo", HALF, e)), ("p3", part_row("oo", HALF, e))]
        if ng == 3:
            w("  const double p4 = lo[1] + hi[1], p5 = hi[1] - lo[1];")
            rows += [("p4", part_row("ee", HALF, z)), ("p5", part_row("oe", HALF, z))]
        acc_T(rows)
        w("}")
        w("")

    def emit_coef_T(fname, C, n):
        w(f"__device__ __forceinline__ void {fname}(const double* cb, double* db) {{")
        for j in range(19):
            terms = [(C[t, j], f"cb[{t}]") for t in range(n) if C[t, j] != 0]
            if not terms:
                continue
            acc = f"db[{j}]"
            for c, e in terms:
                acc = f"fma({cnum(c)}, {e}, {acc})"
            w(f"  db[{j}] = {acc};")
        w("}")

    w("// fb += the transpose of p0_coeffs applied to cb[15]")
    w("__device__ __forceinline__ void p0_coeffs_T(const double* cb, double* fb) {")
    acc_T([(f"cb[{t}]", fold_rows[t]) for t in range(15)])
    w("}")
    for n in (1, 2, 3, 4):
        emit_coef_T(f"p{n}_coeffs_T", pq[n][1], 6)

    def emit_grad(G, n, name):
        w(f"// gradient 2 G c of the quadratic form c^T G c")
        w(f"__device__ __forceinline__ void {name}(const double* c, double* g) {{")
        for t in range(n):
            terms = [(2 * G[t, u], f"c[{u}]") for u in range(n) if G[t, u] != 0]
            w(f"  g[{t}] = {emit_sum(terms)};")
        w("}")

    emit_grad(G4, 15, "beta_p0_grad")
    emit_grad(G2, 6, "beta_pq_grad")
    for ng in (2, 3):
        nodes = gauss_nodes(ng)
        pts = ([(-HALF, e) for e in nodes] + [(HALF, e) for e in nodes]
               + [(e, -HALF) for e in nodes] + [(e, HALF) for e in nodes])
        w(f"// transpose of edge_quad: cb[s] += mono_s(point i) * qb")
        w(f"__device__ __forceinline__ void edge_quad_ng{ng}_T(double qb, int i, double* cb) {{")
        w("  switch (i) {")
        for i, (x, y) in enumerate(pts):
            body = " ".join(f"cb[{t}] = fma({cnum(x ** p * y ** q)}, qb, cb[{t}]);"
                            for t, (p, q) in enumerate(mons2) if x ** p * y ** q != 0)
            w(f"  case {i}: {body} break;")
        w("  }")
        w("}")
    w("")
    w("}  // namespace hw2")
    sys.stdout.write("\n".join(out) + "\n")


if __name__ == "__main__":
    main()
