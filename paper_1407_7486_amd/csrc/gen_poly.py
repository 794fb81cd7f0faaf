"""Generate wl_poly.h: polynomial branches of the field functions used by
the GPU kernels near the tube axis, where the closed forms cancel.

  q(v)  = (u tanh u - ln cosh u) / u^2 ,  v = u^2   (sech^2 tube: e A_phi/rho
          divided by eB0, as a function of v = rho^2/lambda^2)
  p(v)  = (1 - exp(-v)) / v                          (Gaussian tube: 2 e A_phi
          /(rho eB0))

and two elementary functions of the FP64 path:

  2^f on [-1/2, 1/2]                 (exp2 after the reduction t = n + f)
  ln(1 + E) / E on [0, 1/e]          (sech^2 tube away from the axis, where
                                      E = exp(-2u) <= 1/e)
  cos(2 pi f), sin(2 pi f) / f       (the per-loop cos(Phi) after the
    as functions of v = f^2,          reduction of Phi to the nearest
    |f| <= 1/8                        quarter turn)

and, for the FP64 segment walk's table-driven forms,

  2^(j/64), j = 0 .. 63, and          (exp2 after the reduction
  (2^f - 1)/f on [-1/128, 1/128]       t = n + j/64 + f)
  (c_j, 1 + log2 c_j), j = 0 .. 127,  (log2(1 + E) for E < 1/2: c_j the
  c_j = 1/(1 + (j + 1/2)/256), and     double nearest the reciprocal of the
  log2(1 + r)/r on [-1/511, 1/511]     middle of 1 + E's interval of width
                                       1/256, r = (1 + E) c_j - 1)

All are analytic on their intervals.  Coefficients come from Chebyshev
interpolation of the exact function (mpmath, 60 digits) on the stated
interval, converted to the monomial basis in v and rounded to the target
precision.  The script prints the achieved max relative error of Horner
evaluation in that precision.  Run: python gen_poly.py > wl_poly.h
"""
import mpmath as mp
import numpy as np

mp.mp.dps = 60


def q_exact(v):
    v = mp.mpf(v)
    if v == 0:
        return mp.mpf(1) / 2
    u = mp.sqrt(v)
    return (u * mp.tanh(u) - mp.log(mp.cosh(u))) / v


def p_exact(v):
    v = mp.mpf(v)
    if v == 0:
        return mp.mpf(1)
    return -mp.expm1(-v) / v


def exp2_exact(f):
    return mp.power(2, mp.mpf(f))


def log1p_exact(E):
    E = mp.mpf(E)
    if E == 0:
        return mp.mpf(1)
    return mp.log1p(E) / E


def cos2pi_exact(v):
    return mp.cos(2 * mp.pi * mp.sqrt(mp.mpf(v)))


def sin2pi_exact(v):
    v = mp.mpf(v)
    if v == 0:
        return 2 * mp.pi
    f = mp.sqrt(v)
    return mp.sin(2 * mp.pi * f) / f


def exp2m1_exact(f):
    f = mp.mpf(f)
    if f == 0:
        return mp.log(2)
    return mp.expm1(f * mp.log(2)) / f


def log2p1_exact(r):
    r = mp.mpf(r)
    if r == 0:
        return 1 / mp.log(2)
    return mp.log1p(r) / r / mp.log(2)


def emit_table(name, values, comment):
    print(f"/* {name}: {comment} */")
    print(f"static __constant__ double {name}[{len(values)}] = {{")
    for x in values:
        print(f"    {repr(float(x))},")
    print("};")
    print()


def cheb_monomial(f, a, b, deg):
    """Chebyshev interpolant of f on [a,b] (deg+1 Chebyshev points), returned
    as monomial coefficients c[0..deg] in v (high precision)."""
    n = deg + 1
    xs = [mp.cos(mp.pi * (k + mp.mpf(1) / 2) / n) for k in range(n)]
    vs = [(b - a) / 2 * x + (a + b) / 2 for x in xs]
    fs = [f(v) for v in vs]
    # Chebyshev coefficients
    cc = []
    for j in range(n):
        s = mp.fsum(fs[k] * mp.cos(mp.pi * j * (k + mp.mpf(1) / 2) / n) for k in range(n))
        cc.append(2 * s / n)
    cc[0] /= 2
    # T_j(x) as monomials in x, then substitute x = (2v - a - b)/(b - a)
    Tm = [[mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]]
    for j in range(2, n):
        prev, pprev = Tm[-1], Tm[-2]
        nxt = [mp.mpf(0)] * (j + 1)
        for i, c in enumerate(prev):
            nxt[i + 1] += 2 * c
        for i, c in enumerate(pprev):
            nxt[i] -= c
        Tm.append(nxt)
    px = [mp.mpf(0)] * n
    for j in range(n):
        for i, c in enumerate(Tm[j]):
            px[i] += cc[j] * c
    alpha = 2 / mp.mpf(b - a)
    beta = -mp.mpf(a + b) / (b - a)
    # x = alpha v + beta ; expand sum px[i] (alpha v + beta)^i
    pv = [mp.mpf(0)] * n
    for i, c in enumerate(px):
        for k in range(i + 1):
            pv[k] += c * mp.binomial(i, k) * alpha ** k * beta ** (i - k)
    return pv


def horner(coef, v, dtype):
    acc = dtype(coef[-1])
    for c in coef[-2::-1]:
        acc = dtype(acc * dtype(v) + dtype(c)) if dtype is np.float64 else \
            np.float32(np.float32(acc) * np.float32(v) + np.float32(c))
    return acc


def emit(name, f, a, b, deg, dtype, ctype, suffix, const_mem=None):
    c = cheb_monomial(f, a, b, deg)
    cr = [dtype(float(x)) for x in c]
    worst = 0.0
    for v in np.linspace(a, b, 4001):
        got = float(horner(cr, dtype(v), dtype))
        want = f(float(dtype(v)))
        worst = max(worst, abs(got - float(want)) / float(abs(want)))
    print(f"/* {name}: degree {deg} on v in [{a}, {b}], Horner in {ctype}: "
          f"max rel err {worst:.2e} */")
    print(f"#define {name}_DEG {deg}")
    # FP64 coefficients of the segment walk live in constant memory, read
    # with scalar loads into scalar registers, which an FMA takes as its
    # addend; as compile-time constants each would be copied into a vector
    # register at every use.  The per-loop cosine's are compile-time
    # constants that its FMA takes in scalar registers (see cos2pi).
    if const_mem is None:
        const_mem = ctype == "double"
    storage = "static __constant__" if const_mem else "static constexpr"
    print(f"{storage} {ctype} {name}[{deg + 1}] = {{")
    for x in cr:
        print(f"    {repr(float(x))}{suffix},")
    print("};")
    print()


if __name__ == "__main__":
    print("/* Generated by gen_poly.py -- do not edit.  Monomial coefficients in")
    print("   v, lowest order first. */")
    print("#pragma once")
    print()
    emit("WL_Q_SECH2_F32", q_exact, 0.0, 0.25, 4, np.float32, "float", "f")
    emit("WL_Q_SECH2_F64", q_exact, 0.0, 0.25, 12, np.float64, "double", "")
    emit("WL_P_GAUSS_F32", p_exact, 0.0, 0.25, 4, np.float32, "float", "f")
    emit("WL_P_GAUSS_F64", p_exact, 0.0, 0.5, 13, np.float64, "double", "")
    emit("WL_EXP2_F64", exp2_exact, -0.5, 0.5, 11, np.float64, "double", "")
    emit("WL_LOG1P_F64", log1p_exact, 0.0, float(mp.exp(-1)), 13, np.float64, "double", "")
    emit("WL_COS2PI_F64", cos2pi_exact, 0.0, 1 / 64, 7, np.float64, "double", "",
         const_mem=False)
    emit("WL_SIN2PI_F64", sin2pi_exact, 0.0, 1 / 64, 7, np.float64, "double", "",
         const_mem=False)
    emit("WL_EXP2M1_F64", exp2m1_exact, -1 / 128, 1 / 128, 4, np.float64, "double", "")
    emit("WL_LOG2P1_F64", log2p1_exact, -1 / 511, 1 / 511, 4, np.float64, "double", "")
    emit_table("WL_EXP2_TAB", [mp.power(2, mp.mpf(j) / 64) for j in range(64)],
               "2^(j/64), rounded to double")
    inv = [mp.mpf(float(1 / (1 + (mp.mpf(j) + 0.5) / 256))) for j in range(128)]
    emit_table("WL_LOG2_TAB", [v for c in inv for v in (c, 1 + mp.log(c, 2))],
               "pairs c_j, 1 + log2 c_j")
