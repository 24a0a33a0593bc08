"""Constants of the exponentials of fp64_math.hpp, from the mathematics in many-digit arithmetic.

exp_neg_f64: coefficients of the degree-11 polynomial for e^t on |t| ≤ ln2/2, the interpolant of e^t at the 12 Chebyshev nodes of the interval
(near-minimax), solved in the monomial basis in 60-digit arithmetic and rounded to doubles.
Prints the coefficients (t^0 first) and the largest relative error of their Horner
evaluation on a 4001-point grid, measured in 60-digit arithmetic (1.7e-17; the Taylor
series to degree 13 gives 5.2e-18, the FP64 rounding unit is 1.1e-16).

exp_neg_tab_f64, the table-driven method of P. T. P. Tang ("Table-driven implementation of the exponential
function in IEEE floating-point arithmetic", ACM Trans. Math. Softw. 15, 1989): exp_table.hpp (written beside this
file) with 2^{i/256} as the nearest double and the rest, and the coefficients of e^r ≈ 1 + r + r²(c2 + c3 r + c4 r²) on |r| ≤ ln2/512, the quadratic through
(e^r − 1 − r)/r² at its three Chebyshev nodes (relative error of e^r 9.5e-18).

    python paper_1709_08070_amd/csrc/exp_coeffs.py
"""
import os

import mpmath as mp

mp.mp.dps = 60
DEG = 11
L = mp.log(2) / 2
nodes = [L * mp.cos(mp.pi * (2 * k + 1) / (2 * (DEG + 1))) for k in range(DEG + 1)]
A = mp.matrix([[x ** j for j in range(DEG + 1)] for x in nodes])
c = mp.lu_solve(A, mp.matrix([mp.e ** x for x in nodes]))
coef = [float(c[j]) for j in range(DEG + 1)]
worst = mp.mpf(0)
for i in range(4001):
    t = -L + 2 * L * i / 4000
    p = mp.mpf(0)
    for cj in reversed(coef):
        p = p * t + mp.mpf(cj)
    worst = max(worst, abs(p / mp.e ** t - 1))
for j, v in enumerate(coef):
    print(f"c{j} = {v!r}")
print(f"max relative error {float(worst):.2e}")

mp.mp.dps = 200  # (e^r − 1 − r)/r² loses two thirds of the digits at the middle node
N = 256
L = mp.log(2) / (2 * N)
nodes = [L * mp.cos(mp.pi * (2 * k + 1) / 6) for k in range(3)]
A = mp.matrix([[x ** j for j in range(3)] for x in nodes])
c = mp.lu_solve(A, mp.matrix([(mp.e ** x - 1 - x) / x ** 2 if abs(x) > 1e-50 else mp.mpf(1) / 2 for x in nodes]))
coef = [float(c[j]) for j in range(3)]
worst = mp.mpf(0)
for i in range(2001):
    r = -L + 2 * L * i / 2000
    worst = max(worst, abs((1 + r + r * r * (coef[0] + r * (coef[1] + r * mp.mpf(coef[2])))) / mp.e ** r - 1))
print(f"c2..c4 = {coef!r}, max relative error {float(worst):.2e}")
step = mp.log(2) / N
hi = float(step)
print(f"ln2/{N} = {hi!r} + {float(step - mp.mpf(hi))!r}; {N}/ln2 = {float(1 / step)!r}")
rows = []
for i in range(N):
    t = mp.mpf(2) ** (mp.mpf(i) / N)
    rows.append("{%s, %s}" % (float(t).hex(), float(t - mp.mpf(float(t))).hex()))
with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "exp_table.hpp"), "w") as f:
    f.write("// 2^{i/256}: the nearest double and the rest. Written by exp_coeffs.py, which names the method.\n")
    f.write("#pragma once\n\n")
    f.write("#include <hip/hip_runtime.h>\n\nnamespace pb {\n\n")
    f.write("static __device__ const double2 kExpTable[%d] = {\n" % N)
    for i in range(0, N, 2):
        f.write("    %s,\n" % ", ".join(rows[i:i + 2]))
    f.write("};\n\n}  // namespace pb\n")
