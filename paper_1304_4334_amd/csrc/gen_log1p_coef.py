"""Coefficients of the FP64 logarithm in model.h (kLog1pCoef, log1p_pos).

With s = f / (2 + f), log(1 + f) = 2 atanh(s) = f - s (f - z Q(z)), z = s^2,
Q(z) = 2/3 + 2 z / 5 + 2 z^2 / 7 + ...  The polynomial of degree DEG for Q that
minimises the largest error of z Q(z) / 2, the logarithm's relative error, over
1 + f in [sqrt(1/2), sqrt(2)] (Remez exchange in 50-digit arithmetic, started
from Chebyshev points), printed as C99 hex doubles with that error as the
coefficients are rounded.  Run with `python gen_log1p_coef.py`; needs mpmath.
"""
import mpmath as mp

mp.mp.dps = 50
DEG = 6
S = (mp.sqrt(2) - 1) / (mp.sqrt(2) + 1)
HI = S * S


def q(z):
    if z == 0:
        return mp.mpf(2) / 3
    s = mp.sqrt(z)
    return (2 * mp.atanh(s) / s - 2) / z


def err(c, z):
    return z * (mp.polyval(c[::-1], z) - q(z)) / 2


def remez(n, iters=12):
    # the error vanishes at 0, so the reference points lie in (0, HI]
    xs = [HI * (1 - mp.cos(mp.pi * (2 * k + 3) / (2 * n + 5))) / 2 for k in range(n + 1)] + [HI]
    grid = [HI * k / 6000 for k in range(1, 6001)]
    for _ in range(iters):
        M = mp.matrix(n + 2, n + 2)
        rhs = mp.matrix(n + 2, 1)
        for i, x in enumerate(xs):
            for j in range(n + 1):
                M[i, j] = x ** (j + 1) / 2
            M[i, n + 1] = (-1) ** i
            rhs[i] = x * q(x) / 2
        sol = mp.lu_solve(M, rhs)
        c = [sol[j] for j in range(n + 1)]
        vals = [err(c, x) for x in grid]
        ext = [grid[k] for k in range(1, len(grid) - 1)
               if (vals[k] - vals[k - 1]) * (vals[k + 1] - vals[k]) <= 0]
        ext.append(grid[-1])
        if len(ext) != n + 2:
            break
        xs = ext
    return c


def main():
    cd = [float(x) for x in remez(DEG)]
    worst = max(abs(err([mp.mpf(x) for x in cd], HI * k / 20000)) for k in range(1, 20001))
    print(f"// degree {DEG}, relative error {mp.nstr(worst, 3)} with double coefficients")
    for x in cd:
        print(f"  {x.hex()},")


if __name__ == "__main__":
    main()
