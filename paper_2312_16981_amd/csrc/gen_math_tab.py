"""Print the coefficients of MathTab (device_math.hpp): polynomials that interpolate their
function at the Chebyshev nodes of an interval, in 60-digit arithmetic, each rounded
once.  Run by hand; a test compares the header with coefficients().
"""
import mpmath as mp


def interpolate(f, lo, hi, degree):
    """Monomial coefficients, ascending, of the interpolant at the Chebyshev nodes of [lo, hi]."""
    n = degree + 1
    nodes = [(lo + hi) / 2 + (hi - lo) / 2 * mp.cos((2 * k + 1) * mp.pi / (2 * n)) for k in range(n)]
    A = mp.matrix(n, n)
    b = mp.matrix(n, 1)
    for i, x in enumerate(nodes):
        for j in range(n):
            A[i, j] = x ** j
        b[i] = f(x)
    return [float(c) for c in mp.lu_solve(A, b)]


def bernoulli_over_factorial(k):
    return mp.bernoulli(2 * k) / mp.factorial(2 * k)


def polylog_tail(m):
    """sum_{n >= 2} z^{n-2} / n^m"""
    return lambda z: sum(z ** (n - 2) / mp.mpf(n) ** m for n in range(2, 120))


def coefficients():
    with mp.workdps(60):
        four, two, one, zero = mp.mpf(4), mp.mpf(2), mp.mpf(1), mp.mpf(0)
        tail = mp.exp(-two)                          # z = e^{-x}, x >= 2
        half = mp.log(two) / 2 * mp.mpf("1.0001")    # the reduced argument of the exponential
        t = {}
        # (int_0^x t^3/(e^t - 1) dt - x^3/3 + x^4/8) / x^5 of x^2
        t["head"] = interpolate(lambda z: sum(bernoulli_over_factorial(k) / (2 * k + 3) * z ** (k - 1)
                                              for k in range(1, 45)), zero, four, 10)
        # (x/(e^x - 1) - 1 + x/2) / x^2 of x^2
        t["weight"] = interpolate(lambda z: sum(bernoulli_over_factorial(k) * z ** (k - 1) for k in range(1, 60)),
                                  zero, four, 10)
        for m, degree in ((1, 10), (2, 9), (3, 9), (4, 8)):
            t[f"L{m}"] = interpolate(polylog_tail(m), zero, tail, degree)
        # (e^{-r} - 1 + r) / r^2
        t["ex"] = interpolate(lambda r: sum((-1) ** n * r ** (n - 2) / mp.factorial(n) for n in range(2, 40)),
                              -half, half, 9)
        t["exf"] = interpolate(lambda r: sum((-1) ** n * r ** (n - 2) / mp.factorial(n) for n in range(2, 40)),
                               -half, half, 10)
        # (1 - e^{-x}) / x
        t["one_ex"] = interpolate(lambda x: sum((-1) ** n * x ** n / mp.factorial(n + 1) for n in range(60)),
                                  zero, two, 14)
        # (C4 - e^{-s}) / s
        t["w"] = interpolate(lambda s: sum((-1) ** (n + 1) * n * s ** (n - 1) / mp.factorial(n + 1)
                                           for n in range(1, 60)), zero, one, 11)
        # (C2/dt) / s
        t["c2"] = interpolate(lambda s: sum((-1) ** (n + 1) * (n - 1) * s ** (n - 2) / mp.factorial(n + 1)
                                            for n in range(2, 70)), zero, two, 14)
        # (atanh(s)/s - 1) / z of z = s^2, s = (m - 1)/(m + 1) with m up to sqrt(2) (rounded up)
        top = ((mp.sqrt(two) - 1) / (mp.sqrt(two) + 1)) ** 2 * mp.mpf("1.0000001")
        t["ln"] = interpolate(lambda z: sum(z ** (k - 1) / (2 * k + 1) for k in range(1, 60)), zero, top, 6)
    return t


if __name__ == "__main__":
    for name, c in coefficients().items():
        print(f"// {name}\n{{" + ", ".join(x.hex() for x in c) + "}")
