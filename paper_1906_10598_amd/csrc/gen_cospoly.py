"""Write cospoly.h: polynomial coefficients of cos(2 pi r) and sin(2 pi r), |r| <= 1/2.

The device kernels reduce the phase to turns r in [-1/2, 1/2] exactly
(r = x - rint(x)) and evaluate cos(2 pi r) = p(r^2) with a near-minimax
polynomial p fitted on u = r^2 in [0, 1/4] at Chebyshev nodes (mpmath
chebyfit, 50 digits).  Degree 10 in u gives an approximation error of
3.3e-17 (below FP64 rounding), degree 9 gives 6.2e-15; degree 6 gives 1.1e-8
(below FP32 rounding).  Phases known to lie within 1/8 or 1/48 of a
turn take degree 6 or 4 in FP64.

Run:  python gen_cospoly.py  (rewrites cospoly.h next to this script).
"""
import os

import mpmath

mpmath.mp.dps = 50
HERE = os.path.dirname(os.path.abspath(__file__))


def fit(deg, odd=False, rmax=mpmath.mpf(1) / 2):
    if odd:  # sin(2 pi r) / r as a polynomial in u = r^2
        f = lambda u: (mpmath.sin(2 * mpmath.pi * mpmath.sqrt(u)) / mpmath.sqrt(u)  # noqa: E731
                       if u != 0 else 2 * mpmath.pi)
    else:
        f = lambda u: mpmath.cos(2 * mpmath.pi * mpmath.sqrt(u))  # noqa: E731
    poly, err = mpmath.chebyfit(f, [0, rmax ** 2], deg + 1, error=True)
    # chebyfit returns highest degree first
    return [float(c) for c in poly], float(err)


def main():
    p64, e64 = fit(10)
    p64s, e64s = fit(9)
    s64, es64 = fit(10, odd=True)
    cn, ecn = fit(6, rmax=mpmath.mpf(1) / 8)
    sn, esn = fit(6, odd=True, rmax=mpmath.mpf(1) / 8)
    c8, ec8 = fit(4, rmax=mpmath.mpf(1) / 48)
    s8, es8 = fit(4, odd=True, rmax=mpmath.mpf(1) / 48)
    p32, e32 = fit(6)
    lines = [
        "// Generated by gen_cospoly.py -- do not edit.",
        "// cos(2 pi r) = p(r^2) for |r| <= 1/2; coefficients highest degree first.",
        f"// FP64: degree 10, approximation error {e64:.2e}.  FP32: degree 6, {e32:.2e}.",
        "#pragma once",
        "namespace pt {",
        f"constexpr int kCosDeg64 = {len(p64) - 1};",
        "constexpr double kCos64[] = {",
    ]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in p64]
    lines += ["};", f"// FP64, degree 9: approximation error {e64s:.2e}.",
              f"constexpr int kCosDeg64s = {len(p64s) - 1};", "constexpr double kCos64s[] = {"]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in p64s]
    lines += ["};", f"// sin(2 pi r) = r q(r^2), FP64, degree 10 in u: error of q {es64:.2e}.",
              f"constexpr int kSinDeg64 = {len(s64) - 1};", "constexpr double kSin64[] = {"]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in s64]
    lines += ["};", f"// |r| <= 1/8: cos(2 pi r) and sin(2 pi r) / r, degree 6 in u: errors {ecn:.2e}, {esn:.2e}.",
              f"constexpr int kNarDeg64 = {len(cn) - 1};", "constexpr double kCosNar64[] = {"]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in cn]
    lines += ["};", "constexpr double kSinNar64[] = {"]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in sn]
    lines += ["};", f"// |r| <= 1/48, degree 4 in u: errors {ec8:.2e}, {es8:.2e}.",
              f"constexpr int kNar8Deg64 = {len(c8) - 1};", "constexpr double kCosNar8[] = {"]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in c8]
    lines += ["};", "constexpr double kSinNar8[] = {"]
    lines += [f"    {c.hex()},  // {c:.17e}" for c in s8]
    lines += ["};", f"constexpr int kCosDeg32 = {len(p32) - 1};", "constexpr float kCos32[] = {"]
    for c in p32:
        cf = float(mpmath.mpf(c))
        import struct
        c32 = struct.unpack("f", struct.pack("f", cf))[0]
        lines.append(f"    {c32.hex()}f,  // {c32:.9e}")
    lines += ["};", "}  // namespace pt", ""]
    with open(os.path.join(HERE, "cospoly.h"), "w") as fh:
        fh.write("\n".join(lines))


if __name__ == "__main__":
    main()
