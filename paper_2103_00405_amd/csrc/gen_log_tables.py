"""Generate log_tables.inc: constants of the GPU's correctly rounded -ln(u).

Method (table-driven argument reduction in the style of Tang, 1990, with a
Ziv-style two-phase evaluation):
  u = 2^e f; the top 9 mantissa bits of f select a reciprocal r_i with 9
  significant bits, so that z = f r_i - 1 is exact in binary64 and |z| <= 2^-8;
  then ln u = e ln 2 - ln r_i + ln(1 + z).
Tables written here:
  RTAB[i]          r_i (binary64, 9 significant bits)
  LNR_H/LNR_L[i]   ln r_i as a double-double (fast phase)
  LNR_FIX[i][9]    ln r_i in two's-complement fixed point, 2^-256 units
                   (32-bit limbs, little-endian; accurate phase)
  LN2_FIX[9]       ln 2 in the same format
  INVK_FIX[j][9]   1/(j+1) in the same format, j = 0..KMAX (Horner for ln(1+z))
  LN2_H, LN2_L     ln 2 split so that e * LN2_H is exact for |e| <= 64
  THIRD_H, THIRD_L 1/3 as a double-double
First (quick) phase, a table of 256 triples for the top 8 mantissa bits of f in
[1, 2), with -ln u = -e ln 2 + ln r - ln(1 + z) and r in [1/2, 1]:
  LOGQ[3 i ..]     (H, L, r_i): H is ln r_i to a multiple of 2^-46, L the rest
  QLN2_H, QLN2_L   ln 2 in the same form: at u just below 1 (r = 1/2, e = -1)
                   the table's terms cancel to exactly 0
  LOGQ_C[j]        coefficients of (ln(1+z) - z + z^2/2) / z^3 to degree 5 on
                   |z| <= 2^-8: the Taylor terms through z^9 with the last
                   replaced by its Chebyshev economization
Every value is computed with Python's decimal module at 120 significant
digits; no other source is consulted.  Run: python gen_log_tables.py > log_tables.inc
"""
from decimal import Decimal, getcontext
from fractions import Fraction
import math
import sys

getcontext().prec = 120
NBITS = 9            # index bits and reciprocal significant bits
NT = 1 << NBITS
I_HALF = 212         # intervals with f >= 1 + I_HALF/512 (about sqrt 2) use f/2
FRAC = 256           # fixed-point fraction bits of the accurate phase
LIMBS = 9            # 32 integer bits + 256 fraction bits
KMAX = 31            # ln(1+z) = z * sum_{j<=KMAX} (-z)^j / (j+1)


def round_sig(x: Fraction, bits: int) -> Fraction:
    """Round a positive rational to `bits` significant bits, ties to even."""
    e = math.floor(math.log2(x))
    if Fraction(2) ** e > x:
        e -= 1
    if Fraction(2) ** (e + 1) <= x:
        e += 1
    scale = Fraction(2) ** (bits - 1 - e)
    v = x * scale
    n = v.numerator // v.denominator
    rem = v - n
    if rem > Fraction(1, 2) or (rem == Fraction(1, 2) and n % 2 == 1):
        n += 1
    return Fraction(n) / scale


def dec(fr: Fraction) -> Decimal:
    return Decimal(fr.numerator) / Decimal(fr.denominator)


def fix(x: Decimal) -> list:
    """Signed fixed point, 2^-FRAC units, rounded to nearest, as LIMBS 32-bit limbs."""
    v = int((x * (Decimal(2) ** FRAC)).to_integral_value())
    v &= (1 << (32 * LIMBS)) - 1
    return [(v >> (32 * i)) & 0xFFFFFFFF for i in range(LIMBS)]


QBITS = 8            # index bits of the quick phase's table
QGRID = 46           # H is a multiple of 2^-QGRID


def quick_tables():
    grid = Fraction(2) ** QGRID
    r, hl = [], []
    n = 1 << QBITS
    for i in range(n):
        lo, hi = Fraction(n + i, n), Fraction(n + i + 1, n)
        ri = Fraction(1) if i == 0 else round_sig(2 / (lo + hi), 9)
        zmax = max(abs(lo * ri - 1), abs(hi * ri - 1))
        assert Fraction(1, 2) <= ri <= 1 and zmax <= Fraction(1, 256), (i, float(zmax))
        ln_r = dec(ri).ln()
        H = Fraction(int((ln_r * Decimal(2 ** QGRID)).to_integral_value())) / grid
        L = ln_r - dec(H)
        r.append(ri)
        hl.append((float(H), float(L)))
        assert Fraction(hl[-1][0]) == H
    assert r[n - 1] == Fraction(1, 2)
    ln2_h, ln2_l = -hl[n - 1][0], -hl[n - 1][1]
    # the sum h - ln(1 + z), h = -e ln2_h + H: h is 0 or its exponent is not
    # below that of any ln(1 + z) of its interval (checked where |h| is
    # smallest, e = -1; larger -e only adds to a non-negative h)
    for i in range(n):
        h = Fraction(ln2_h) + Fraction(hl[i][0])
        assert h >= 0 and (h == 0) == (i == n - 1)
        if h:
            lo, hi = Fraction(n + i, n), Fraction(n + i + 1, n)
            s = max(abs(dec(x * r[i]).ln()) for x in (lo, hi))
            assert math.frexp(float(h))[1] >= math.frexp(float(s))[1], (i, float(h), float(s))
    # (ln(1+z) - z + z^2/2) / z^3 = sum_j (-1)^j z^j / (j + 3), j <= 6, with
    # x^6 = (48 x^4 - 18 x^2 + 1) / 32 + T_6(x) / 32, x = 2^8 z
    c = [Fraction((-1) ** j, j + 3) for j in range(7)]
    a2 = Fraction(1, 2 ** 16)
    c[4] += c[6] * a2 * Fraction(48, 32)
    c[2] -= c[6] * a2 ** 2 * Fraction(18, 32)
    c[0] += c[6] * a2 ** 3 * Fraction(1, 32)
    return [(h, l, float(x)) for (h, l), x in zip(hl, r)], ln2_h, ln2_l, [float(x) for x in c[:6]]


def hexd(x: float) -> str:
    return float.hex(x)


def main(out):
    rtab, lnr_h, lnr_l, lnr_fix = [], [], [], []
    for i in range(NT):
        lo = Fraction(NT + i, NT)
        hi = Fraction(NT + i + 1, NT)
        if i >= I_HALF:
            lo, hi = lo / 2, hi / 2
        mid = (lo + hi) / 2
        r = round_sig(1 / mid, NBITS)
        # z = f r - 1 is linear in f: its extremes sit at the interval ends
        zmax = max(abs(lo * r - 1), abs(hi * r - 1))
        assert zmax <= Fraction(1, 256), (i, float(zmax))
        rf = float(r)
        assert Fraction(rf) == r
        L = dec(r).ln()
        h = float(L)
        l_ = float(L - Decimal(h))
        rtab.append(rf)
        lnr_h.append(h)
        lnr_l.append(l_)
        lnr_fix.append(fix(L))
    ln2 = Decimal(2).ln()
    # ln 2 high part with 42 significant bits: e * LN2_H is exact for |e| < 2^11
    ln2_h = float(round_sig(Fraction(ln2), 42))
    ln2_l = float(ln2 - Decimal(ln2_h))
    third_h = 1.0 / 3.0
    third_l = float(Decimal(1) / Decimal(3) - Decimal(third_h))
    w = out.write
    w("// Generated by gen_log_tables.py -- do not edit.\n")
    w("#define RT_LOG_NBITS %d\n#define RT_LOG_I_HALF %d\n#define RT_LOG_KMAX %d\n" % (NBITS, I_HALF, KMAX))
    w("#define RT_LOG_LIMBS %d\n#define RT_LOG_FRAC %d\n" % (LIMBS, FRAC))
    w("#define RT_LN2_H %s\n#define RT_LN2_L %s\n" % (hexd(ln2_h), hexd(ln2_l)))
    w("#define RT_THIRD_H %s\n#define RT_THIRD_L %s\n" % (hexd(third_h), hexd(third_l)))

    def arr_d(name, vals):
        w("RT_LOG_CONST double %s[%d] = {\n" % (name, len(vals)))
        for k in range(0, len(vals), 4):
            w("  " + ", ".join(hexd(v) for v in vals[k:k + 4]) + ",\n")
        w("};\n")

    def arr_fix(name, rows):
        w("RT_LOG_CONST uint32_t %s[%d][%d] = {\n" % (name, len(rows), LIMBS))
        for row in rows:
            w("  {" + ", ".join("0x%08xu" % v for v in row) + "},\n")
        w("};\n")

    arr_d("RT_RTAB", rtab)
    arr_d("RT_LNR_H", lnr_h)
    arr_d("RT_LNR_L", lnr_l)
    rows, qln2_h, qln2_l, qc = quick_tables()
    w("#define RT_LOGQ_BITS %d\n" % QBITS)
    w("#define RT_QLN2_H %s\n#define RT_QLN2_L %s\n" % (hexd(qln2_h), hexd(qln2_l)))
    for j, v in enumerate(qc):
        w("#define RT_LOGQ_C%d %s\n" % (j, hexd(v)))
    arr_d("RT_LOGQ", [x for row in rows for x in row])
    arr_fix("RT_LNR_FIX", lnr_fix)
    w("RT_LOG_CONST uint32_t RT_LN2_FIX[%d] = {" % LIMBS + ", ".join("0x%08xu" % v for v in fix(ln2)) + "};\n")
    arr_fix("RT_INVK_FIX", [fix(Decimal(1) / Decimal(j + 1)) for j in range(KMAX + 1)])


if __name__ == "__main__":
    main(sys.stdout)
