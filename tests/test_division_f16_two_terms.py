"""The binary16 step's division by the total mass as a (hi + lo) in two packed
binary16 operations: correctly rounded for every finite dividend from 0.0646 on
(exhaustive), and the dividends of a step whose episode goes on lie above that."""
import numpy as np

f16 = np.float16
M = f16(f16(0.1) + f16(1.0))


def quotient(a):  # correctly rounded: binary64 and then binary16, 53 >= 2 * 11 + 2
    return (a.astype(np.float64) / float(M)).astype(f16)


def test_two_terms_exhaustive():
    a = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16).view(f16)
    a = a[np.isfinite(a) & (np.abs(a.astype(np.float64)) >= 0.0646)]
    hi = f16(1.0 / float(M))
    lo = f16(1.0 / float(M) - float(hi))
    low = (a.astype(np.float64) * float(lo)).astype(f16)
    with np.errstate(over="ignore"):
        # the exact sum of a 22-bit and an 11-bit number, rounded once
        got = (a.astype(np.float64) * float(hi) + low.astype(np.float64)).astype(f16)
        want = quotient(a)
    assert np.array_equal(got.view(np.uint16), want.view(np.uint16))


def test_dividends_of_going_steps():
    limit = f16(12 * 2 * np.pi / 360)
    th = np.arange(0, int(limit.view(np.uint16)) + 1, 7, dtype=np.uint16).view(f16)
    thd = np.concatenate([np.linspace(-24, 24, 1501).astype(f16)])
    least = [np.inf, np.inf]
    pml = f16(f16(0.1) * f16(0.5))
    for v in thd:  # the mirrored angles give mirrored dividends
        t = th[np.abs(th + f16(0.02) * v) <= limit]
        sn = np.sin(t.astype(np.float64)).astype(f16)
        c = np.cos(t.astype(np.float64)).astype(f16)
        den = f16(0.5) * (f16(4 / 3) - quotient(f16(0.1) * (c * c)))
        for force in (f16(10), f16(-10)):
            first = force + pml * (v * v) * sn
            temp = quotient(first)
            num = f16(9.8) * sn - c * temp
            acc = (num.astype(np.float64) / den.astype(np.float64)).astype(f16)
            second = pml * acc * c
            for k, d in enumerate((first, second)):
                if d.size:
                    least[k] = min(least[k], float(np.abs(d).min()))
    assert least[0] > 5.0 and least[1] > 0.2, least
