"""The device's FP64 normals against extended precision, value by value, from both
generators (the LB stream's polynomials, the tables of the other streams): 4 M
normals each, whose uniforms reach 2^-20 and 1 - 2^-20.

Bars, in units of 2^-52.  A normal z = r c has the radius' relative error, half of
the logarithm's (1.023, tests/test_bm_exact.py) and a rounding of the square root
(1/2), its product's rounding (1/2), and r times the absolute error of the sine or
cosine (0.76): at most r (1.52 |c| + 0.76) <= 2.3 r.  Root mean square: 0.392 (the
same test's bar for a normal), and 1% for the sample."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def philox(site, step, block, tag, seed):
    """Philox4x32-10 of the counters (site, step, block, tag), site an array."""
    mask, m0, m1 = np.uint64(0xFFFFFFFF), np.uint64(0xD2511F53), np.uint64(0xCD9E8D57)
    c = [site.astype(np.uint64)] + [np.full(site.shape, v, np.uint64) for v in (step, block, tag)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        p0, p1 = m0 * c[0], m1 * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
    return c


@pytest.mark.parametrize("tag", [0, 1, 2])
def test_normals_are_exact(tag):
    from paper_1104_0078_amd import lbl
    assert np.finfo(np.longdouble).nmant >= 63
    n, seed, step, unit = 1 << 20, (0x9E3779B9 << 32) + 77, 5, np.longdouble(2.0) ** -52
    z = lbl.diag_normals(lbl.LBL_FP64, seed, step, tag, 11, n, 4)
    k = philox(11 + np.arange(n, dtype=np.uint64), step, 0, tag, seed)
    worst, sum2 = 0.0, 0.0
    for a in (0, 2):
        ua, ub = [(v.astype(np.longdouble) + np.longdouble(0.5)) / np.longdouble(2.0) ** 32
                  for v in (k[a], k[a + 1])]
        r = np.sqrt(-2 * np.log(ua))
        angle = np.longdouble("6.283185307179586476925286766559005768") * ub
        for j, ref in ((a, r * np.cos(angle)), (a + 1, r * np.sin(angle))):
            err = ((z[:, j].astype(np.longdouble) - ref) / unit).astype(np.float64)
            worst = max(worst, float(np.abs(err / r.astype(np.float64)).max()))
            sum2 += float((err ** 2).sum())
    rms = (sum2 / (4 * n)) ** 0.5
    print("tag %d: rms %.4f, worst %.3f r" % (tag, rms, worst), flush=True)
    assert worst <= 2.3
    assert rms <= 0.392 * 1.01
