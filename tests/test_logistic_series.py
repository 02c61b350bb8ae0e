"""The logistic kernels evaluate log(1 + e), e = exp(-|t|) in [0, 1], by the series 2 atanh(u) = 2 u (1 + u^2/3 + ... +
u^30/31), u = e / (2 + e) (device_util.h: log1p_unit).  This checks the claim made there -- within 2 ulp of the exact
value on that range -- with the same operations in fp64 on the host against numpy's extended-precision log1p.  (The
device path itself is held to the oracle by the GPU parity tests of the objective.)"""
import numpy as np


def series(e):
    u = e / (2.0 + e)
    w = u * u
    p = np.full_like(e, 1.0 / 31.0)
    for k in range(14, -1, -1):
        p = p * w + 1.0 / (2 * k + 1)
    return 2.0 * u * p


def test_series_is_within_two_ulp_on_the_unit_interval():
    rng = np.random.default_rng(2008)
    t = np.concatenate([rng.uniform(0.0, 40.0, 1_000_000), rng.uniform(0.0, 1.0, 300_000), rng.uniform(0.0, 0.01, 100_000),
                        np.array([0.0, 1e-300, 1e-17, 36.0, 37.0, 600.0])])
    e = np.exp(-t)
    assert e.min() > 0.0 and e.max() <= 1.0
    exact = np.log1p(e.astype(np.longdouble))
    rel = np.abs((series(e).astype(np.longdouble) - exact) / exact)
    assert float(rel.max()) <= 2 * np.finfo(np.float64).eps          # 2 ulp = 4.4e-16
    assert float(rel.mean()) <= 1e-16
    # the first term left out, relative to the sum, at the largest u = 1/3
    assert (1.0 / 9.0) ** 16 / 33.0 < 2e-17


def test_series_at_the_ends():
    assert series(np.array([0.0]))[0] == 0.0
    assert abs(series(np.array([1.0]))[0] - np.log(2.0)) <= 2 * np.finfo(np.float64).eps * np.log(2.0)


def test_logarithm_of_the_product_is_no_further_off_than_the_sum_of_the_series():
    """LossSum: log(1 + p) with p -> p + e + p e over up to 256 rows a time (then scaled by 2^-256 where it is large), against
    extended precision, for losses of any size; bound: the roundings of the additions, two an addend, relative to the sum."""
    rng = np.random.default_rng(2009)
    for scale in (0.0, 0.3, 3.0, 20.0, 300.0):
        t = scale * rng.random((1500, 64))
        e = np.exp(-t)
        lin, p = np.zeros(64), np.zeros(64)
        for i, row in enumerate(e):
            p = p * row + (p + row)
            if i % 256 == 255:
                large = p > 2.0 ** 256
                p = np.where(large, p * 2.0 ** -256 - 1.0, p)
                lin = lin + np.where(large, 256.0 * 0.6931471805599453, 0.0)
        exact = np.log1p(e.astype(np.longdouble)).sum(axis=0)
        rel = np.abs(((lin + np.log1p(p)).astype(np.longdouble) - exact) / exact)
        assert float(rel.max()) <= 2 * 1500 * np.finfo(np.float64).eps / 2
        assert float(rel.max()) <= 1e-14                                          # far inside it: measured 2e-15
        summed = np.zeros(64)   # the losses one by one, as they were added before
        for row in e:
            summed = summed + series(row)
        before = np.abs((summed.astype(np.longdouble) - exact) / exact)
        assert float(rel.mean()) <= float(before.mean()) and float(rel.max()) <= float(before.max())


def test_exponential_of_non_positive_arguments():
    """exp_nonpositive with the same operations in fp64 (its fused multiply-adds through extended precision): 1 ulp."""
    rng = np.random.default_rng(2010)
    x = -np.concatenate([rng.uniform(0.0, 40.0, 200_000), rng.uniform(0.0, 1.0, 200_000), rng.uniform(0.0, 700.0, 200_000), [0.0, 1e-300, 745.0]])
    ld = np.longdouble

    def fma(a, b, c):
        return (a.astype(ld) * ld(b) + np.asarray(c, dtype=ld)).astype(np.float64)

    k = np.rint(x * 1.4426950408889634)
    r = fma(k, -2.3190468138462996e-17, fma(k, -0.6931471805599453, x))
    q = np.full_like(r, 2.0914686968086876e-09)
    for c in (2.5105217004720745e-08, 2.75572736431103e-07, 2.7557255400206422e-06, 2.4801587325547743e-05, 0.00019841269874820627,
              0.0013888888888883748, 0.008333333333326136, 0.04166666666666667, 0.1666666666666667, 0.5):
        q = (q.astype(ld) * r.astype(ld) + ld(c)).astype(np.float64)
    t = ((r * r).astype(ld) * q.astype(ld) + r.astype(ld)).astype(np.float64)
    e = np.ldexp(1.0 + t, k.astype(int))
    exact = np.exp(x.astype(ld))
    normal = exact > 1e-300
    rel = np.abs((e.astype(ld)[normal] - exact[normal]) / exact[normal])
    assert float(rel.max()) <= np.finfo(np.float64).eps
    assert np.all(np.abs(e[~normal] - exact[~normal].astype(np.float64)) <= 5e-324 + 1e-15 * exact[~normal].astype(np.float64))
