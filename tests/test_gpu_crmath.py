"""The kernels' arithmetic on which the per-particle contract rests: shared reciprocals, quotients and
roots round as the operators do; sine, cosine, exponential and logarithm from tables are correctly
rounded; the unrounded sine and cosine keep the error that the rounding test allows for."""
import math
from decimal import Decimal, getcontext

import numpy as np
import pytest

import crmath_probe as P
import oracle
from test_oracle_crmath import _series

pytestmark = pytest.mark.gpu
getcontext().prec = 60


def _same_bits(got, want, *args):
    ok = (got == want) & (np.signbit(got) == np.signbit(want)) | np.isnan(got) & np.isnan(want)
    i = np.flatnonzero(~ok)
    assert not len(i), (len(i), [(a[i[0]], got[i[0]], want[i[0]]) for a in args])


def _steps(x, k):
    """x moved by k units in its last place (x > 0)."""
    t = np.int64 if x.dtype == np.float64 else np.int32
    return (x.view(t) + k.astype(t)).view(x.dtype)


def _operands(rng, dtype, n, lo, hi):
    return (rng.uniform(1, 2, n) * 2.0 ** rng.integers(lo, hi, n)).astype(dtype)


# exponents that the reciprocal forms are made for: FP64 up to +-900, FP32 up to +-90
@pytest.mark.parametrize("dtype,e", [(np.float64, 900), (np.float32, 60)])
def test_quotients_round_as_the_operator(dtype, e):
    rng = np.random.default_rng(1)
    n = 2_000_000
    b = _operands(rng, dtype, n, -40, 41)
    q = _operands(rng, dtype, n, -e // 2, e // 2)
    a = np.concatenate([
        _operands(rng, dtype, n, -e, e) * rng.choice(np.array([-1, 1], dtype=dtype), n),
        _steps(q * b, rng.integers(-1, 2, n)),                                         # quotients next to a number
        (np.longdouble(q) * b * (1 + np.longdouble(np.finfo(dtype).eps) / 2)).astype(dtype)])  # and to a midpoint
    b = np.concatenate([b, b, b])
    got = P.call(P.QUOT, a, b)
    _same_bits(got[0] if dtype == np.float64 else got, a / b, a, b)


@pytest.mark.parametrize("dtype,e", [(np.float64, 900), (np.float32, 90)])
def test_roots_and_quotients_by_them_round_as_the_operator(dtype, e):
    rng = np.random.default_rng(2)
    n = 2_000_000
    s = _operands(rng, dtype, n, 0, e // 2)
    a = np.concatenate([_operands(rng, dtype, n, 0, e), np.maximum(_steps(s * s, rng.integers(-2, 3, n)), dtype(1)),
                        (np.longdouble(s) * s * (1 + np.longdouble(np.finfo(dtype).eps))).astype(dtype)])
    first = lambda r: r[0] if dtype == np.float64 else r
    _same_bits(first(P.call(P.ROOT, a)), np.sqrt(a), a)
    x = _operands(rng, dtype, len(a), -e // 2, e // 2)
    _same_bits(first(P.call(P.QUOT_BY_ROOT, x, a)), x / np.sqrt(a), x, a)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_special_operands(dtype):
    v = np.array([0.0, -0.0, 1.0, -1.0, 1.5, 3.0, 1e30, np.inf, -np.inf, np.nan], dtype=dtype)
    a, b = (t.ravel() for t in np.meshgrid(v, v))
    first = lambda r: r[0] if dtype == np.float64 else r
    with np.errstate(all="ignore"):
        _same_bits(first(P.call(P.QUOT, a, b)), a / b, a, b)
        r = np.array([1.0, np.nextafter(dtype(1), dtype(2)), 4.0, np.inf, np.nan], dtype=dtype)
        _same_bits(first(P.call(P.ROOT, r)), np.sqrt(r), r)
        a, b = (t.ravel() for t in np.meshgrid(v, r))
        _same_bits(first(P.call(P.QUOT_BY_ROOT, a, b)), a / np.sqrt(b), a, b)


def _vec(fn, x):
    return np.array([fn(v) for v in x.tolist()])


def _angles(rng, n):
    """Angles over the accepted range, and next to the table's nodes, where a term vanishes."""
    k = np.concatenate([np.arange(-1100, 1101), rng.integers(-2**26, 2**26, n)]).astype(np.float64)
    node = np.abs((k.astype(np.longdouble) * np.longdouble("3.14159265358979323846264338327950288") / 256)
                  .astype(np.float64)) + 1e-300
    near = np.concatenate([_steps(node, np.full(len(node), d)) for d in (-2, -1, 0, 1, 2)])
    half = (rng.integers(-10**6, 10**6, n) + 0.5) * math.pi / 256
    x = np.concatenate([rng.uniform(-10, 10, n), rng.uniform(-1e3, 1e3, n), rng.uniform(-2.0**20, 2.0**20, n), near,
                        -near, half, 10.0 ** rng.uniform(-20, 0, n),
                        [0.0, 5e-324, 1e-308, 1e-30, math.pi, math.pi / 2, 1048575.9999999999]])
    return x[np.abs(x) < 2.0**20]


def test_sine_and_cosine_are_correctly_rounded():
    L = oracle.lib()
    x = _angles(np.random.default_rng(3), 60_000)
    s, c = _vec(L.oracle_cr_sin, x), _vec(L.oracle_cr_cos, x)
    for fn, want in ((P.SIN, s), (P.COS, c), (P.SIN_OF_BOTH, s), (P.COS_OF_BOTH, c)):
        got = P.call(fn, x)[0]
        bad = np.flatnonzero(got != want)
        assert not len(bad), (fn, len(bad), x[bad[0]].hex(), got[bad[0]], want[bad[0]])
    # the photon sweep's functions: 2e-16 absolute, with the argument's reduction (k pi/256, k below 2^27) in
    # two parts of pi/256 whose rest is below 2^-96 k
    m = np.abs(x) < 1e5
    for fn, want in ((P.FAST_SIN, s), (P.FAST_COS, c)):
        assert np.max(np.abs(P.call(fn, x[m])[0] - want[m])) < 3e-16  # 2e-16, and the rounding of `want`


def test_unrounded_sine_and_cosine_leave_the_rounding_test_its_margin():
    # stated: below 2^-67 of the result; the rounding test allows for 2^-66
    x = _angles(np.random.default_rng(4), 1500)
    x = np.random.default_rng(5).permutation(x[np.abs(x) > 1e-18])[:12_000]
    for fn, first, start in ((P.DD_SIN, lambda r: r, 1), (P.DD_COS, lambda r: Decimal(1), 0)):
        hi, lo = P.call(fn, x)
        worst = Decimal(0)
        for v, h, l in zip(x.tolist(), hi.tolist(), lo.tolist()):
            e = _series(v, first, start)
            worst = max(worst, abs((Decimal(h) + Decimal(l)) / e - 1))
        print("fn %d: 2^%.2f" % (fn, math.log2(worst)))
        assert worst < Decimal(2) ** -67


def test_exponential_and_logarithm_are_correctly_rounded():
    L = oracle.lib()
    rng = np.random.default_rng(6)
    n = 100_000
    node = rng.integers(-64000, 64000, n) * math.log(2) / 64
    x = np.concatenate([rng.uniform(-699, 708, n), rng.uniform(-40, 5, n), node, (node + math.log(2) / 128),
                        rng.choice([-1, 1], n) * 10.0 ** rng.uniform(-320, 0, n), [0.0, -0.0, 1.0, -1.0, 708.9, -699.9]])
    x = x[(x > -700) & (x < 709)]
    _same_bits(P.call(P.EXP, x)[0], _vec(L.oracle_cr_exp, x), x)
    edge = (0.5 + np.arange(0, 129) / 256.0)[:, None] * 2.0 ** np.arange(-40, 41)[None, :]
    edge = np.concatenate([_steps(edge.ravel(), np.full(edge.size, d)) for d in (-1, 0, 1)])
    one = np.concatenate([1 + np.arange(-3000, 3001) * 2.0**-53, 1 + rng.choice([-1, 1], n) * 2.0 ** -rng.uniform(1, 52, n)])
    y = np.concatenate([2.0 ** rng.uniform(-1020, 1020, n), 2.0 ** rng.uniform(-40, 40, n), edge, one, rng.uniform(0, 1, n),
                        [2.0**-1021, 2.0**-1022, 5e-324, 1.7976931348623157e308, 2.0**-54]])
    y = y[y > 0]
    _same_bits(P.call(P.LOG, y)[0], _vec(L.oracle_cr_log, y), y)
