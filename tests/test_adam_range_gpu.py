"""The optimizer's arithmetic where its short forms begin and end.

A wave takes short divisions and a short square root when the updated moments
of all its elements lie in a middle range (|m| in 2^-60..2^20, v in
2^-96..2^60) or are zero, and the step constants are ordinary ones; any other
wave takes the general form.  Either way every bit must be the oracle's.  With beta = 0.5 and a zero
gradient the updated moments are exactly half the given ones, so both ends of
the ranges and every significand can be hit on the spot.
"""
import numpy as np
import pytest

import oracle
from gpu_common import assert_parity, to_dev, to_host, torch

pytestmark = pytest.mark.gpu


def _step(g, p, m, v, t, hp):
    import paper_2409_00918_amd as dd
    dp, dm, dv, d16 = to_dev(p), to_dev(m), to_dev(v), to_dev(np.zeros(p.size, np.uint16))
    dd.adam_step(to_dev(g), dp, dm, dv, d16, lr=hp["lr"], beta1=hp["beta1"], beta2=hp["beta2"],
                 eps=hp["eps"], weight_decay=hp["wd"], step=t)
    torch().cuda.synchronize()
    got = {"p": to_host(dp), "m": to_host(dm), "v": to_host(dv), "p16": to_host(d16)}
    p1, m1, v1, p16 = oracle.adamw(g, p, m, v, t=t, **hp)
    return got, {"p": p1, "m": m1, "v": v1, "p16": p16}


def _hp(beta1=0.5, beta2=0.5, eps=1e-8, lr=1.0, wd=0.0):
    f = np.float32
    return dict(lr=f(lr), beta1=f(beta1), beta2=f(beta2), eps=f(eps), wd=f(wd))


@pytest.mark.parametrize("exponent", [-40, 59])
def test_square_root_of_every_significand(exponent):
    # v over two binades: every significand at both parities of the exponent
    n = 1 << 24
    v = (np.arange(n, dtype=np.uint32) + np.uint32((127 + exponent) << 23)).view(np.float32)
    zero = np.zeros(n, np.float32)
    m = np.full(n, 2.0, np.float32)
    got, want = _step(zero, zero, m, v, 1, _hp(eps=0.0))
    assert_parity(got, want, f"exponent {exponent}")


@pytest.mark.parametrize("exponent", [-95, -40, 1, 38])
def test_square_root_of_every_significand_seen_exactly(exponent):
    # the weight is -m/d with m just below the root d, so the quotient lies
    # just below 1, where neighbouring d give quotients a unit apart or more
    n = 1 << 24
    v = (np.arange(n, dtype=np.uint32) + np.uint32((127 + exponent) << 23)).view(np.float32)
    m = (np.sqrt(v.astype(np.float64)) * (1 - 2.0**-22)).astype(np.float32)
    zero = np.zeros(n, np.float32)
    got, want = _step(zero, zero, m, v, 1, _hp(eps=0.0))
    assert_parity(got, want, f"exponent {exponent}")
    root = np.sqrt(v)
    assert np.all(m / np.nextafter(root, np.float32(0)) != m / root)
    assert np.all(m / np.nextafter(root, np.float32(np.inf)) != m / root)


@pytest.mark.parametrize("eps", [1e-8, 2.0**-48, np.nextafter(np.float32(2.0**-48), np.float32(0)),
                                 0.0])
@pytest.mark.parametrize("lr", [1e-3, -1e-3])
@pytest.mark.parametrize("share", [1 / 64, 0.3, 1.0])
def test_zero_moments_among_ordinary_ones(eps, lr, share):
    # m, v or both at zero (rows that have had no gradient), alone in their
    # wave or all of it; eps at the end of where it may divide alone and past it
    n = 64 * 256 + 7
    rng = np.random.default_rng(9)
    p = rng.standard_normal(n).astype(np.float32) * np.float32(0.02)
    p[rng.random(n) < 0.2] = 0.0
    p[rng.random(n) < 0.1] = -0.0
    g = rng.standard_normal(n).astype(np.float32) * np.float32(1e-4)
    m = rng.standard_normal(n).astype(np.float32) * np.float32(1e-4)
    v = m * m + np.float32(1e-12)
    zm, zv = rng.random(n) < share, rng.random(n) < share
    g[zm | zv] = np.where(rng.random(n) < 0.5, np.float32(0), np.float32(-0.0))[zm | zv]
    m[zm], v[zv] = 0.0, 0.0
    m[rng.random(n) < 1e-3] = -0.0
    for beta1, beta2 in ((0.9, 0.95), (0.0, 0.0), (0.5, 0.999)):
        got, want = _step(g, p, m, v, 3, _hp(beta1, beta2, eps, lr=lr, wd=0.1))
        assert_parity(got, want, f"eps {eps} lr {lr} share {share} betas {beta1} {beta2}")


@pytest.mark.parametrize("beta1,beta2,eps,t", [
    (0.5, 0.5, 1e-8, 1), (0.5, 0.5, 0.0, 1), (0.9, 0.95, 1e-8, 3), (0.9, 0.999, 1e-8, 1000),
    (0.0, 0.0, 1e-8, 1), (1 - 2.0**-24, 1 - 2.0**-24, 1e-8, 1),     # bias corrections 1 and 2^-24
    (0.5, 0.5, 2.0**40, 1), (0.5, 0.5, 2.0**41, 1)])                # eps at the end and past it
def test_moments_at_the_ends_of_the_range(beta1, beta2, eps, t):
    def around(x):
        x = np.float32(x)
        return [np.nextafter(x, np.float32(0)), x, np.nextafter(x, np.float32(np.inf))]
    special = [0.0, -0.0, 2.0**-149, 2.0**-126, np.inf, np.nan, 3.4e38]
    ms = np.array(sum([around(2.0**e) for e in (-61, -60, -59, 19, 20, 21, 0)], []) + special
                  + [-1e-5, -2.0**-59, -2.0**21, -np.inf], np.float32)
    vs = np.array(sum([around(2.0**e) for e in (-97, -96, -95, 59, 60, 61, -30)], []) + special
                  + [-1e-9], np.float32)
    m, v = (x.reshape(-1) for x in np.meshgrid(ms, vs))
    # alone in a lane of ordinary elements, and four to a lane
    rng = np.random.default_rng(5)
    k = m.size
    M = np.concatenate([rng.standard_normal((k, 4)).astype(np.float32) * np.float32(1e-4),
                        np.repeat(m, 4).reshape(k, 4)])
    V = np.concatenate([rng.random((k, 4), dtype=np.float32) * np.float32(1e-8) + np.float32(1e-12),
                        np.repeat(v, 4).reshape(k, 4)])
    at = np.arange(k) % 4
    M[np.arange(k), at] = m
    V[np.arange(k), at] = v
    M, V = M.reshape(-1), V.reshape(-1)
    p = rng.standard_normal(M.size).astype(np.float32)
    p[::97] = -0.0
    for g in (np.zeros(M.size, np.float32),
              rng.standard_normal(M.size).astype(np.float32) * np.float32(1e-4)):
        got, want = _step(g, p, M, V, t, _hp(beta1, beta2, eps, lr=1e-3, wd=0.1))
        assert_parity(got, want, f"betas {beta1} {beta2} eps {eps} t {t}")


def test_copy_of_nan_weights_is_the_quiet_nan_with_its_sign():
    # the hardware's conversion would keep payload bits
    n = 4096
    rng = np.random.default_rng(6)
    u = rng.standard_normal(n).astype(np.float32).view(np.uint32).copy()
    at = rng.choice(n, 300, replace=False)
    u[at] = (u[at] & 0x80000000) | 0x7F800000 | rng.integers(1, 1 << 23, 300).astype(np.uint32)
    p = u.view(np.float32)
    m = np.full(n, 1e-4, np.float32)
    got, want = _step(np.zeros(n, np.float32), p, m, m * m, 2, _hp(0.9, 0.95, lr=1e-3))
    assert_parity(got, want, "NaN weights")
    c = got["p16"][at]
    assert np.all((c & 0x7FFF) == 0x7FC0)
    assert np.array_equal(c >> 15, got["p"].view(np.uint32)[at] >> 31)
