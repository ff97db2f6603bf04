"""The encoders' division, step by step as the kernels form it but on the CPU: the reciprocal a little above 1/f (over_reciprocal
and encode_record in csrc/), and the quotient as the low word of a double.  Every mass, with the single-precision reciprocal
off by up to two units either way (the instruction promises one), under states at both ends of the multiples of the mass."""
import numpy as np
import pytest

MASSES = np.arange(1, (1 << 16) - 255 + 1, dtype=np.int64)  # the largest mass is 2^16 - 255


def _single_reciprocal(units):
    """1/f in single precision, `units` last places off."""
    nearest = (np.float32(1.0) / MASSES.astype(np.float32)).view(np.int32)
    return (nearest + np.int32(units)).view(np.float32).astype(np.float64)


def _newton(r0, target):
    """fma(r0, fma(-f, r0, target), r0) with one rounding.  Plain double precision gives it: r0 has 24 bits and f 16, so f r0
    is exact, the difference has at most 20 bits, its product with r0 at most 44, and only the last sum is rounded."""
    return r0 * (target - MASSES * r0) + r0


def _over_reciprocal(units):
    return _newton(_single_reciprocal(units), 1.0 + 2.0**-35)


def _record_reciprocal(units, cum):
    """encode_record's, of which the lowest 16 bits are the symbol's cum (times 2^1022 there, which changes only the exponent)."""
    r = _newton(_single_reciprocal(units), 1.0) * (1.0 + 2.0**-35)
    return ((r.view(np.uint64) & np.uint64(0xFFFFFFFFFFFF0000)) | np.uint64(cum)).view(np.float64)


def _times(s, r):
    """floor(s r) and whether s r is whole, exactly (s below 2^32)."""
    m, e = np.frexp(r)
    m = np.ldexp(m, 53).astype(np.uint64)  # r = m 2^(e - 53), m of 53 bits
    shift = (53 - e).astype(np.uint64)
    s = s.astype(np.uint64)
    low27 = np.uint64((1 << 27) - 1)
    low = s * (m & low27)
    high = s * (m >> np.uint64(27)) + (low >> np.uint64(27))  # s m = high 2^27 + (low mod 2^27)
    shift -= np.uint64(27)
    whole = ((high & ((np.uint64(1) << shift) - np.uint64(1))) | (low & low27)) == 0
    return (high >> shift).astype(np.int64), whole


def _states():
    """The states f q - 1, f q and f q + f - 1 of the smallest, a middle and the largest quotients below 2^32 / f."""
    most = ((1 << 32) - 1) // MASSES
    for q in (np.ones_like(MASSES), np.full_like(MASSES, 2), (most + 1) // 2, most - 1, most):
        for s in (MASSES * q - 1, MASSES * q, MASSES * q + MASSES - 1):
            yield np.clip(s, MASSES, (1 << 32) - 1)
    yield np.full_like(MASSES, (1 << 32) - 1)


@pytest.mark.parametrize("units", [-2, -1, 0, 1, 2])
@pytest.mark.parametrize("form", ["nearest", 0, 0xFFFF])
def test_quotient_of_every_mass(form, units):
    # "nearest": s r + 2^52 - 1/2 rounded to the nearest whole number is 2^52 + floor(s r) unless s r is whole; otherwise
    # 1 + s r 2^-52 rounded towards zero, which is floor(s r) as it stands.  r is above 1/f, so s r is no multiple's own.
    r = _over_reciprocal(units) if form == "nearest" else _record_reciprocal(units, form)
    for s in _states():
        q, whole = _times(s, r)
        assert np.array_equal(q, s // MASSES)
        if form == "nearest":
            assert not whole.any()


def test_a_reciprocal_that_is_not_above_fails_it():
    r = _newton(_single_reciprocal(0), 1.0)
    assert any(not np.array_equal(_times(s, r)[0], s // MASSES) for s in _states())
