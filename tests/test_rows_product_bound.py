"""The bound by which the k-means build decides that a point's nearest centre is known from the keys alone, against a model
of the product's arithmetic: values split into two bf16 each, three matrix instructions per 32 values, each of which takes
its products in four groups of eight (what lies under 2^-24 of the largest product cut off) with one rounding of the fp32
accumulator per group.  Rows on which the roundings do not cancel are the ones that matter: equal values, equal values with
gaps, signs that alternate, one value that outweighs the others."""
import numpy as np
import pytest


def _bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).view(np.float32)


def _split(x):
    hi = _bf16(x)
    return hi, _bf16(x - hi)


def _product(q, c, chain):
    """sum over d of q c as the kernel forms it: q, c [pairs, d] fp32; a new sum every `chain` k-steps of 32 values."""
    (qh, ql), (ch, cl) = _split(q), _split(c)
    pairs, d = q.shape
    total = np.zeros(pairs, np.float32)
    for k0 in range(0, d // 32, chain):
        acc = np.zeros(pairs, np.float32)
        for k in range(k0, min(k0 + chain, d // 32)):
            for a, b in ((qh, ch), (qh, cl), (ql, ch)):
                for g in range(32 * k, 32 * k + 32, 8):
                    x, y = a[:, g:g + 8].astype(np.float64), b[:, g:g + 8].astype(np.float64)
                    p = x * y
                    e = np.frexp(np.abs(p).max(1))[1] - 1                 # the largest product is in [2^e, 2^(e + 1))
                    lsb = np.exp2(np.maximum(e, -900) - 24.0)[:, None]
                    acc = (acc + (np.trunc(p / lsb) * lsb).sum(1)).astype(np.float32)
        total = total + acc
    return total


def _key_error(nk, chain, slots):
    """key_error of the kernel's source."""
    return (3.1e-5 + 5.97e-8 * (12.0 * min(chain, nk) + slots + 12.0)) * (1.0 + 5.97e-8 * 8.0 * nk)


def _independent(nk):
    """An allowance that takes the roundings as independent: eight times the root of their number."""
    return 3.1e-5 + 5.96e-8 * (16.0 + 8.0 * np.sqrt(3.0 * nk))


def _rows(kind, pairs, d, rng):
    q, c = 0.5 + 1.5 * rng.random((pairs, 1)), 0.5 + 1.5 * rng.random((pairs, 1))
    one = np.ones((1, d))
    if kind == "gaps":
        one = np.where(np.arange(d) // 512 % 2 == 0, 1.0, 0.0625)[None]
    if kind == "relu":
        return (np.maximum(rng.standard_normal((pairs, d)), 0.0).astype(np.float32), np.maximum(rng.standard_normal((pairs, d)), 0.0).astype(np.float32))
    q, c = q * one, c * one
    if kind == "alternating":
        q, c = q * np.where(np.arange(d) % 2, -1.0, 1.0), c * np.where(np.arange(d) % 2, -1.0, 1.0)
    if kind == "large first":
        q[:, 0], c[:, 0] = 300.0, 300.0
    return q.astype(np.float32), c.astype(np.float32)


@pytest.mark.parametrize("kind", ["constant", "gaps", "relu", "alternating", "large first"])
@pytest.mark.parametrize("d,chain", [(32768, 1024), (8192, 196), (32768, 100)])
def test_bound_holds(kind, d, chain):
    rng = np.random.default_rng(d + chain)
    q, c = _rows(kind, 48, d, rng)
    nk = d // 32
    q64, c64 = q.astype(np.float64), c.astype(np.float64)
    norms = np.sqrt((q64 * q64).sum(1) * (c64 * c64).sum(1))
    err = np.abs(_product(q, c, chain).astype(np.float64) - (q64 * c64).sum(1)) / norms
    assert err.max() <= _key_error(nk, chain, -(-nk // chain)), err.max()
    if kind == "constant" and chain == nk:
        # the roundings do add up here: their root would not have done
        assert err.max() > _independent(nk), err.max()
