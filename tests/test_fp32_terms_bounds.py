"""CPU check of the arithmetic behind fp32 products in three bf16 terms: what the six products keep, and that the line of the GPU test lies below what a
missing one would cost."""
import numpy as np
import pytest

ORDER = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]
GPU_LINE = 8e-7   # test_fp32_terms_hold_24_bits


def bf16(x):
    """fp32 values rounded to bf16 (to nearest, ties to even)."""
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000
    return u.astype(np.uint32).view(np.float32)


def terms(x):
    x = np.asarray(x, np.float32)
    t0 = bf16(x)
    t1 = bf16(x - t0)
    t2 = bf16(x - t0 - t1)
    return [t.astype(np.float64) for t in (t0, t1, t2)]


def test_three_terms_are_the_value():
    x = np.random.default_rng(1).standard_normal(200000).astype(np.float32)
    assert np.array_equal(sum(terms(x)), x.astype(np.float64))


def test_what_is_left_out_of_a_product():
    rng = np.random.default_rng(2)
    a, b = (rng.standard_normal(2000000).astype(np.float32) for _ in range(2))
    ta, tb = terms(a), terms(b)
    left = np.abs(sum(ta[i] * tb[j] for i, j in ((1, 2), (2, 1), (2, 2))) / (a.astype(np.float64) * b))
    assert 2. ** -28 < np.sqrt((left ** 2).mean()) < 2. ** -27 and left.max() <= 2. ** -24
    worst = np.float32(float.fromhex("0x1.00ff8p0"))   # (the bound is reached)
    t = terms(worst)
    assert 0.99 * 2. ** -24 < abs(t[1] * t[2] * 2 + t[2] * t[2]) <= 2. ** -24


@pytest.mark.parametrize("missing", ORDER[1:], ids=str)
def test_a_missing_product_shows(missing):
    rng = np.random.default_rng(3)
    q, k, v = (rng.standard_normal((n, 64)).astype(np.float32) for n in (64, 1024, 1024))
    tq, tk = terms(q), terms(k)

    def out(products):
        s = sum(tq[i] @ tk[j].T for i, j in products) * 0.125
        p = np.exp(s - s.max(1, keepdims=True))
        return p @ v.astype(np.float64) / p.sum(1, keepdims=True)

    want = out([(i, j) for i in range(3) for j in range(3)])
    err = lambda products: np.linalg.norm(out(products) - want) / np.linalg.norm(want)
    assert err(ORDER) < 0.1 * GPU_LINE
    assert err([p for p in ORDER if p != missing]) > 2 * GPU_LINE
