"""What the bound on fp32 products sees (CPU only): products formed from terms of 16 bits in numpy, as the matrix kernels
form them and as they must not."""
import numpy as np
import pytest

from gen import rng
from tests.harness import WEIGHT_PATTERNS, assert_product, patterned_weights


def bf16(x):
    """Round to nearest even, as fp32."""
    b = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return ((b + 0x7fff + (b >> 16 & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def terms(x, n, form):
    out, rest = [], x.astype(np.float32)
    for _ in range(n):
        t = bf16(rest) if form == "bf16" else rest.astype(np.float16).astype(np.float32)
        out.append(t)
        rest = rest - t
    return out


def product(a, b, pairs, form="bf16"):
    """fp32 accumulator, 16 k-values and one pair of terms per addition.  fp16: one power of two per row of a and column
    of b puts its largest element below 2^15."""
    ea = eb = np.zeros(1)
    if form == "fp16":
        ea, eb = (14 - np.floor(np.log2(np.maximum(np.abs(x).max(axis=axis, keepdims=True), 2.0 ** -100))) for x, axis in ((a, 1), (b, 0)))
        a, b = (a * np.exp2(ea)).astype(np.float32), (b * np.exp2(eb)).astype(np.float32)
    n = max(max(p) for p in pairs) + 1
    ta, tb = terms(a, n, form), terms(b, n, form)
    acc = np.zeros((a.shape[0], b.shape[1]), dtype=np.float32)
    for k in range(0, a.shape[1], 16):
        for i, j in pairs:
            acc = (acc + ta[i][:, k:k + 16].astype(np.float64) @ tb[j][k:k + 16].astype(np.float64)).astype(np.float32)
    return acc * np.exp2(-ea - eb)


def test_three_bf16_terms_are_the_value_and_six_products_all_but_2_to_the_minus_24_of_theirs():
    """Over every significand; the extremes of |m| and |l| bound what three of the nine products can hold."""
    x = (np.arange(1 << 23, dtype=np.uint32) | np.uint32(127 << 23)).view(np.float32)
    h, m, l = terms(x, 3, "bf16")
    assert np.array_equal(h.astype(np.float64) + m + l, x.astype(np.float64))
    m, l = np.abs(m / x), np.abs(l / x)
    assert m.max() <= 2.0 ** -8 and l.max() <= 2.0 ** -17
    assert 2 * m.max() * l.max() + l.max() ** 2 <= 2.0 ** -24


SIX = [(0, 0), (0, 1), (0, 2), (1, 0), (1, 1), (2, 0)]  # three bf16 terms per operand
THREE = [(0, 0), (0, 1), (1, 0)]                        # two terms per operand


def operands(kind):
    """The weight patterns; a weight gradient over many rows, and one whose rows with the largest features have no gradient."""
    g = rng.stream("tests", f"terms_{kind}")
    if kind in WEIGHT_PATTERNS:
        return g.standard_normal((300, 128)).astype(np.float32), patterned_weights(kind, 128, 96, g)
    n = 33001
    x, go = np.abs(g.standard_normal((n, 24))).astype(np.float32), g.standard_normal((n, 40)).astype(np.float32)
    if kind == "hub":
        x[100] *= 2.0 ** 30
        go[100] = 0.0
    return np.ascontiguousarray(x.T), go


@pytest.mark.parametrize("kind", WEIGHT_PATTERNS + ["rows", "hub"])
def test_six_products_of_three_bf16_terms_are_within_the_bound(kind):
    a, b = operands(kind)
    assert_product(product(a, b, SIX), [a], [b], kind)


@pytest.mark.parametrize("kind", WEIGHT_PATTERNS + ["rows", "hub"])
def test_leading_terms_alone_are_not(kind):
    a, b = operands(kind)
    with pytest.raises(AssertionError, match="of the bound"):
        assert_product(product(a, b, [(0, 0)]), [a], [b], kind)
    with pytest.raises(AssertionError, match="of the bound"):
        assert_product(product(a, b, [(0, 0)], "fp16"), [a], [b], kind)


@pytest.mark.parametrize("kind", WEIGHT_PATTERNS)  # (over 33,001 rows the accumulator rounds away as much)
def test_two_bf16_terms_are_not(kind):
    a, b = operands(kind)
    with pytest.raises(AssertionError, match="of the bound"):
        assert_product(product(a, b, THREE), [a], [b], kind)


def test_two_fp16_terms_do_not_hold_the_range():
    """Scaled by the largest element of their row, the other rows of a hub's column are below the last bit of two terms."""
    a, b = operands("hub")
    with pytest.raises(AssertionError, match="of the bound"):
        assert_product(product(a, b, THREE, "fp16"), [a], [b], "hub")
