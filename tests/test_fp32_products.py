"""The arithmetic of fp32 contractions, emulated: what the bound of tests/fp32_products.py lets pass and what it does not."""
import numpy as np
import pytest

from tests import fp32_products as F

# scales of the two operands: ordinary, small, smallest normal, subnormal (2^-130 and 2^-140, with results that are normal)
SCALES = [(1.0, 1.0), (1e-34, 1.0), (1.0, 1e-36), (1.2e-38, 1.0), (7e-40, 1e20), (7e-43, 1e22), (1e-19, 1e-15)]


def _operands(K, scales):
    rng = np.random.default_rng(K)
    return (rng.normal(size=(64, K)) * scales[0]).astype(np.float32), (rng.normal(0, 0.05, (K, 64)) * scales[1]).astype(np.float32)


@pytest.mark.parametrize("K", [64, 256, 1024])
@pytest.mark.parametrize("scales", SCALES)
def test_products_of_parts_are_no_less_accurate_than_a_chain(K, scales):
    a, b = _operands(K, scales)
    ref, bound = F.reference(a, b)
    assert F.rel(F.split_product(a, b), ref) <= 0.5 * bound


@pytest.mark.parametrize("K", [64, 256, 1024])
def test_the_bound_tells_a_missing_product_and_a_missing_scale(K):
    a, b = _operands(K, (1.0, 1.0))
    ref, bound = F.reference(a, b)
    for left_out in F.SMALL:
        assert F.rel(F.split_product(a, b, small=[p for p in F.SMALL if p != left_out]), ref) > 3 * bound
    for scales in SCALES[2:6]:
        a, b = _operands(K, scales)
        ref, bound = F.reference(a, b)
        assert F.rel(F.split_product(a, b, scale=1.0), ref) > 3 * bound


def test_columns_are_the_oracle_s_convolutions():
    import oracle as O
    rng = np.random.default_rng(2)
    big, small, w = rng.normal(size=(2, 6, 6, 3)), rng.normal(size=(2, 3, 3, 5)), rng.normal(size=(4, 4, 3, 5))
    ref = O.conv2d(big.transpose(0, 3, 1, 2), w.transpose(3, 2, 0, 1), None).transpose(0, 2, 3, 1)
    np.testing.assert_allclose(F.columns_down(big) @ w.reshape(48, 5), ref.reshape(-1, 5), rtol=1e-12, atol=1e-12)
    ref = O.conv_transpose2d(small.transpose(0, 3, 1, 2), w.transpose(3, 2, 0, 1), None).transpose(0, 2, 3, 1)
    np.testing.assert_allclose(F.columns_up(small) @ w.reshape(16, 3, 5).transpose(0, 2, 1).reshape(80, 3), ref.reshape(-1, 3), rtol=1e-12, atol=1e-12)
