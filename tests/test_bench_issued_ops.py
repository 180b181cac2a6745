"""bench.py's counts of what the kernels issue, on the CPU: the digit products of
the transform's multiply against a walk over its columns, the additions of each
butterfly form, and vmul's and axpy's products on both sides of their lines."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

RATES = {k: bench.PEAK_INT_OPS for k in ("add_u32", "add_co_addc_u32", "mad_u64_u32", "mul_lo_u32", "mul_hi_u32")}
RATES["mad_addc_u32"] = 2 * bench.PEAK_INT_OPS  # (a product with its carry step then costs 1)


@pytest.mark.parametrize("L", [2, 4, 8, 10, 12, 20, 24, 28, 29, 32])
@pytest.mark.parametrize("full", [False, True])
def test_twiddle_multiply(L, full):
    b, D = bench.digits_of(L, full)
    assert b * D >= 32 * L - (0 if full else 1) > b * (D - 1)
    quot = sum(1 for c in range(D - 2, 2 * D - 1) for j in range(D) if 0 <= c - j < D)
    low = sum(1 for c in range(D) for j in range(c + 1))
    n = bench.product_counts(L, full)
    assert n["schoolbook"] == quot + 2 * low == 3 * D * (D + 1) // 2 + D - 1
    h = (D + 1) // 2
    z0 = sum(1 for c in range(min(2 * h - 1, D)) for i in range(h) if 0 <= c - i < h)
    cross = sum(1 + (i < D - h and c - i < D - h) for c in range(D) if c + h < D for i in range(c + 1))
    assert n["karatsuba"] == quot + z0 + cross + low
    assert bench.product_counts(8)["schoolbook"] == 143


def test_additions_follow_the_butterfly_form():
    adds = lambda *a, **k: bench.issued_butterfly_ops(*a, RATES, **k)["add_class_ops"]
    assert adds(8, 2, False) == 16 and adds(8, 1, False) == 40 and adds(5, 2, False) == 25
    assert adds(20, 1, False) == 40 and adds(19, 1, False) == 95 and adds(20, 1, True) == 100
    assert adds(10, 2, False) == 50  # the digits of 10 limbs fall short of 320 bits
    assert adds(8, 2, False, full=True) == 64


def test_elementwise_products():
    assert bench.blas_slots("vmul", 4, RATES) == pytest.approx(2 * 16 + 10 + 12)
    D = bench.digits_of(5)[1]
    assert bench.blas_slots("vmul", 5, RATES) == pytest.approx(2 * D * D + 2 * D + 8 * D + 15)
    assert bench.blas_slots("axpy", 3, RATES) == pytest.approx(21 + 15)
    D = bench.digits_of(4)[1]
    assert bench.blas_slots("axpy", 4, RATES) == pytest.approx(bench.product_counts(4)["schoolbook"] + 2 * (2 * D + 1) + 20)
