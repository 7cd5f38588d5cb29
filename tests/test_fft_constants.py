"""The twiddle constants of the register DFTs (csrc/mm_fft.hpp), no GPU: every one is the double
nearest to the cosine or sine it stands for, from 45-digit series."""
import os
import re
from decimal import Decimal, getcontext

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = open(os.path.join(ROOT, "paper_1501_07293_amd", "csrc", "mm_fft.hpp")).read()
PI = Decimal("3.14159265358979323846264338327950288419716939937510")


def series(x, first):
    getcontext().prec = 45
    term = total = Decimal(1) if first == 0 else x
    n = first
    while abs(term) > Decimal(10) ** -44:
        n += 2
        term = -term * x * x / (n * (n - 1))
        total += term
    return total


def root(j, n):
    """exp(-2 pi i j / n) as doubles."""
    getcontext().prec = 45
    a = 2 * PI * j / n
    return float(series(a, 0)), -float(series(a, 1))


def test_every_constant_is_a_nearest_double():
    exact = {abs(v) for n in (3, 5, 7, 8, 9, 16, 25, 32) for j in range(n) for v in root(j, n)}
    written = {abs(float(v)) for v in re.findall(r"-?0\.\d{10,}", SRC)}
    assert len(written) > 30
    assert sorted(written - exact) == []


@pytest.mark.parametrize("j", [1, 2, 3, 4, 6, 8, 9, 12, 16])
def test_twiddles_of_25_points(j):
    body = SRC[SRC.index("w25(int j)"):]
    label = "default" if j == 16 else rf"case {j}"
    re_, im = re.search(label + r": return \{\(T\)([-\d.]+), \(T\)([-\d.]+)\}", body).groups()
    assert (float(re_), float(im)) == root(j, 25)
