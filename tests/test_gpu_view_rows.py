"""The one-workgroup item sort's share of rows for each wavefront (16 of them,
rows of 64 items): every number of rows from one to eight per wavefront, full,
one item short and one over, against the oracle."""
import math

import pytest

import scenes as S
from test_gpu_binning import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 65, 1023, 1024, 1025, 2048, 2049, 3072, 3073, 5120, 5121, 7168, 7169])
def test_rows(n):
    g = S.gaussians(n, math.log(0.4 * n ** (-1 / 3)), 0.3, 730 + n % 97)
    _check(g, [0.2, 1.3], [(64, 48), (33, 40)], 16, f"{n} items")
