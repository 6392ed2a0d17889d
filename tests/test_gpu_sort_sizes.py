"""The item sort's partition sizes (2048, 4096 and 8192 items), at the edges of
the rule that picks them and of a partition, against the oracle."""
import math

import pytest

import scenes as S
from test_gpu_binning import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views", [
    (10_240, 1), (10_241, 1), (12_289, 3),    # 2048: full partitions, one item more
    (131_072, 1), (131_073, 1),               # 64 partitions of 2048 in a view, 33 of 4096
    (16_384, 32), (16_385, 28),               # 256 of 2048 in all, 140 of 4096
    (16_384, 33), (32_769, 28),               # 132 of 4096, 252 of 4096
    (32_769, 29),                             # 261 of 4096: 145 of 8192
    (524_288, 1), (524_289, 1),               # 128 of 4096 in a view, 65 of 8192
])
def test_sizes(n, views):
    g = S.gaussians(n, math.log(0.1 * n ** (-1 / 3)), 0.3, 740 + n % 97)
    _check(g, [0.2 + 0.19 * k for k in range(views)], [(40, 24)] * views, 16, f"{n} items, {views} views", sample=4)
