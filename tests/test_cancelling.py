"""The inputs of tests/cancelling.py tell weights of 24 bits from weights of 16 and 8 (CPU only)."""
import numpy as np
import pytest

from tests import cancelling


@pytest.mark.parametrize("name", ["O", "dV", "dK", "dQ"])
def test_only_three_parts_of_a_weight_are_enough(name):
    sums = cancelling.inputs(64, 7)[-1]
    ref, bound = cancelling.expected(sums, name)
    worst = [float((np.abs(cancelling.with_parts(sums, name, k) - ref) / bound).max()) for k in (1, 2, 3)]
    print(name, worst)
    assert worst[2] <= 1.0 < worst[1] < worst[0]
