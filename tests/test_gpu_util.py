"""The helpers of the GPU tests."""
import numpy as np

from gpu_util import relmax


def test_a_row_that_is_not_finite_fails_a_bound_over_rows():
    ref = np.ones((3, 4), np.float32)
    for bad in (np.nan, np.inf):
        for row in range(3):
            got = ref.copy()
            got[row, 2] = bad
            assert not max(relmax(got[i], ref[i]) for i in range(3)) <= 1.0
    assert relmax(ref, ref) == 0.0
