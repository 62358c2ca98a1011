"""The camera array of the binding: sizes that are no numbers are refused as int() refuses them."""
import numpy as np
import pytest

from paper_2409_08270_amd import _lib as L


@pytest.mark.parametrize("size,error", [(np.nan, ValueError), (np.inf, OverflowError), (-np.inf, OverflowError)])
@pytest.mark.parametrize("col", [16, 17])
def test_sizes_must_be_numbers(size, error, col):
    rows = np.ones((3, 18), np.float32)
    rows[1, col] = size
    with pytest.raises(error):
        L.cameras(rows)
    with pytest.raises(error):
        int(float(rows[1, col]))
