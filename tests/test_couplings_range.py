"""Batch.get_couplings with a range outside the batch: IndexError, whatever the count (CPU: the
range is looked at before the library is called)."""
import numpy as np
import pytest

from paper_2011_08560_amd import nfm


@pytest.mark.parametrize("r0,count", [(3, 1), (0, 4), (2, 2), (-4, 1), (0, 2 ** 40), (-1, 2 ** 40)])
def test_range_outside_the_batch_is_an_index_error(r0, count):
    b = nfm.Batch.__new__(nfm.Batch)
    b.Ls = np.array([4, 6, 8], np.int32)
    with pytest.raises(IndexError):
        b.get_couplings(r0, count)
