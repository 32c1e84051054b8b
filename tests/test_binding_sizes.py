"""Sizes the binding works out for itself: payload bounds of a set of layers against anszp_pack_bound layer by layer, and
the job array against one filled record by record; what does not fit a field is refused."""
import ctypes as C

import numpy as np
import pytest

from paper_2406_06237_amd import binding as B


@pytest.mark.parametrize("table_log,n_streams", [(1, 1), (9, 17), (12, 64)])
def test_bounds_and_jobs_of_a_set(table_log, n_streams):
    sizes = [0, 1, 31, 32, 33, 65536, 65537, 2359296, (1 << 33) + 7, 5]
    chunks = [1, 1, 16, 7, 64, 65536, 65536, 1000, 262144, (1 << 32) - 1]
    bound = first = chunk = 0
    jobs = B.pack_jobs(sizes, chunks)
    for i, (n, c) in enumerate(zip(sizes, chunks)):
        nc, words = C.c_uint64(), C.c_uint64()
        assert B.lib().anszp_pack_bound(n, table_log, n_streams, c, C.byref(nc), C.byref(words)) == 0
        bound += words.value
        want = np.zeros(1, dtype=B.JOB_DTYPE)
        want[0] = (first, n, c, chunk, (0, 0))
        assert jobs[i:i + 1].tobytes() == want.tobytes()
        first += n
        chunk += nc.value
    assert B._pack_bound_words(sizes, chunks, table_log, n_streams) == bound
    assert len(B.pack_jobs([], [])) == 0


def test_sizes_of_layers_that_are_not_there():
    assert B.pack_jobs([5, 6], [2, 3, 0, -1]).tobytes() == B.pack_jobs([5, 6], [2, 3]).tobytes()
    assert B.pack_jobs([5, 6], iter([2, 3])).tobytes() == B.pack_jobs([5, 6], [2, 3]).tobytes()
    assert len(B.pack_jobs([], [7])) == 0


def test_what_a_field_cannot_hold_is_refused():
    for sizes, chunks, error in (([-1], [4], OverflowError), ([4], [-4], OverflowError), ([4], [1 << 32], OverflowError),
                                 ([1 << 33, 1], [1, 1], OverflowError), ([4], [0], ZeroDivisionError)):
        with pytest.raises(error):
            B.pack_jobs(sizes, chunks)
