"""gv_compact3_noalloc at the sizes where its launches can go wrong: one
input, the edges of a thread's and a block's share (4 and 16 inputs, 1,024 and
4,096), both sides of the sizes where one launch becomes two (2^13) and where the
share changes (2^20), the largest call (2^24), and codes at addresses that rule
out wide loads.  Whole numbers, against
numpy: no tolerance."""
import ctypes as C

import numpy as np
import pytest

from test_zz_no_alloc import _Hip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 1025, 4096, 4097, 8191, 8192, 8193, 32769, 262145, (1 << 20) - 1,
                               1 << 20, (1 << 20) + 4097, (1 << 24) - 15, 1 << 24])
def test_queues_and_counts(n, offset):
    import paper_2005_00949_amd as gv
    if n > 1 << 21 and offset == 4:
        pytest.skip("the same branch as offset 1 at this size")
    gv.load()
    hip = _Hip()
    rng = np.random.default_rng(n + offset)
    codes = rng.integers(-1, 3, size=3 * n, dtype=np.int8)
    if n % 3 == 0:
        codes[: 3 * (n // 2)] = 1            # a run of one queue: blocks whose other counts are zero
    bad = n == 1025
    if bad:
        codes[-1], codes[5] = 3, -2          # dropped, and reported in counts[3]
    d_codes = hip.put(np.concatenate([np.zeros(offset, np.int8), codes]))
    d_index = hip.put(np.full(9 * n + 1, -7, dtype=np.int32))
    d_counts = hip.put(np.full(4, 99, dtype=np.uint32))
    gv.compact3_noalloc(d_codes + offset, n, 128, d_index, d_counts, None)
    assert hip.lib.hipDeviceSynchronize() == 0
    counts = hip.get(d_counts, np.uint32, 4)
    index = hip.get(d_index, np.int32, 9 * n + 1)
    hip.free(d_codes, d_index, d_counts)
    assert counts[3] == (4 if bad else 0)
    assert index[9 * n] == -7
    for q in range(3):
        at = np.flatnonzero(codes == q)
        want = (at // 3 * 4 + at % 3).astype(np.int32)
        got = index[3 * n * q : 3 * n * (q + 1)]
        assert counts[q] == len(want)
        assert np.array_equal(got[: len(want)], want)
        assert (got[len(want):] == -7).all()
