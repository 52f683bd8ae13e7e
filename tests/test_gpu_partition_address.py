"""The allocation-free compaction of codes that begin at any address: against numpy's
stable partition around the edges of its blocks and of one launch, between bytes that
are no codes; and the time of an odd address beside that of an aligned one."""
import time

import numpy as np
import pytest

from gvtest import stable_partition_reference
from test_zz_no_alloc import _Hip

pytestmark = pytest.mark.gpu


def _call(gv, hip, host, off, n):
    buf, index, counts = hip.put(host), hip.put(np.full(9 * n, -7, np.int32)), hip.put(np.full(4, 9, np.uint32))
    gv.compact3_noalloc(buf + off, n, 256, index, counts, None)
    assert hip.lib.hipDeviceSynchronize() == 0
    out = hip.get(index, np.int32, 9 * n).reshape(3, -1), hip.get(counts, np.uint32, 4)
    hip.free(buf, index, counts)
    return out


@pytest.mark.parametrize("off", [1, 2, 3, 4, 6, 8, 13])
def test_codes_at_any_address(off):
    import paper_2005_00949_amd as gv
    gv.load()
    hip = _Hip()
    rng = np.random.default_rng(off)
    for n in (1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 18, 255, 1023, 1024, 1025, 1026, 4099, 8191, 8192, 8193, 100003,
              (1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 17):
        codes = rng.integers(-1, 3, 3 * n).astype(np.int8)
        host = np.full(3 * n + 64, 77, dtype=np.int8)      # 77 is no code: it would be counted as an error
        host[off:off + 3 * n] = codes
        index, counts = _call(gv, hip, host, off, n)
        assert counts[3] == 0, n
        if n <= 100003:
            want = stable_partition_reference(codes)
        else:
            at = [np.flatnonzero(codes == q) for q in range(3)]
            want = [(a // 3 * 4 + a % 3).astype(np.int32) for a in at]
        for q in range(3):
            assert counts[q] == len(want[q]) and np.array_equal(index[q, :counts[q]], want[q]), (n, q)


@pytest.mark.parametrize("n", [5000, 8192])
def test_an_odd_address_costs_no_more(n):
    """A word more to load and a shift per word, of a call that is bound by its launch;
    byte loads took 1.4 and 1.6 times as long."""
    import paper_2005_00949_amd as gv
    gv.load()
    hip = _Hip()
    buf, index, counts = (hip.put(np.zeros(k, np.int8)) for k in (3 * n + 64, 36 * n, 16))
    us = {}
    for off in (0, 1):
        best = 1e9
        for _ in range(10):
            assert hip.lib.hipDeviceSynchronize() == 0
            t = time.perf_counter()
            for _ in range(100):
                gv.compact3_noalloc(buf + off, n, 256, index, counts)
            assert hip.lib.hipDeviceSynchronize() == 0
            best = min(best, (time.perf_counter() - t) * 1e4)
        us[off] = best
    hip.free(buf, index, counts)
    print(f"\n{n} inputs: {us[0]:.2f} us aligned, {us[1]:.2f} us at an odd address")
    assert us[1] < 1.25 * us[0]
