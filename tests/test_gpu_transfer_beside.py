"""Transfers of different domains run side by side: a small read-back does not
wait for a large one to end, and more callers than there are pinned buffers
(16 pairs a device) all get their own values."""
import threading
import time

import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def test_small_beside_large(capi):
    print("[gpu] a small read-back beside a large one", flush=True)
    large, small = capi.Domain(I.periodic_box(160), periodic=7), capi.Domain(I.periodic_box(16), periodic=7)
    buf = np.zeros((27, 160, 160, 160), np.float32)  # 442 MB
    exports, waits, stop = [], [], threading.Event()

    def export():
        while not stop.is_set():
            t = time.perf_counter()
            capi.check(capi.lbm_get_populations(large.h, buf.ctypes.data_as(capi._fp)))
            exports.append(time.perf_counter() - t)

    small.moments()
    th = threading.Thread(target=export)
    th.start()
    while len(exports) < 2:
        time.sleep(0.01)
    for _ in range(40):
        t = time.perf_counter()
        small.moments()
        waits.append(time.perf_counter() - t)
    stop.set()
    th.join()
    large.destroy()
    small.destroy()
    # taking turns, the small one waits for a whole export at the median
    assert np.median(waits) <= 0.25 * np.median(exports), (np.median(waits), np.median(exports))


def test_more_callers_than_buffers(capi):
    print("[gpu] transfers from 24 threads", flush=True)
    shape, bad, start = (24, 64, 96), [], threading.Barrier(24)

    def work(seed):
        rng = np.random.default_rng(seed)
        u = (0.04 * rng.uniform(-1, 1, (3,) + shape)).astype(np.float32)
        d = capi.Domain(np.zeros(shape, np.uint8), periodic=7)
        d.init_fields(None, u)
        f = d.populations()
        start.wait()
        for _ in range(3):
            d.set_populations(f)
            if not np.array_equal(d.populations(), f) or np.abs(d.moments()[1] - u).max() > 4e-6:
                bad.append(seed)
        d.destroy()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(24)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
