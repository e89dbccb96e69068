"""Destroying a domain does not wait for other work on the device, also not the
last one and after a transfer large enough for several pinned buffers; those
are given back when a batch is destroyed."""
import time

import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def test_destroy_beside_other_work(capi):
    import torch

    print("[gpu] destroy beside other work", flush=True)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    side = torch.cuda.Stream()

    def products(n):
        with torch.cuda.stream(side):
            for _ in range(n):
                torch.mm(a, a)
        done = torch.cuda.Event()
        done.record(side)
        return done

    torch.cuda.synchronize()
    products(40).synchronize()
    t = time.perf_counter()
    products(40).synchronize()
    each = (time.perf_counter() - t) / 40
    beside = []
    # a stream may share a hardware queue with the other work and then waits
    # for it in any case: not every one of eight does
    for stream in [torch.cuda.Stream() for _ in range(8)]:
        d = capi.Domain(I.periodic_box(80), periodic=7, stream=stream.cuda_stream)
        d.populations()  # 55 MB
        done = products(int(0.25 / each))  # a quarter of a second of them
        d.destroy()
        beside.append(not done.query())
        done.synchronize()
        if beside[-1]:
            break
    assert any(beside)


def test_a_destroyed_batch_gives_pinned_memory_back(capi):
    """... and what is left serves the transfers that follow."""
    print("[gpu] pinned memory given back", flush=True)
    for _ in range(2):
        d = capi.Domain(I.periodic_box(72), periodic=7)
        f = d.populations()
        many = [capi.Domain(I.periodic_box(4), periodic=7) for _ in range(1030)]
        b = capi.Batch(1 << 30, "fp32")
        b.destroy()
        for e in many:
            assert e.step_status(1) == capi.OK
            e.destroy()
        b = capi.Batch(1 << 30, "fp32")
        b.destroy()
        d.set_populations(f)
        assert np.array_equal(d.populations(), f)
        assert d.step_status(2) == capi.OK
        d.destroy()
