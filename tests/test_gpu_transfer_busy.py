"""Fields moved while large kernels of another stream hold the device: the
same values, through the same calls, in a time that does not grow by one such
kernel for every chunk."""
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


@pytest.fixture(scope="module")
def products():
    """products(): enqueue 0.2 s of matrix products; its time per product."""
    import torch

    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    side = torch.cuda.Stream()

    def run(n):
        with torch.cuda.stream(side):
            for _ in range(n):
                torch.mm(a, a)
        return side

    torch.cuda.synchronize()
    run(20).synchronize()
    t = time.perf_counter()
    run(40).synchronize()
    each = (time.perf_counter() - t) / 40
    return lambda: run(int(0.2 / each)), each


# moments: 3, 9 and 28 chunks; populations: 20, 61 and 193 (four threads)
SHAPES = [(40, 64, 128), (64, 128, 144), (130, 128, 220)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage", ["fp32", "fp16s"])
def test_fields_beside_other_kernels(capi, products, shape, storage):
    print(f"[gpu] fields beside products {shape} {storage}", flush=True)
    rng = np.random.default_rng(1)
    rho = rng.uniform(0.98, 1.02, shape).astype(np.float32)
    u = (0.04 * rng.uniform(-1, 1, (3,) + shape)).astype(np.float32)
    ref, got = (capi.Domain(np.zeros(shape, np.uint8), periodic=7, storage=storage) for _ in range(2))
    for given in ((rho, u), (rho, None), (None, u)):
        ref.init_fields(*given)
        ref.step(3)
        want = ref.moments(), ref.populations()
        side = products[0]()
        got.init_fields(*given)
        side.synchronize()
        got.step(3)
        side = products[0]()
        rho1, u1 = got.moments()
        f1 = got.populations()
        side.synchronize()
        assert np.array_equal(rho1, want[0][0]) and np.array_equal(u1, want[0][1])
        assert np.array_equal(f1, want[1])
    other = np.ascontiguousarray(f1[:, :, ::-1])
    side = products[0]()
    got.set_populations(other)
    side.synchronize()
    ref.set_populations(other)
    assert np.array_equal(got.populations(), ref.populations())
    assert got.step_status(2) == ref.step_status(2) == capi.OK
    assert np.array_equal(got.populations(), ref.populations())
    ref.destroy()
    got.destroy()


def test_without_a_device_buffer(capi, products):
    """The buffer refused in every size: chunk by chunk after all."""
    print("[gpu] fields beside products, no device buffer", flush=True)
    shape = (64, 64, 64)
    f = I.random_populations(shape, 2).astype(np.float32)
    d = capi.Domain(np.zeros(shape, np.uint8), periodic=7)
    for refused in range(1, 12):
        d.init_fields()
        side = products[0]()
        capi.check(capi.lbm_debug_fail_after(refused))
        try:
            d.set_populations(f)
            failed = None
        except capi.LbmError as e:
            failed = e.code
        capi.check(capi.lbm_debug_fail_after(0))
        side.synchronize()
        assert failed in (None, capi.ERR_OOM, capi.ERR_DEVICE)
        if failed is None:
            assert np.array_equal(d.populations(), f)
            assert d.step_status(1) == capi.OK
        elif failed == capi.ERR_OOM and refused == 1:
            assert d.step_status(1) == capi.OK
    d.destroy()


def test_time_beside_other_kernels(capi, products):
    print("[gpu] time beside products", flush=True)
    run, each = products
    d = capi.Domain(I.periodic_box(64), periodic=7)
    f = d.populations()
    calls = {"populations": d.populations, "set_populations": lambda: d.set_populations(f)}
    for name, fn in calls.items():
        alone, beside = [], []
        for _ in range(5):
            t = time.perf_counter()
            fn()
            alone.append(time.perf_counter() - t)
            side = run()
            time.sleep(0.003)
            t = time.perf_counter()
            fn()
            beside.append(time.perf_counter() - t)
            side.synchronize()
        # 14 chunks: one by one they wait for 14 products
        assert np.median(beside) <= 2 * np.median(alone) + 6 * each, (name, alone, beside, each)
    d.destroy()
