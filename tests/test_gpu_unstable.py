"""A run that goes unstable costs about what a stable one costs, though every
wave of every later step finds the state unstable; and a state that replaces
an unstable one starts clear, and is reported in its turn."""
import time

import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


@pytest.mark.parametrize("storage", ["fp32", "fp16s"])
def test_unstable_run_costs_what_a_stable_one_does(capi, storage):
    print(f"[gpu] unstable run {storage}", flush=True)
    n, steps = 96, 200
    d = capi.Domain(I.periodic_box(n), periodic=7, storage=storage)
    d.prepare_steps()
    took = {}
    for rho, want in ((1.0, capi.OK), (-1.0, capi.ERR_UNSTABLE)):
        for _ in range(3):
            d.init_fields(np.full((n, n, n), rho, np.float32))
            t = time.perf_counter()
            assert d.step_status(steps) == want
            took[want] = min(took.get(want, 1e9), time.perf_counter() - t)
    d.destroy()
    # a word written over PCIe by every wave of every step takes 70 times as long
    assert took[capi.ERR_UNSTABLE] <= 5.0 * took[capi.OK], took


@pytest.mark.parametrize("adopted", [False, True])
def test_new_states_start_clear(capi, adopted):
    import torch

    print(f"[gpu] new states, adopted {adopted}", flush=True)
    n = 12
    raw = torch.full((int(capi.lbm_array_bytes(n, n, n, 0)),), 255, dtype=torch.uint8, device="cuda")
    d = capi.Domain(I.periodic_box(n), periodic=7, array=raw.data_ptr() if adopted else None)
    assert d.step_status(3) == capi.OK
    image = d.save_state()
    bad = np.full((n, n, n), -1.0, np.float32)
    for replace in (lambda: d.init_fields(), lambda: d.load_state(image), lambda: d.init_fields(np.ones_like(bad))):
        d.init_fields(bad)
        assert d.step_status(2) == capi.ERR_UNSTABLE
        assert d.step_status(1) == capi.ERR_UNSTABLE  # sticky
        replace()
        assert d.step_status(5) == capi.OK
        # unstable steps that nobody waited for
        d.init_fields(bad)
        d.step_async(2)
        replace()
        assert d.step_status(4) == capi.OK
    d.destroy()
