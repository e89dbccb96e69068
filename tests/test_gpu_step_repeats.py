"""Runs of 64 to 255 steps made over and over replay the step graph too, once
256 steps have been asked for since the last change: they take the host no
longer than with the graph built beforehand, and end bit for bit where single
steps end."""
import time

import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def make(capi, n=24):
    d = capi.Domain(I.periodic_box(n), periodic=7)
    d.set_params(0.6)
    d.init_fields(None, I.taylor_green_velocity(n, n, n, 0.03).astype(np.float32))
    return d


@pytest.mark.parametrize("runs", [(100,) * 5, (64,) * 6, (63,) * 6 + (64, 65), (255, 65, 1, 64), (65, 1) * 5])
def test_repeated_runs_equal_single_steps(capi, runs):
    print(f"[gpu] repeated runs {runs}", flush=True)
    got, ref = make(capi), make(capi)
    for tau in (0.6, 0.7):  # a change starts the count again
        got.set_params(tau)
        ref.set_params(tau)
        for n in runs:
            got.step(n)
            for _ in range(n):
                ref.step_async(1)
            assert ref.wait_status() == capi.OK
        assert np.array_equal(got.populations(), ref.populations())
    got.destroy()
    ref.destroy()


def test_repeated_runs_replay_the_graph(capi):
    print("[gpu] host time of repeated runs", flush=True)
    took = {}
    for prepared in (True, False):
        d = make(capi)
        if prepared:
            d.prepare_steps()
        for _ in range(8):
            t = time.perf_counter()
            for _ in range(8):
                d.step_async(64)
            took[prepared] = min(took.get(prepared, 1e9), time.perf_counter() - t)
            assert d.wait_status() == capi.OK
        d.destroy()
    # launched one by one they take the host three times as long
    assert took[False] <= 1.7 * took[True], took
