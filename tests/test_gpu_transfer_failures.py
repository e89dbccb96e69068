"""Transfers that fail (forced from the host with lbm_debug_fail_after): a
lack of pinned memory changes nothing, or costs a large transfer some of its
threads; a state that was replaced in part is not stepped on silently, and is
left by the next initialisation."""
import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def make(capi, n, seed=1):
    d = capi.Domain(I.periodic_box(n), periodic=7)
    d.set_params(0.6)
    rng = np.random.default_rng(seed)
    u = (0.04 * rng.uniform(-1, 1, (3, n, n, n))).astype(np.float32)
    d.init_fields(None, u)
    return d, u


def code(capi, step, fn):
    """Error code of a call whose step-th fallible step fails."""
    capi.check(capi.lbm_debug_fail_after(step))
    try:
        fn()
    except capi.LbmError as e:
        return e.code
    finally:
        capi.check(capi.lbm_debug_fail_after(0))
    return capi.OK


@pytest.mark.parametrize("call", ["init_fields", "set_populations", "load_state"])
@pytest.mark.parametrize("steps", [2, 3])
def test_replacing_the_state(capi, call, steps):
    print(f"[gpu] failing {call} after {steps} steps", flush=True)
    n = 33  # two chunks of populations
    d, u = make(capi, n)
    f, image = d.populations(), d.save_state()
    d.step(steps)
    before = d.save_state()
    new = {"init_fields": lambda: d.init_fields(None, u), "set_populations": lambda: d.set_populations(f),
           "load_state": lambda: d.load_state(image)}[call]
    assert code(capi, 1, new) == capi.ERR_OOM
    assert np.array_equal(d.save_state(), before)
    assert d.step_status(1) == capi.OK
    d.load_state(before)
    assert code(capi, 2, new) == capi.ERR_DEVICE
    # (before the first chunk: the state is still whole)
    assert np.array_equal(d.save_state(), before)
    if call != "init_fields":  # its fields are one chunk
        assert code(capi, 3, new) == capi.ERR_DEVICE
        assert d.step_status(1) == capi.ERR_UNSTABLE
        d.init_fields()
        assert d.step_status(1) == capi.OK
    new()
    want = {"init_fields": make(capi, n)[0].populations(), "set_populations": f, "load_state": f}[call]
    assert np.array_equal(d.populations(), want)
    assert d.step_status(2) == capi.OK
    d.destroy()


def test_reading_the_state(capi):
    print("[gpu] failing read-backs", flush=True)
    d, _ = make(capi, 33)
    d.stats_enable()
    d.step(3)
    want = d.moments(), d.populations(), d.save_state(), d.stats()
    for fn in (d.moments, d.populations, d.save_state, d.stats):
        assert code(capi, 1, fn) == capi.ERR_OOM
        assert code(capi, 2, fn) == capi.ERR_DEVICE
    assert np.array_equal(d.moments()[1], want[0][1]) and np.array_equal(d.populations(), want[1])
    assert np.array_equal(d.save_state(), want[2]) and np.array_equal(d.stats()[2], want[3][2])
    assert d.step_status(1) == capi.OK
    d.destroy()


@pytest.mark.parametrize("refused", [2, 3, 4])
def test_fewer_threads(capi, refused):
    """Enough data for four threads, and no pinned memory for some of them."""
    print(f"[gpu] transfers with {refused - 1} threads", flush=True)
    d, _ = make(capi, 72)
    f = d.populations()
    got = []
    assert code(capi, refused, lambda: got.append(d.populations())) == capi.OK
    assert np.array_equal(got[0], f)
    other = np.ascontiguousarray(f[:, ::-1])
    assert code(capi, refused, lambda: d.set_populations(other)) == capi.OK
    assert np.array_equal(d.populations(), other)
    d.destroy()
