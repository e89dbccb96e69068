"""The halfway rule everywhere, asked for again: at no cost where no wall
fractions are set, and back to the bits of a domain that never had any where
they are."""
import time

import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def test_nothing_to_reset_costs_nothing(capi):
    print("[gpu] halfway rule on a domain that has it", flush=True)
    d = capi.Domain(I.channel_flags(192, 192, 192), periodic=I.PERIODIC_X | I.PERIODIC_Z)
    took = []
    for _ in range(10):
        t = time.perf_counter()
        d.set_wall_distances(None)
        took.append(time.perf_counter() - t)
    d.destroy()
    # the tile list and link masks, fetched and sent back, take 0.7 ms
    assert min(took) <= 1e-4, took


@pytest.mark.parametrize("steps", [0, 3, 4])
@pytest.mark.parametrize("storage", ["fp32", "fp16s"])
def test_reset_gives_the_halfway_bits(capi, storage, steps):
    print(f"[gpu] halfway rule again after {steps} steps {storage}", flush=True)
    noz = I.Nozzle(n=20, length=70, R=9.5, r_throat=3.5, inlet_len=12, throat_len=20)
    flags = noz.flags()
    q = noz.wall_distances(flags).astype(np.float32)
    got, ref = (capi.Domain(flags, storage=storage) for _ in range(2))
    rng = np.random.default_rng(5)
    u = (0.02 * rng.uniform(-1, 1, (3,) + flags.shape)).astype(np.float32)
    for d in (got, ref):
        d.set_params(0.6)
        d.init_fields(None, u)
        d.step(steps)
    size = got.info().device_bytes
    got.set_wall_distances(q)
    assert got.info().device_bytes > size
    got.set_wall_distances(None)
    got.set_wall_distances(None)
    assert got.info().device_bytes == size
    for d in (got, ref):
        d.step(5)
    assert np.array_equal(got.populations(), ref.populations())
    got.destroy()
    ref.destroy()
