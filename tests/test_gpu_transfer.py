"""Fields through the chunked transfers: sizes around one chunk (2 MiB), an
odd number of chunks, and above the size from which several threads copy,
against the same values through the device (lbm_get_moments_device) and
through each other, and from several threads at once."""
import threading

import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def fields(shape, seed):
    rng = np.random.default_rng(seed)
    rho = rng.uniform(0.98, 1.02, shape).astype(np.float32)
    return rho, (0.04 * rng.uniform(-1, 1, (3,) + shape)).astype(np.float32)


# cells per chunk: 131072 of 16 bytes (moments), 19392 of 108 (populations)
SHAPES = [(1, 1, 1), (3, 7, 11), (1, 303, 64), (1, 303, 65), (8, 128, 128), (9, 127, 129), (41, 97, 131),
          (130, 128, 160)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("given", ["both", "rho", "u"])
def test_fields_in_and_out(capi, shape, given):
    import torch

    print(f"[gpu] fields {shape} {given}", flush=True)
    rho, u = fields(shape, 1)
    d = capi.Domain(np.zeros(shape, np.uint8), periodic=7)
    d.init_fields(rho if given != "u" else None, u if given != "rho" else None)
    rho1, u1 = d.moments()
    r2 = torch.empty(shape, dtype=torch.float32, device="cuda")
    u2 = torch.empty((3,) + shape, dtype=torch.float32, device="cuda")
    d.moments_device(r2.data_ptr(), u2.data_ptr())
    assert np.array_equal(rho1, r2.cpu().numpy()) and np.array_equal(u1, u2.cpu().numpy())
    # the moments of f^eq are its fields: 27 terms rounded to FP32 each way
    assert np.abs(rho1 - (rho if given != "u" else 1.0)).max() <= 4e-6
    assert np.abs(u1 - (u if given != "rho" else 0.0)).max() <= 4e-6
    f = d.populations()
    e = capi.Domain(np.zeros(shape, np.uint8), periodic=7)
    e.set_populations(f)
    assert np.array_equal(e.populations(), f)
    assert np.array_equal(e.moments()[1], u1)
    image = d.save_state()
    e.load_state(image)
    assert np.array_equal(e.save_state(), image)
    d.destroy()
    e.destroy()


def test_transfers_from_several_threads(capi):
    print("[gpu] transfers from four threads", flush=True)
    shape, bad = (24, 64, 96), []

    def work(seed):
        rho, u = fields(shape, seed)
        d = capi.Domain(np.zeros(shape, np.uint8), periodic=7)
        d.init_fields(rho, u)
        first = d.moments()
        f = d.populations()
        for _ in range(4):
            d.set_populations(f)
            again = d.moments()
            if not (np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
                    and np.array_equal(f, d.populations()) and np.abs(first[1] - u).max() <= 4e-6):
                bad.append(seed)
        d.destroy()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
