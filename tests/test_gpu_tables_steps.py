"""The device-built tables over several steps: values handed from the last
plane to outlet cells, and leaving values parked there, are read again by the
steps that follow, so a wrong outlet target, edge mark or tile position shows.
Last planes that mix outlet, fluid and solid cells at random, many tiles
without an updated cell, against the oracle in FP32 and FP16S with both outlet
conditions; and the statistics, whose sums are laid out by a tile's position
in the list, against the moments of the state they were taken from."""
import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu

# the per-step bounds of the random configurations (FP16S: 2^-11 |f - w| a store)
TOL = {"fp32": 4e-7, "fp16s": 5e-5}


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def geometry(size, kind, periodic, seed):
    nx, ny, nz = size
    rng = np.random.default_rng(seed)
    fl = np.zeros((nz, ny, nx), np.uint8)
    fl[rng.random(fl.shape) < 0.15] = I.SOLID
    fl[rng.random(fl.shape) < 0.05] = I.INLET
    if kind == "slabs":  # whole tiles without an updated cell, before and between the others
        fl.reshape(-1)[:200] = I.SOLID
        fl[nz // 2, : ny // 2] = I.SOLID
    plane = fl[:, :, -1]
    plane[(plane == I.FLUID) & (rng.random(plane.shape) < 0.6)] = I.OUTLET
    return fl


@pytest.mark.parametrize("size,periodic", [((23, 11, 9), 0), ((64, 9, 7), 6), ((128, 17, 8), 4), ((131, 40, 7), 2)])
@pytest.mark.parametrize("kind", ["mixed", "slabs"])
@pytest.mark.parametrize("storage", ["fp32", "fp16s"])
@pytest.mark.parametrize("outlet", ["zero_gradient", "pressure"])
def test_several_steps(capi, orc, size, periodic, kind, storage, outlet):
    print(f"[gpu] tables over steps {size} {kind} {storage} {outlet}", flush=True)
    fl = geometry(size, kind, periodic, size[0])
    upd = (fl == I.FLUID) | (fl == I.OUTLET)
    rng = np.random.default_rng(2)
    uin = np.zeros((3,) + fl.shape, np.float32)
    uin[:, fl == I.INLET] = 0.03 * rng.uniform(-1, 1, (3, int((fl == I.INLET).sum())))
    f0 = I.random_populations(fl.shape, 3).astype(np.float32)
    for steps in (3, 4):
        d = capi.Domain(fl, periodic=periodic, storage=storage)
        d.set_params(0.7)
        d.set_inlet(uin)
        d.set_outlet(outlet, 1.02)
        d.set_populations(f0)
        start = d.populations().astype(np.float64)
        d.step(steps)
        got = d.populations()
        d.destroy()
        st, want = orc.step(fl, start, orc.rates_vector(1 / 0.7), steps, periodic=periodic, uin=uin,
                            outlet=("pressure", 1.02) if outlet == "pressure" else None)
        assert st == 0
        assert np.abs(got[:, upd] - want[:, upd]).max() <= steps * TOL[storage]


@pytest.mark.parametrize("size", [(23, 11, 9), (128, 17, 8)])
def test_statistics_by_tile_position(capi, size):
    print(f"[gpu] statistics by tile {size}", flush=True)
    fl = geometry(size, "slabs", 0, size[0])
    d = capi.Domain(fl)
    d.set_params(0.7)
    d.set_populations(I.random_populations(fl.shape, 4).astype(np.float32))
    info = d.info()
    assert info.n_tiles < -(-fl.size // 64)
    d.stats_enable()
    d.step(2)
    _, u = d.moments()
    mean, _, _, samples = d.stats()
    d.destroy()
    # one sample; collision conserves u, which both sum from 27 FP32 terms
    assert samples == 1
    assert np.abs(mean - u).max() <= 4e-6
