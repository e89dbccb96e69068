"""The tables that a domain's creation builds on the device, at the sizes
where tiles (64 cells) and the groups of its scan and hash (16384 cells) end:
counts against numpy, the flags' hash of a state image against the serial
FNV-1a, and one step of a random state against the oracle, whose links are
found cell by cell."""
import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu

# the per-step bound of the random configurations
TOL = 4e-7


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def fnv1a64(data):
    h = 0xCBF29CE484222325
    for b in data:
        h = ((h ^ b) * 0x100000001B3) & (2 ** 64 - 1)
    return h


SIZES = [(1, 1, 1), (63, 1, 1), (64, 1, 1), (65, 1, 1), (1, 5, 13), (128, 128, 1), (127, 43, 3), (145, 113, 1),
         (128, 64, 4), (131, 97, 11)]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("kind", ["mixed", "sparse", "fluid", "solid"])
def test_tables(capi, orc, size, kind):
    nx, ny, nz = size
    seed = SIZES.index(size)
    rng = np.random.default_rng(seed)
    periodic = [0, 7, 6, 2, 5][seed % 5]
    fl = np.zeros((nz, ny, nx), np.uint8)
    if kind == "mixed":
        fl[rng.random(fl.shape) < 0.2] = I.SOLID
        fl[rng.random(fl.shape) < 0.1] = I.INLET
    elif kind == "sparse":  # most tiles hold no updated cell
        fl[:] = I.SOLID
        fl[rng.random(fl.shape) < 0.004] = I.FLUID
        fl[rng.random(fl.shape) < 0.004] = I.INLET
    elif kind == "solid":
        fl[:] = I.SOLID
    if not periodic & 1 and kind != "solid":
        plane = fl[:, :, -1]
        plane[(plane == I.FLUID) & (rng.random(plane.shape) < 0.7)] = I.OUTLET
    print(f"[gpu] tables {size} {kind} periodic {periodic}", flush=True)

    d = capi.Domain(fl, periodic=periodic)
    info = d.info()
    upd = (fl == I.FLUID) | (fl == I.OUTLET)
    tiles = np.zeros(-(-fl.size // 64) * 64, bool)
    tiles[:fl.size] = upd.ravel()
    assert info.n_updated == upd.sum()
    assert info.n_tiles == tiles.reshape(-1, 64).any(1).sum()
    assert info.n_inlet == (fl == I.INLET).sum()
    # wall tiles: a tile of updated cells with a cell that is not updated, an
    # outlet, or a link that does not end in a fluid or outlet cell
    plain = upd & (fl != I.OUTLET)
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    for i in range(27):
        at, ok = [], np.ones(fl.shape, bool)
        for v, c, n, bit in ((x, i % 3 - 1, nx, 1), (y, (i // 3) % 3 - 1, ny, 2), (z, i // 9 - 1, nz, 4)):
            s = v - c
            if periodic & bit:
                s = s % n
            ok &= (s >= 0) & (s < n)
            at.append(np.clip(s, 0, n - 1))
        src = fl[at[2], at[1], at[0]]
        plain &= ok & (src != I.SOLID) & (src != I.INLET)
    inner = np.zeros_like(tiles)
    inner[:fl.size] = plain.ravel()
    listed = tiles.reshape(-1, 64).any(1)
    assert info.n_wall_tiles == (listed & ~inner.reshape(-1, 64).all(1)).sum()

    image = d.save_state()
    assert int(image[32:40].view(np.uint64)[0]) == fnv1a64(fl.tobytes())

    d.set_params(0.7)
    uin = np.zeros((3,) + fl.shape, np.float32)
    n_in = int((fl == I.INLET).sum())
    if n_in:
        uin[:, fl == I.INLET] = 0.03 * rng.uniform(-1, 1, (3, n_in))
        d.set_inlet(uin)
    d.set_populations(I.random_populations(fl.shape, seed).astype(np.float32))
    f0 = d.populations().astype(np.float64)
    d.step(1)
    got = d.populations()
    d.destroy()
    st, want = orc.step(fl, f0, orc.rates_vector(1 / 0.7), 1, periodic=periodic, uin=uin if n_in else None)
    assert st == 0
    assert not upd.any() or float(np.abs(got[:, upd] - want[:, upd]).max()) <= TOL
    assert np.array_equal(got[:, ~upd], f0[:, ~upd].astype(np.float32))
