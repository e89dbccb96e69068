"""A release succeeds whether or not there is device memory to compact the
packed tables: with the compaction's memory refused at each fallible step in
turn (lbm_debug_fail_after), the slots are released, the survivors of both
parity classes and the domains admitted next end bit for bit where they end
alone, and a later release compacts and hands the slots on."""
import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def make(capi, n, seed):
    d = capi.Domain(I.periodic_box(n), periodic=7, storage="fp16s")
    d.set_params(0.6)
    rng = np.random.default_rng(seed)
    d.init_fields(None, (0.04 * rng.uniform(-1, 1, (3, n, n, n))).astype(np.float32))
    return d


@pytest.mark.parametrize("refused", [1, 2, 3, 4, 5, 6])
def test_release_without_memory_for_a_compaction(capi, refused):
    print(f"[gpu] release, fallible step {refused} refused", flush=True)
    b = capi.Batch(1 << 34, "fp16s")
    resident, results = {}, []

    def admit(n, seed, steps):
        d = make(capi, n, seed)
        slot = b.admit(d, steps)
        resident[slot] = (d, n, seed, steps)
        return slot

    def finish(slot, refused=0):
        capi.check(capi.lbm_debug_fail_after(refused))
        b.release(slot)
        capi.check(capi.lbm_debug_fail_after(0))
        d, n, seed, steps = resident.pop(slot)
        results.append((d.populations(), n, seed, steps))
        d.destroy()

    # 52^3 cells are 2197 tiles: two of them leave a compaction to do
    large = [admit(52, 1, 1), admit(52, 2, 2)]
    admit(12, 3, 9)
    admit(17, 4, 8)
    b.step(1)
    admit(16, 5, 9)  # the other parity class
    b.step(1)
    assert set(large) <= set(b.poll(wait=True))
    finish(large[0])
    finish(large[1], refused)
    admit(20, 6, 4)
    # the next release compacts, and then the large ones' slots are free
    while len(resident) > 2:
        b.step(2)
        for slot in b.poll(wait=True):
            finish(slot)
    reused = [admit(9, 7, 3), admit(10, 8, 3)]
    assert set(reused) & set(large)
    while resident:
        b.step(4)
        for slot in b.poll(wait=True):
            finish(slot)
    b.destroy()
    assert len(results) == 8
    for got, n, seed, steps in results:
        d = make(capi, n, seed)
        d.step(steps)
        assert np.array_equal(got, d.populations()), (n, seed)
        d.destroy()
