"""The packed tables kept on the device: admissions append a domain's tile
records there and compactions gather the survivors.  Survivors in both parity
classes, slots handed on at once after a compaction, a domain without any
updated cell and one of a single tile all end bit for bit where they end
alone."""
import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def make(capi, n, seed, storage, solid=False):
    fl = np.full((n, n, n), I.SOLID, np.uint8) if solid else I.periodic_box(n)
    d = capi.Domain(fl, periodic=7, storage=storage)
    d.set_params(0.6)
    rng = np.random.default_rng(seed)
    d.init_fields(None, (0.04 * rng.uniform(-1, 1, (3, n, n, n))).astype(np.float32))
    return d


@pytest.mark.parametrize("storage,group", [("fp16s", None), ("fp32", (1, 3))])
def test_compaction_with_survivors_and_slot_reuse(capi, storage, group):
    print(f"[gpu] table compaction {storage} {group}", flush=True)
    b = capi.Batch(1 << 34, storage)
    if group:
        b.set_cache_block(*group)
    keep, steps = {}, 12
    # (edge, seed, steps): the large ones finish first and leave more than
    # half of the table's tiles (and over 4096) to a compaction
    large = [(52, 1, 2), (48, 2, 2), (52, 3, 2)]
    small = [(4, 4, steps), (17, 5, steps), (12, 6, steps + 1)]
    got, ref = [], []

    def alone(n, seed, k):
        d = make(capi, n, seed, storage)
        d.step(k)
        ref.append(d.populations())
        d.destroy()

    first = []
    for n, seed, k in large[:2] + small[:2]:
        d = make(capi, n, seed, storage)
        first.append((b.admit(d, k), d, n, seed, k))
    empty = make(capi, 5, 0, storage, solid=True)
    empty_slot = b.admit(empty, 1)
    b.step(1)  # the next ones stream while the first collide locally
    for n, seed, k in large[2:] + small[2:]:
        d = make(capi, n, seed, storage)
        first.append((b.admit(d, k), d, n, seed, k))
    keep = {slot: rest for slot, *rest in first}
    b.step(2)
    b.step(1)
    done = b.poll(wait=True)
    assert empty_slot in done
    reused = 0
    released = []
    for slot in done:
        b.release(slot)
        released.append(slot)
        if slot == empty_slot:
            empty.destroy()
            continue
        d, n, seed, k = keep.pop(slot)
        got.append(d.populations())
        d.destroy()
        alone(n, seed, k)
    # the freed slots go to new domains before any further step
    for seed in (7, 8, 9):
        d = make(capi, 20, seed, storage)
        slot = b.admit(d, 5)
        reused += slot in released
        keep[slot] = (d, 20, seed, 5)
    assert reused > 0
    while keep:
        b.step(4)
        for slot in b.poll(wait=True):
            d, n, seed, k = keep.pop(slot)
            b.release(slot)
            got.append(d.populations())
            d.destroy()
            alone(n, seed, k)
    b.destroy()
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)
