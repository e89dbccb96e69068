"""How the steps of a run reach the GPU does not change them: runs around the
lengths where the launching changes (single launches below 64 steps, replays
of a 64-step graph from a run of 256 steps on or after lbm_prepare_steps),
from either phase and across a change of rates, equal single steps bit for
bit; and a status word handed from one domain to the next starts clear."""
import numpy as np
import pytest

from paper_2204_10566_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def capi():
    from paper_2204_10566_amd import capi

    return capi


def make(capi, storage):
    spec = I.DomainSpec(kind="channel", nx=20, ny=9, nz=7, tau=0.6, steps=0).materialise()
    d = capi.Domain(spec.flags, periodic=spec.periodic, storage=storage)
    d.set_params(spec.tau)
    d.init_fields(None, spec.u.astype(np.float32))
    return d


@pytest.mark.parametrize("storage", ["fp32", "fp16s"])
@pytest.mark.parametrize("runs", [(63, 64, 65), (255, 1, 256), (1, 321, 64), (257, -1, 130)])
@pytest.mark.parametrize("prepare", [False, True])
def test_runs_equal_single_steps(capi, storage, runs, prepare):
    """A run of -1 stands for a change of the rates."""
    print(f"[gpu] runs {runs} {storage} prepare {prepare}", flush=True)
    got, ref = make(capi, storage), make(capi, storage)
    if prepare:
        got.prepare_steps()
    for n in runs:
        if n < 0:
            got.set_params(0.7)
            ref.set_params(0.7)
            continue
        got.step(n)
        for _ in range(n):
            ref.step_async(1)
        assert ref.wait_status() == capi.OK
        assert np.array_equal(got.populations(), ref.populations())
    got.destroy()
    ref.destroy()


def test_status_words_are_handed_on_clear(capi):
    """More domains than one block of words holds, unstable ones among them:
    each reports its own state only, and a new domain starts stable."""
    print("[gpu] status words", flush=True)
    fl = I.periodic_box(4)
    bad_state = np.full((27,) + fl.shape, -0.01, np.float32)
    doms = []
    for k in range(1030):
        d = capi.Domain(fl, periodic=7)
        if k % 100 == 0:
            d.set_populations(bad_state)
        doms.append(d)
    for k in (0, 1, 100, 1023, 1024, 1029):
        assert doms[k].step_status(1) == (capi.ERR_UNSTABLE if k % 100 == 0 else capi.OK)
    for d in doms:
        d.destroy()
    for _ in range(3):
        d = capi.Domain(fl, periodic=7)
        assert d.step_status(1) == capi.OK
        d.destroy()
