"""Compaction decides by the pair windows of the photons that sit in the slots now: after a sort,
which moves the photons, and before the first step of a binding, when no window exists yet."""
import numpy as np
import pytest

from paper_1311_5551_amd import capi, workloads as W
from paper_1311_5551_amd.sim import Run, Tables

pytestmark = pytest.mark.gpu

PRECISIONS = [capi.QED_FP64, capi.QED_FP32_MIXED]


@pytest.fixture(scope="module")
def tables():
    return Tables.build(n_eta=64, n_chi=64, n_chi_pair=64, n_f=64)


def _same(ra, rb):
    for name in ("electron", "positron", "photon"):
        a, b = ra.species(0, name), rb.species(0, name)
        oa, ob = np.argsort(a["uid"]), np.argsort(b["uid"])
        assert len(oa) == len(ob), (name, len(oa), len(ob))
        for k in a:
            np.testing.assert_array_equal(a[k][oa], b[k][ob], err_msg="%s.%s" % (name, k))
    la, lb = ra.ledger()[0], rb.ledger()[0]
    for k in ("count", "n_emit", "n_pair", "n_retired", "photon_steps_in_field", "photon_steps_active", "status"):
        assert la[k] == lb[k], k
    return la


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("static", [False, True])
def test_retirement_after_a_sort(static, precision, tables):
    def make():
        w = W.grid_config3(n=4000, nx=250, ny=61, a0=700.0, n_steps=120, seed=4)
        w.capacity = dict(electron=30 * w.n, positron=30 * w.n, photon=100 * w.n)
        r = Run(w, tables, precision=precision)
        r.set_retire(16)
        return r
    ra, rb = make(), make()
    sort = rb.sort_static if static else rb.sort
    for i in range(12):
        for r in (ra, rb):
            for _ in range(10):
                r.step(1)
        sort()
        if i % 3 == 2:
            sort()
        if i % 2:
            ra.compact()
            rb.compact()
            if i % 4 == 3:
                rb.compact()  # nothing left to retire
    la = _same(ra, rb)
    assert ra.retired_spectrum() == rb.retired_spectrum()
    assert la["n_retired"] > 1000 and la["n_pair"] > 50 and la["status"] == "QED_OK"


@pytest.mark.parametrize("retire", [0, 16])
def test_compaction_before_the_first_step(retire, tables):
    w = W.collision(200, a0=450.0, gamma_mean=4000.0, n_steps=200, meet_step=100, fwhm_fs=4.0, sigma_um=0.3)
    w.capacity = dict(electron=40 * w.n, positron=40 * w.n, photon=400 * w.n)
    ph = W.photon_population(1500, seed=3)
    ra, rb = (Run(w, tables, photons=ph, step0=70) for _ in range(2))
    for r in (ra, rb):
        if retire:
            r.set_retire(retire)
    rb.compact()
    assert rb.count(0, "photon") == 1500 and rb.ledger()[0]["n_retired"] == 0
    for r in (ra, rb):
        for _ in range(60):
            r.step(1)
        r.compact()
    la = _same(ra, rb)
    assert la["n_pair"] > 0 and (la["n_retired"] > 0) == bool(retire)


def test_a_captured_compaction_leaves_the_windows_to_the_next_step(tables):
    # recorded after a sort and not replayed: the next step still makes the windows again
    def make():
        w = W.grid_config3(n=3000, nx=250, ny=61, a0=700.0, n_steps=120, seed=4)
        w.capacity = dict(electron=30 * w.n, positron=30 * w.n, photon=100 * w.n)
        return Run(w, tables)
    ra, rb = make(), make()
    for r in (ra, rb):
        for _ in range(60):
            r.step(1)
    rb.sort()
    rb.synchronize()
    g = rb.torch.cuda.CUDAGraph()
    with rb.torch.cuda.graph(g, stream=rb.stream):
        rb.compact()
    for i in range(60):
        for r in (ra, rb):
            r.step(1)
        if i == 30:
            rb.sort()
            with rb.torch.cuda.stream(rb.stream):
                g.replay()
    for r in (ra, rb):
        r.compact()
    assert _same(ra, rb)["n_pair"] > 0
