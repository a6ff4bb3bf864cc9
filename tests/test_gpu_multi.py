"""A run advances each particle by many steps at once where the field leaves particles
independent; single steps advance all particles together.  Both use the same arithmetic and the
same random streams, so every particle, per uid, and every count of the ledger is equal bit for
bit.  Lengths at the edges of the rule (4 steps and more go the many-step way, in pieces of at most
256), strong fields whose pairs radiate and convert again within one run, ragged batches, the
pair-event queue's fallback, compaction between runs, and buffers that overflow."""
import numpy as np
import pytest

from paper_1311_5551_amd import capi, workloads as W
from paper_1311_5551_amd.sim import Run, Tables

pytestmark = pytest.mark.gpu

FULL = W.FLAG_EMIT | W.FLAG_PAIRS | W.FLAG_PROPAGATE
PRECISIONS = [capi.QED_FP64, capi.QED_FP32_MIXED]
COUNTS = ("count", "n_emit", "n_null", "n_pair", "n_dropped", "n_range", "n_nonfinite", "photon_steps_in_field",
          "photon_steps_active", "lepton_steps_in_field", "particle_steps", "n_retired")
ENERGIES = ("work", "defect_emit", "defect_pair", "radiated", "retired_energy")


@pytest.fixture(scope="module")
def tables():
    return Tables.build(n_eta=64, n_chi=64, n_chi_pair=64, n_f=64)


def _single(run, n):
    for _ in range(n):
        run.step(1)


def _same(ra, rb):
    for i in range(len(ra.bufs)):
        for name in ("electron", "positron", "photon"):
            a, b = ra.species(i, name), rb.species(i, name)
            oa, ob = np.argsort(a["uid"]), np.argsort(b["uid"])
            assert len(oa) == len(ob), (i, name, len(oa), len(ob))
            for k in a:
                np.testing.assert_array_equal(a[k][oa], b[k][ob], err_msg="%d %s.%s" % (i, name, k))
    for la, lb in zip(ra.ledger(), rb.ledger()):
        assert la["status"] == lb["status"] == "QED_OK"
        for k in COUNTS:
            assert la[k] == lb[k], k
        # single steps also read the windows behind stale live bits (a photon converted in the step
        # before, a slot behind the photons that a compaction left)
        assert lb["photon_steps_active"] <= lb["photon_window_reads"] <= la["photon_window_reads"]
        scale = abs(la["energy0"]) + sum(map(abs, la["energy"]))
        for k in ENERGIES + ("energy",):
            # each term is exact to 2^-64 or the rounding of one step's group of 64
            np.testing.assert_allclose(np.asarray(la[k]), np.asarray(lb[k]), rtol=1e-12, atol=1e-13 * scale, err_msg=k)
        assert lb["drift"] < 1e-9


def _standing(n, seed):
    z = np.zeros(n)
    rng = np.random.default_rng(seed)
    e = dict(x=rng.uniform(0, 20, n), y=z, z=z, ux=rng.normal(0, 2000, n), uy=rng.normal(0, 2000, n), uz=z,
             uid=np.arange(n, dtype=np.uint64))
    return W.Workload(name="standing", field_kind=W.FIELD_CP_STANDING, field=(1000.0 / W.KAPPA,), dt=0.01, n_steps=200,
                      flags=FULL, electrons=e, seed=seed)


def _make(kind, n, steps, flags=FULL, seed=5):
    if kind == "uniform":
        w = W.uniform_b(n, 1000.0, 9e-3, 0.15 * W.dt_qed(9e-3), steps, flags, seed)
    elif kind == "pulse":
        w = W.collision(n, a0=450.0, gamma_mean=4000.0, n_steps=steps, meet_step=steps // 2, fwhm_fs=4.0, sigma_um=0.3,
                        seed=seed, flags=flags)
    elif kind == "wave":
        w = W.cp_wave_test2(n, 0.1, seed)
        w.field, w.flags = (6 * w.field[0], 0.0), flags
    else:
        w = _standing(n, seed)
        w.flags = flags
    w.capacity = dict(electron=60 * n + 4096, positron=60 * n + 4096, photon=400 * n + 8192)
    return w


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("kind", ["uniform", "pulse", "wave", "standing"])
@pytest.mark.parametrize("n,pieces", [(1, (4, 96)), (63, (5, 59, 3, 60)), (700, (150,)), (3001, (259, 30))])
def test_run_equals_single_steps(kind, n, pieces, precision, tables):
    w = _make(kind, n, sum(pieces))
    ra, rb = Run(w, tables, precision=precision), Run(w, tables, precision=precision)
    for k in pieces:
        _single(ra, k)
        rb.run(k, graph_steps=k)
    _same(ra, rb)
    if n >= 700:
        assert ra.ledger()[0]["n_pair"] > 0


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("flags", [0, W.FLAG_EMIT, W.FLAG_PAIRS | W.FLAG_PROPAGATE, capi.QED_RR_QUANTUM,
                                   capi.QED_RR_CLASSICAL])
@pytest.mark.parametrize("kind", ["uniform", "pulse"])
def test_run_equals_single_steps_flags(kind, flags, precision, tables):
    w = _make(kind, 517, 120, flags)
    ph = W.photon_population(1000, seed=3) if flags & W.FLAG_PAIRS else None
    ra, rb = (Run(w, tables, precision=precision, photons=ph) for _ in range(2))
    _single(ra, 120)
    rb.run(120)
    _same(ra, rb)
    # the live masks of photons emitted without a photon pass serve a later one
    if flags == W.FLAG_EMIT:
        for r in (ra, rb):
            r.params.flags = FULL
            _single(r, 20)
        for la, lb in zip(ra.ledger(), rb.ledger()):
            assert la["photon_steps_active"] == lb["photon_steps_active"] and la["n_pair"] == lb["n_pair"]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("queue", [None, 1])
def test_batched_runs_with_compaction(queue, precision, tables):
    ws = []
    for i, (n, a0, g0) in enumerate([(300, 450.0, 4000.0), (1, 300.0, 2000.0), (0, 100.0, 1000.0), (65, 500.0, 5000.0)]):
        w = W.collision(n, a0=a0, gamma_mean=g0, n_steps=600, meet_step=300, fwhm_fs=8.0, sigma_um=0.4, seed=2, instance=i)
        w.capacity = dict(electron=60 * n + 4096, positron=60 * n + 4096, photon=600 * n + 8192)
        ws.append(w)
    ra, rb = Run(ws, tables, precision=precision), Run(ws, tables, precision=precision)
    for r in (ra, rb):
        r.set_retire(16)
        if queue:
            r.set_event_queue(queue)
    for _ in range(6):
        _single(ra, 100)
        rb.run(100)
        ra.compact()
        rb.compact()
    _same(ra, rb)
    for i in range(len(ws)):
        np.testing.assert_array_equal(ra.retired_spectrum(i), rb.retired_spectrum(i))
    assert sum(l["n_pair"] for l in ra.ledger()) > 100


@pytest.mark.parametrize("precision", PRECISIONS)
def test_more_chunks_than_blocks(precision, tables):
    """Blocks take further chunks as they become free: more beams than blocks, ragged."""
    ws = []
    for i in range(600):
        n = i % 24
        w = W.uniform_b(n, 1000.0, 9e-3, 0.15 * W.dt_qed(9e-3), 24, FULL, seed=7)
        w.instance = i
        w.capacity = dict(electron=8 * n + 64, positron=8 * n + 64, photon=40 * n + 64)
        ws.append(w)
    ra, rb = Run(ws, tables, precision=precision), Run(ws, tables, precision=precision)
    _single(ra, 24)
    rb.run(24)
    _same(ra, rb)


@pytest.mark.parametrize("precision", PRECISIONS)
def test_several_chunks_per_block(precision, tables):
    """Large runs have several chunks per block (from 4.2e6 leptons on)."""
    n = 4_300_037
    w = W.uniform_b(n, 1000.0, 9e-3, 0.15 * W.dt_qed(9e-3), 5, 0, seed=3)
    w.capacity = dict(electron=n, positron=1, photon=1)
    ra, rb = Run(w, tables, precision=precision), Run(w, tables, precision=precision)
    _single(ra, 5)
    rb.run(5)
    ra.synchronize()
    rb.synchronize()
    a, b = ra.bufs[0]["electron"], rb.bufs[0]["electron"]
    for k in a:
        if a[k] is not None and hasattr(a[k], "shape") and len(a[k]) == n:
            assert a[k].equal(b[k]), k
    la, lb = ra.ledger()[0], rb.ledger()[0]
    assert la["particle_steps"] == lb["particle_steps"] and la["lepton_steps_in_field"] == lb["lepton_steps_in_field"]


def test_full_photon_buffer_in_a_run(tables):
    # a run whose photons do not fit: everything dropped is counted and its energy booked
    w = W.uniform_b(900, 1000.0, 1e-3, 0.15, 64, W.FLAG_EMIT)
    r = Run(w, tables, capacity=dict(photon=5000))
    r.run(64)
    led = r.ledger()[0]
    assert led["status"] == "QED_ERR_CAPACITY"
    assert led["count"][2] == 5000 and led["n_dropped"] == led["n_emit"] - 5000 > 0
    assert led["drift"] < 1e-12 and led["dropped_energy"] > 0


@pytest.mark.parametrize("static", [False, True])
def test_sort_keeps_photons_without_a_pair_rate_in_front(static, tables):
    # sorts between the steps of a grid run put the photons below the pair threshold in front and
    # leave them there: the particles stay those of a run without sorts, through compactions before
    # and after a sort and a clock set back, and the sweep visits fewer groups
    def make():
        w = W.grid_config3(n=4000, nx=250, ny=61, a0=700.0, n_steps=200, seed=4)
        w.capacity = dict(electron=30 * w.n, positron=30 * w.n, photon=100 * w.n)
        return Run(w, tables)
    ra, rb = make(), make()
    sort = rb.sort_static if static else rb.sort
    for i in range(12):
        for r in (ra, rb):
            _single(r, 10)
            if i % 4 == 1:
                r.compact()
        sort()
        if i % 4 == 3:
            rb.compact()  # windows not rebuilt yet
            ra.compact()
        if i == 5:
            sort()
    _same_particles(ra, rb)
    la, lb = ra.ledger()[0], rb.ledger()[0]
    for k in COUNTS:
        assert la[k] == lb[k], k
    assert la["n_pair"] > 0 and la["photon_steps_active"] < 0.9 * la["particle_steps"][2]
    # back in time: the front is emptied, and the photons' windows serve the repeated steps
    # (new uids, so that the children made again do not repeat the uids of those made before)
    for r in (ra, rb):
        r.synchronize()
        for name in ("electron", "positron", "photon"):
            r.bufs[0][name]["uid"][:r.count(0, name)] ^= 0x5DEECE66D
        r.torch.cuda.synchronize()
        capi.qed_set_step(r.ws, 60, r._s())
        _single(r, 3)
    _same_particles(ra, rb)


def _same_particles(ra, rb):
    for name in ("electron", "positron", "photon"):
        a, b = ra.species(0, name), rb.species(0, name)
        oa, ob = np.argsort(a["uid"]), np.argsort(b["uid"])
        assert len(oa) == len(ob), name
        for k in a:
            np.testing.assert_array_equal(a[k][oa], b[k][ob], err_msg="%s.%s" % (name, k))
