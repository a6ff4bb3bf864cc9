"""The step-by-step path: qed_step, and qed_run's captured graphs where it still replays them (grid
fields, and runs of fewer than 4 steps).  Run.step(n > 1) is one qed_run, which in the other fields
advances each particle by many steps at once; here every step is a launch of the sweeps."""
import numpy as np
import pytest

from paper_1311_5551_amd import capi, workloads as W
from paper_1311_5551_amd.sim import Run, Tables
from test_gpu_multi import COUNTS, FULL, _make, _same, _same_particles, _single

pytestmark = pytest.mark.gpu

PRECISIONS = [capi.QED_FP64, capi.QED_FP32_MIXED]
LEDGER = ("energy", "energy0", "work", "defect_emit", "defect_pair", "dropped_energy", "radiated", "drift", "count",
          "n_emit", "n_null", "n_pair")


@pytest.fixture(scope="module")
def tables():
    return Tables.build(n_eta=64, n_chi=64, n_chi_pair=64, n_f=64)


def _grid(n=3000, steps=120):
    w = W.grid_config3(n=n, nx=250, ny=61, a0=700.0, n_steps=steps, seed=4)
    w.capacity = dict(electron=30 * n, positron=30 * n, photon=100 * n)
    return w


@pytest.mark.parametrize("precision", PRECISIONS)
def test_graph_replay_equals_single_steps_on_a_grid(precision, tables):
    # replays of one captured graph, with the program's own work, a sort and a compaction between them
    ra, rb = (Run(_grid(), tables, precision=precision) for _ in range(2))
    _single(ra, 120)
    for i in range(4):
        rb.run(30, graph_steps=10)
        assert rb.ledger()[0]["status"] == "QED_OK"
        rb.torch.ones(1000, device=rb.dev).sum().item()
        if i == 1:
            rb.sort()
        if i == 2:
            rb.compact()
            ra.compact()
    la, lb = ra.ledger()[0], rb.ledger()[0]
    for k in COUNTS:
        if k not in ("particle_steps", "count"):  # (the runs compact at other steps)
            assert la[k] == lb[k], k
    ra.compact()
    rb.compact()
    _same_particles(ra, rb)
    assert la["n_pair"] > 0


@pytest.mark.parametrize("precision", PRECISIONS)
def test_graph_replay_of_short_runs(precision, tables):
    w = _make("pulse", 700, 150)
    ra, rb = (Run(w, tables, precision=precision) for _ in range(2))
    _single(ra, 150)
    for i in range(50):
        rb.run(3, graph_steps=1 + i % 3)
        if i % 7 == 0:
            rb.ledger()
    _same_particles(ra, rb)
    la, lb = ra.ledger()[0], rb.ledger()[0]
    for k in COUNTS:
        assert la[k] == lb[k], k
    assert la["n_pair"] > 0


@pytest.mark.parametrize("kind,flags", [("pulse", FULL), ("pulse", capi.QED_RR_QUANTUM), ("uniform", FULL),
                                        ("uniform", capi.QED_RR_CLASSICAL), ("standing", FULL), ("grid", FULL)])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_single_step_ledger_is_independent_of_launch_shape(precision, kind, flags, tables):
    leds, runs = [], []
    for (bl, pl), (bp, pp) in [((64, 1), (64, 1)), ((256, 8), (256, 16)), ((128, 2), (192, 4)), ((192, 4), (64, 8))]:
        r = Run(_grid(2000) if kind == "grid" else _make(kind, 2000, 120, flags), tables, precision=precision)
        r.set_kernel_launch(capi.QED_KERNEL_LEPTON, bl, pl)
        r.set_kernel_launch(capi.QED_KERNEL_PHOTON, bp, pp)
        for _ in range(4):
            _single(r, 30)
            r.compact()
        leds.append(r.ledger()[0])
        runs.append(r)
    assert leds[0]["status"] == "QED_OK"
    for led in leds[1:]:
        for k in LEDGER:
            assert led[k] == leds[0][k], k
    assert leds[0]["defect_emit" if flags == FULL else "radiated"] != 0.0  # (a magnetic field does no work)
    for r in runs[1:]:
        _same_particles(runs[0], r)


def test_photon_windows_past_16_bit_single_steps(tables):
    # the packed windows hold 16-bit step indices and saturate from step 65535 on
    s0, n = 68000, 5000
    w = W.collision(1, a0=450.0, n_steps=s0 + 1000, meet_step=s0 + 500, fwhm_fs=8.0, sigma_um=0.3, seed=9,
                    flags=W.FLAG_PAIRS | W.FLAG_PROPAGATE)
    w.electrons = {k: v[:0] for k, v in w.electrons.items()}
    w.capacity = dict(electron=2 * n + 1024, positron=2 * n + 1024, photon=n + 1024)
    ph = W.photon_population(n, sigma_um=0.3, seed=9)
    ph["x"] = ph["x"] - np.sqrt(1.0 - 1.0 / 2000.0 ** 2) * s0 * w.dt  # where the beam is at step s0
    ph["birth_step"] = np.full(n, s0, dtype=np.int64)
    ra, rb = (Run(w, tables, photons=ph, step0=s0) for _ in range(2))
    for _ in range(5):
        _single(ra, 200)
        rb.run(200)
        ra.compact()
        rb.compact()
    _same(ra, rb)
    assert ra.ledger()[0]["n_pair"] > 20


def test_set_step_back_single_steps(tables):
    # the front that compactions made is emptied when the clock is set back
    w = W.collision(1500, a0=450.0, gamma_mean=4000.0, n_steps=900, meet_step=450, fwhm_fs=8.0, sigma_um=0.3, seed=11)
    w.capacity = dict(electron=60 * w.n, positron=60 * w.n, photon=900 * w.n)
    ra, rb = (Run(w, tables) for _ in range(2))
    advance = ((ra, _single), (rb, lambda r, k: r.run(k)))
    for r, step in advance:
        for _ in range(6):
            step(r, 100)
            r.compact()
        r.synchronize()
        for name in ("electron", "positron", "photon"):  # new uids for the children made again
            r.bufs[0][name]["uid"][:r.count(0, name)] ^= 0x5DEECE66D
        r.torch.cuda.synchronize()
        capi.qed_set_step(r.ws, 350, r._s())
    before = ra.ledger()[0]["n_pair"]
    for r, step in advance:
        step(r, 250)
    _same(ra, rb)
    assert ra.ledger()[0]["n_pair"] > before > 0
