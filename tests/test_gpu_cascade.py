"""Cascades with many generations of leptons within one run of many steps (k_multi_tail carries those
after the third): per uid the particles of single steps, bit for bit, and no slower than they."""
import math
import time

import numpy as np
import pytest

from paper_1311_5551_amd import capi, workloads as W
from paper_1311_5551_amd.sim import Run, Tables
from test_gpu_multi import FULL, _make, _same, _same_particles, _single

pytestmark = pytest.mark.gpu

PRECISIONS = [capi.QED_FP64, capi.QED_FP32_MIXED]


@pytest.fixture(scope="module")
def tables():
    return Tables.build(n_eta=64, n_chi=64, n_chi_pair=64, n_f=64)


def _at_rest(n, a0, steps, seed=3, instance=0):
    """Electrons at rest in the standing wave of two CP lasers of amplitude a0, dt = lambda/200c."""
    z = np.zeros(n)
    rng = np.random.default_rng(seed + instance)
    e = dict(x=rng.uniform(0, 2 * math.pi, n), y=z, z=z, ux=z, uy=z, uz=z, uid=np.arange(n, dtype=np.uint64))
    w = W.Workload(name="cascade", field_kind=W.FIELD_CP_STANDING, field=(a0 / W.KAPPA,), dt=2 * math.pi / 200,
                   n_steps=steps, flags=FULL, electrons=e, seed=seed, instance=instance)
    w.capacity = dict(electron=100 * n + 4096, positron=100 * n + 4096, photon=700 * n + 8192)
    return w


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n,a0,steps,queue", [(1, 2000.0, 100, None), (40, 2000.0, 90, None), (3001, 1000.0, 190, None),
                                              (700, 1000.0, 190, 1)])
def test_cascade_equals_single_steps(n, a0, steps, queue, precision, tables):
    w = _at_rest(n, a0, steps)
    ra, rb = Run(w, tables, precision=precision), Run(w, tables, precision=precision)
    for r in (ra, rb):
        if queue:
            r.set_event_queue(queue)
    _single(ra, steps)
    rb.run(steps)
    _same(ra, rb)
    if n > 1:
        assert sum(ra.ledger()[0]["count"][:2]) > 10 * n


@pytest.mark.parametrize("precision", PRECISIONS)
def test_batched_cascades(precision, tables):
    ws = [_at_rest(n, a0, 120, instance=i) for i, (n, a0) in enumerate([(300, 1500.0), (0, 900.0), (65, 2000.0),
                                                                        (1, 1000.0), (900, 200.0)])]
    ra, rb = Run(ws, tables, precision=precision), Run(ws, tables, precision=precision)
    _single(ra, 120)
    rb.run(120)
    _same(ra, rb)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("size", [(2, 2, 2, 3), (1024, 40, 1024, 40)])
def test_smallest_and_largest_rate_tables(size, precision):
    tb = Tables.build(**dict(zip(("n_eta", "n_chi", "n_chi_pair", "n_f"), size)))
    w = _at_rest(300, 1500.0, 120)
    ra, rb = Run(w, tb, precision=precision), Run(w, tb, precision=precision)
    _single(ra, 120)
    rb.run(120)
    _same(ra, rb)


def test_cascades_on_two_streams(tables):
    # two tails share the GPU: each advances with the blocks that it has running
    ws = [_at_rest(3000, a0, 150, seed=s) for a0, s in ((1000.0, 3), (1200.0, 8))]
    alone, both = [Run(w, tables) for w in ws], [Run(w, tables) for w in ws]
    for r in alone:
        r.run(150)
        r.synchronize()
    assert both[0].stream.cuda_stream != both[1].stream.cuda_stream
    for _ in range(3):
        for r in both:
            r.run(50)
    for a, b in zip(alone, both):
        _same_particles(a, b)
        assert b.count(0, "positron") > 1000


@pytest.mark.parametrize("precision", PRECISIONS)
def test_cascade_is_no_slower_than_single_steps(precision, tables):
    # with the later generations in one block the run took 3.7 times as long as the single steps
    def best(advance):
        t = []
        for _ in range(3):
            r = Run(_at_rest(10_000, 1000.0, 200), tables, precision=precision)
            advance(r, 1)
            r.synchronize()
            t0 = time.perf_counter()
            advance(r, 199)
            r.synchronize()
            t.append(time.perf_counter() - t0)
            r.close()
        return min(t)
    single, run = best(_single), best(lambda r, k: r.run(k))
    print("single steps %.2f ms, run %.2f ms" % (1e3 * single, 1e3 * run))
    assert run < 1.25 * single


@pytest.mark.parametrize("kind", ["cascade", "pulse"])
def test_run_in_a_captured_graph(kind, tables):
    # a program's own graph of a run and a compaction, replayed with eager work between the replays
    w = _at_rest(500, 1200.0, 121) if kind == "cascade" else _make("pulse", 1500, 121)
    ra, rb = Run(w, tables), Run(w, tables)
    for r in (ra, rb):
        r.step(1)
        r.synchronize()
    torch = rb.torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=rb.stream):
        rb.run(30)
        rb.compact()
    for _ in range(4):
        ra.run(30)
        ra.compact()
        with torch.cuda.stream(rb.stream):
            g.replay()
        assert rb.ledger()[0]["n_emit"] == ra.ledger()[0]["n_emit"]
        torch.ones(100, device=rb.dev).sum().item()
    _same_particles(ra, rb)
    assert ra.ledger()[0]["n_pair"] == rb.ledger()[0]["n_pair"] > 0
