"""Runs of many steps whose buffers fill on the way, in any of their rounds: nothing is written past a
buffer, the counts stop at the capacity, every dropped child is counted and its energy booked."""
import pytest

from paper_1311_5551_amd import capi
from paper_1311_5551_amd.sim import SPECIES, Run, Tables
from test_gpu_cascade import _at_rest
from test_gpu_multi import _make, _single

pytestmark = pytest.mark.gpu

PRECISIONS = [capi.QED_FP64, capi.QED_FP32_MIXED]
GUARD = 64


@pytest.fixture(scope="module")
def tables():
    return Tables.build(n_eta=64, n_chi=64, n_chi_pair=64, n_f=64)


def _bound_smaller(w, tables, precision, caps):
    """A run whose bound capacities end before its arrays, which hold a mark from there on."""
    r = Run(w, tables, precision=precision)
    for si, name in enumerate(SPECIES):
        cap = caps.get(name)
        if cap is None:
            continue
        sb = r.bufs[0][name]
        assert cap + GUARD <= sb["capacity"]
        for k, v in sb.items():
            if k != "count" and r.torch.is_tensor(v):
                v[cap:] = 77
        sb["capacity"] = r.insts[0].s[si].capacity = cap
    r.torch.cuda.synchronize()
    capi.qed_bind(r.ws, r.insts, r.params)
    return r


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("caps", [dict(electron=1500, positron=900), dict(electron=900), dict(positron=0),
                                  dict(photon=20000), dict(electron=2001, positron=1003, photon=40001)])
@pytest.mark.parametrize("kind,n,steps", [("cascade", 400, 190), ("pulse", 800, 150)])
@pytest.mark.parametrize("single", [False, True])
def test_buffers_that_fill_during_a_run(single, kind, n, steps, caps, precision, tables):
    w = _at_rest(n, 1000.0, steps) if kind == "cascade" else _make(kind, n, steps)
    r = _bound_smaller(w, tables, precision, caps)
    if single:
        _single(r, steps)
    else:
        r.run(steps)
    led = r.ledger()[0]
    slots = [r.count(0, s) for s in SPECIES]
    full = [s for s, c in zip(SPECIES, slots) if c == caps.get(s)]
    for name, cap in caps.items():
        sb = r.bufs[0][name]
        for k, v in sb.items():
            if k != "count" and r.torch.is_tensor(v):
                assert bool((v[cap:] == 77).all()), (name, k)
    missing = n + 2 * led["n_pair"] - slots[0] - slots[1] + led["n_emit"] - slots[2]
    assert led["n_dropped"] == missing
    assert led["status"] == ("QED_ERR_CAPACITY" if missing else "QED_OK")
    if kind == "cascade":
        assert full and missing > 0 and led["dropped_energy"] > 0
    assert led["drift"] < 1e-9
    # the next run goes on from the full buffers
    before = led["n_dropped"]
    r.run(8)
    led = r.ledger()[0]
    assert led["n_dropped"] >= before and [r.count(0, s) for s in full] == [caps[s] for s in full]
    assert led["drift"] < 1e-9
