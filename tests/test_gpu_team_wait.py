"""A wait inside the one-launch pass that gave up (its flag, raised from the host) is
reported by the next call that waits for the stream, and leaves the handle usable: with
its fields set again it gives what a fresh handle gives."""
import ctypes
import sys
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import torch  # noqa: F401  (imported at collection: the first import can take minutes)

from paper_2410_02532_amd import opo as B
from test_gpu_lone import _instance

pytestmark = pytest.mark.gpu

NZ, DZ = 20, 2.0 ** -5


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def _fail_wait(h):
    lib = B.load()
    lib.opo_test_fail_wait.argtypes = [ctypes.c_void_p]
    assert lib.opo_test_fail_wait(h.h) == B.OPO_OK


def _read(h, call):
    if call == "sync":
        h.sync()
    elif call == "adaptive":
        h.ssfm_propagate_adaptive(0.1, 1e-3, 0.05)
    else:
        h.get_fields(0, domain=1 if call == "spectrum" else 0)


@pytest.mark.parametrize("precision, nz, call", [("f32", NZ, "sync"), ("f64", NZ, "fields"), ("f32", NZ, "spectrum"),
                                                 ("f64", NZ, "adaptive")])
def test_propagate_reports_a_wait_that_gave_up(precision, nz, call):
    say("team wait, propagate %s nz %d %s" % (precision, nz, call))
    ins = _instance(1 << 13, 3, 3)
    with B.Opo([ins], NZ, precision=precision) as h:
        h.ssfm_propagate(nz, DZ)
        good = h.get_fields()
    with B.Opo([ins], NZ, precision=precision) as h:
        h.ssfm_propagate(nz, DZ)
        _fail_wait(h)
        with pytest.raises(B.OpoError) as e:
            _read(h, call)
        assert e.value.code == B.OPO_EDEVICE
        h.sync()                                # reported once
        h.set_fields(ins["fields"])
        h.ssfm_propagate(nz, DZ)
        assert np.array_equal(h.get_fields(), good)


@pytest.mark.parametrize("precision, graph", [("f32", True), ("f64", False)])
def test_roundtrip_stops_at_a_wait_that_gave_up(precision, graph):
    """As for a non-finite result: the finished round trips stay, the state is the one the
    failed round trip started from, and the run goes on from there bit for bit."""
    say("team wait, round trips %s graph %s" % (precision, graph))
    ins = _instance(1 << 13, 3, 5)
    with B.Opo([ins], NZ, precision=precision, use_graph=graph) as h:
        h.cavity_roundtrip(2)
        two = h.get_fields()
        h.cavity_roundtrip(2)
        four, energies = h.get_fields(), h.energy_history()
    with B.Opo([ins], NZ, precision=precision, use_graph=graph) as h:
        h.cavity_roundtrip(2)
        _fail_wait(h)
        with pytest.raises(B.OpoError) as e:
            h.cavity_roundtrip(3)
        assert e.value.code == B.OPO_EDEVICE
        assert h.progress() == (2, 0.0) and len(h.energy_history()) == 2
        assert np.array_equal(h.get_fields(), two)
        h.cavity_roundtrip(2)
        assert np.array_equal(h.get_fields(), four)
        assert np.array_equal(h.energy_history(), energies)


def test_handles_of_teams_beside_each_other():
    """Four handles whose passes run in one launch each, driven from four threads at once (their
    teams share XCDs), give what they give one after another."""
    say("teams beside each other")
    runs = [("f32", [_instance(1 << 14, 3, 11)]), ("f64", [_instance(1 << 14, 3, 12)]),
            ("f32", [_instance(1 << l, 2, 13) for l in (13, 10, 15, 10, 12)]), ("f64", [_instance(1 << 10, 3, 14)] * 16)]

    def work(precision, insts):
        with B.Opo(insts, NZ, precision=precision) as h:
            for _ in range(5):
                h.ssfm_propagate(7, DZ)
                h.cavity_roundtrip(3)
            return [h.get_fields(i) for i in range(len(insts))], h.energy_history()

    alone = [work(*r) for r in runs]
    with ThreadPoolExecutor(len(runs)) as ex:
        beside = [f.result(timeout=100) for f in [ex.submit(work, *r) for r in runs]]
    for (fa, ea), (fb, eb) in zip(alone, beside):
        assert all(np.array_equal(x, y) for x, y in zip(fa, fb)) and np.array_equal(ea, eb)
