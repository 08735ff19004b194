"""One system used by several threads: readers get each their own fields, whatever
others read meanwhile, and do not disturb a thread that steps the system (alone or
in an engine)."""
import threading

import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("agg_pos", "agg_vel", "agg_acc", "agg_torque", "agg_quat", "agg_spin_body", "agg_spin",
          "sph_pos", "sph_vel", "sph_force", "sph_torque", "sph_body")


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


def _sim(D, n_agg, fused=0):
    w = W.periodic_box(seed=n_agg, n_agg=n_agg, contact_seeded=True)
    sim = D.Sim(w.params)
    sim.set_tuning(fused=fused)
    return sim.add_workload(w)


def _together(jobs):
    """Runs the jobs in threads and raises what any of them raised."""
    failed = []

    def guarded(job):
        try:
            job()
        except BaseException as e:  # noqa: BLE001 - handed to the test's thread
            failed.append(e)

    ts = [threading.Thread(target=guarded, args=(j,)) for j in jobs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    if failed:
        raise failed[0]


def _equal(a, b):
    return all(np.array_equal(a[k], b[k]) for k in b)


@pytest.mark.parametrize("n_agg", [20, 700])
def test_two_readers(D, n_agg):
    print("[case] readers", n_agg, flush=True)
    sim = _sim(D, n_agg)
    sim.step(5)
    groups = [FIELDS[0:3], FIELDS[3:7], FIELDS[7:9], FIELDS[9:12], FIELDS]
    want = [sim.read_state(g, pairs=k % 2 == 0) for k, g in enumerate(groups)]
    assert want[0]["n_pairs"] > 0

    def reader(k):
        for _ in range(150):
            assert _equal(sim.read_state(groups[k], pairs=k % 2 == 0), want[k]), groups[k]

    _together([lambda k=k: reader(k) for k in range(len(groups))])


@pytest.mark.parametrize("engine", [False, True])
@pytest.mark.parametrize("fused", [0, 2])
def test_reader_beside_a_stepping_thread(D, fused, engine):
    """Reading states and forcings between and during the steps of another
    thread leaves the run as it is, and every state read is one of its steps'."""
    print("[case] reader beside stepper", fused, engine, flush=True)
    n, chunk = 12, 5
    ref = _sim(D, 40, fused)
    want = {0: ref.read_state(FIELDS, pairs=True)}
    for k in range(1, n + 1):
        ref.step(chunk)
        want[k * chunk] = ref.read_state(FIELDS, pairs=True)
    sim = _sim(D, 40, fused)
    eng = D.Engine(1 << 30)
    if engine:
        eng.attach(sim)
    done = threading.Event()

    def stepper():
        try:
            for _ in range(n):
                assert (eng.step(chunk) if engine else sim.step(chunk)) == D.DEM_OK
        finally:
            done.set()

    def reader():
        while not done.is_set():
            got = sim.read_state(FIELDS)
            step = got.pop("step")
            assert _equal(got, {k: want[step][k] for k in got}), step
            sim.get_forcing()

    _together([stepper, reader, reader])
    got = sim.read_state(FIELDS, pairs=True)
    assert got["step"] == n * chunk and _equal(got, want[n * chunk])
