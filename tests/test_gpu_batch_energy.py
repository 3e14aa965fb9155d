"""Energies of a batch: a checkpoint's are the final ones of its state, a
target taken from them is reached, and the number of events is not bounded by
a launch's grid."""
import numpy as np
import pytest
import scipy.sparse as sp

import trackgen as tg
from oracle import energy as oenergy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2402_14718_amd as sbt  # noqa: E402


def _scaled(q, s):
    return sbt.Qubo(q.n, q.a * s, q.row_ptr, q.col, q.b * s, q.trip_hits)


@pytest.fixture(scope="module")
def qubos():
    """20 to ~6000 spins; one of very small and one of very large terms."""
    qs = [sbt.build_qubo(tg.generate(tg.plain_spec(p), 100 + p).hits_struct())
          for p in (15, 30, 60, 100, 150, 250, 400, 950)]
    return qs + [_scaled(qs[3], 1e-200), _scaled(qs[4], 1e200)]


def _run(qs, M, mode="dsb", prec="bf16", target=None, **tuning):
    s = sbt.DeviceBatchSolver(qs, mode, prec, sbt.solve_params(agents=M, steps=120, seed=3, c0=0.3,
                                                               energy_every=20),
                              want_agent_energy=True, want_trace=True, want_agent_state=True, target=target,
                              tuning=sbt.batch_tuning(**tuning))
    s.run()
    return s.result()


@pytest.mark.parametrize("M", [1, 33, 100])
def test_checkpoint_energies_are_the_final_ones_and_targets_are_reached(qubos, M):
    qs = qubos[:8]
    ref = _run(qs, M)
    for tuning in ({}, dict(split_n=1), dict(fill=0.2, split_n=600)):
        r = _run(qs, M, **tuning)
        hit = _run(qs, M, target=ref["energy"], **tuning)
        for e, q in enumerate(qs):
            assert np.array_equal(r["agent_trace"][e], ref["agent_trace"][e]), e
            assert np.array_equal(r["agent_trace"][e][-1], r["agent_energy"][e]), e
            assert r["best_agent"][e] == np.argmin(r["agent_energy"][e])
            # the run with this target stops at or before the state that set it
            assert hit["energy"][e] <= ref["energy"][e], e
            assert hit["trace"][e][-1] <= ref["energy"][e], e


def test_energies_to_rounding_of_the_oracle(qubos):
    r = _run(qubos, 40)
    for e, q in enumerate(qubos):
        b = sp.csr_matrix((q.b, q.col, q.row_ptr), shape=(q.n, q.n))
        want = oenergy.qubo_energy(q.a, b, np.asarray(r["agent_T"][e]))
        # a row's term is rounded once per coupling, the sum once
        row = np.abs(q.a) + np.asarray(np.abs(b).sum(axis=1)).ravel()
        tol = 2.0 ** -52 * (np.diff(q.row_ptr).max() + 2) * row.sum()
        assert np.max(np.abs(r["agent_energy"][e] - want)) <= tol, e


def test_more_events_than_a_grid_dimension_holds():
    """70000 events of two spins: each ends in one of its four states, whose
    energy is known."""
    rp, col = np.array([0, 1, 2]), np.array([1, 0], np.int32)
    qs = [sbt.Qubo(2, np.array([-0.5 - 0.25 * (k % 3), 0.25]), rp, col, np.full(2, -0.5 + (k % 2)),
                   np.zeros((2, 3), np.int64)) for k in range(6)]
    E = 70000
    s = sbt.DeviceBatchSolver([qs[k % 6] for k in range(E)], "bsb", "fp16", sbt.solve_params(agents=2, steps=30),
                              want_agent_energy=True, want_agent_state=True)
    s.run()
    r = s.result()
    T = s.agent_T.cpu().numpy().reshape(E, 2, 2).astype(np.float64)
    a = np.array([q.a for q in qs])[np.arange(E) % 6]
    b = np.array([q.b[0] for q in qs])[np.arange(E) % 6]
    want = a[:, 0, None] * T[:, 0] + a[:, 1, None] * T[:, 1] + b[:, None] * T[:, 0] * T[:, 1]
    assert np.array_equal(r["agent_energy"], want)
    assert np.array_equal(r["energy"], want.min(axis=1))


@pytest.mark.parametrize("M", [3, 70])
def test_energies_apart_from_the_step_kernel_are_its_own(qubos, M):
    """Batches of many items sum the final energies in a launch of their own;
    a run that ends at a checkpoint has them from the step kernel."""
    qs = (qubos + [sbt.build_qubo(tg.generate(tg.plain_spec(1200), 77).hits_struct())]) * (120 if M == 3 else 10)
    kw = dict(want_agent_energy=True, want_agent_state=True, tuning=sbt.batch_tuning(split_n=1, fill=0.02))
    runs = []
    for every in (0, 20, 9):  # (9: the last checkpoint is not the end)
        s = sbt.DeviceBatchSolver(qs, "dsb", "bf16", sbt.solve_params(agents=M, steps=20, seed=3, c0=0.3, energy_every=every),
                                  **kw)
        for _ in range(2):
            s.run()
        runs.append(s.result())
    # more than eight items per workgroup, beside the gangs' two bands per agent
    assert s.n_items - 2 * M * sum(q.n > 9216 for q in qs) > 8 * 256
    for r in (runs[0], runs[2]):
        for k in ("agent_energy", "energy", "best_agent"):
            gang = np.array([q.n > 9216 for q in qs])
            assert np.array_equal(r[k][~gang], runs[1][k][~gang]), k
            assert np.allclose(r[k][gang], runs[1][k][gang], rtol=1e-12)
