"""Batches of events whose rows are longer than a thread holds: shapes of one
and two agents per word, items of two slots and of nine, lists in LDS and
couplings read from memory, against the row streaming step, which sums a row
in the same order (equal to the bit where the couplings are exact in 16 bits)."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2402_14718_amd as sbt  # noqa: E402


def _qubo(n, per_spin, seed):
    """Random pairs, about per_spin couplings a spin; multiples of 1/8."""
    rng = np.random.default_rng(seed)
    m = int(n * per_spin / 2)
    i, j = rng.integers(0, n, m), rng.integers(0, n, m)
    b = sp.csr_matrix((rng.integers(1, 17, m) / 8.0 * rng.choice([-1, 1], m), (i, j)), shape=(n, n))
    b = sp.csr_matrix(sp.triu(b + b.T, 1))
    b.data = np.clip(b.data, -2, 2)
    b.eliminate_zeros()
    b = sp.csr_matrix(b + b.T)
    b.sort_indices()
    return sbt.Qubo(n, rng.integers(-8, 9, n) / 8.0, b.indptr.astype(np.int64), b.indices.astype(np.int32),
                    b.data.copy(), np.zeros((n, 3), np.int64))


EVENTS = [(30, 8.0), (200, 12.0), (511, 24.0), (512, 4.0), (1024, 10.0), (1025, 18.0), (2048, 9.0), (2049, 14.0),
          (3000, 30.0), (4608, 4.2), (4608, 7.0), (4609, 5.0), (6145, 6.0), (9216, 3.7), (9216, 5.5)]


@pytest.mark.parametrize("mode,prec", [("bsb", "fp16"), ("dsb", "bf16"), ("asb", "fp16"), ("dsb", "fp16")])
@pytest.mark.parametrize("M", [1, 6, 33])
def test_long_rows_equal_the_row_step(M, mode, prec):
    qs = [_qubo(n, r, n) for n, r in EVENTS]
    kw = dict(agents=M, steps=40, dt=0.1 if mode == "asb" else 0.5, c0=0.05, seed=5)
    runs = []
    for tuning in ({}, dict(tail_words=0), dict(split_n=1, tail_words=2048), dict(fill=0.3)):
        s = sbt.DeviceBatchSolver(qs, mode, prec, sbt.solve_params(energy_every=15, **kw), want_agent_energy=True,
                                  want_agent_state=True, want_trace=True, tuning=sbt.batch_tuning(**tuning))
        s.run()
        runs.append(s.result())
    for e, q in enumerate(qs):
        ref = sbt.solve(q, mode, kernel="stream_rows", event=e, want_state=True, **kw)
        for r in runs:
            assert np.array_equal(r["agent_x"][e], ref["x"]), EVENTS[e]
            assert np.array_equal(r["agent_trace"][e], runs[0]["agent_trace"][e]), EVENTS[e]
            assert np.array_equal(r["agent_energy"][e], runs[0]["agent_energy"][e]), EVENTS[e]
            assert r["best_agent"][e] == np.argmin(r["agent_energy"][e])


def _ms(qs, M, steps, **tuning):
    s = sbt.DeviceBatchSolver(qs, "bsb", "fp16", sbt.solve_params(agents=M, steps=steps), tuning=sbt.batch_tuning(**tuning))
    s.run()
    best = float("inf")
    for _ in range(5):
        b, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        b.record()
        s.run()
        e.record()
        torch.cuda.synchronize()
        best = min(best, b.elapsed_time(e))
    return best


@pytest.mark.parametrize("n,per_spin,M", [(64, 8.0, 100), (2000, 8.0, 1), (4000, 6.0, 16), (4000, 4.5, 100)])
def test_the_chosen_schedule_is_near_the_best_of_others(n, per_spin, M):
    """(2.3 to 3.6 times the best of these where only the size of an event
    chose its shape.)"""
    qs = [_qubo(n, per_spin, k) for k in range(16)]
    chosen = _ms(qs, M, 400)
    others = [_ms(qs, M, 400, **t) for t in (dict(split_n=1), dict(split_n=1, fill=0.25), dict(fill=0.25))]
    assert chosen <= 1.6 * min(others), (chosen, others)
