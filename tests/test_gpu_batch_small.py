"""Items of a batch that fill two slots of a workgroup or fewer take steps
without branches: equal to the row streaming step to the bit at the sizes
where that begins and ends, and as fast as a small item should be."""
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


@pytest.mark.parametrize("mode,prec", [("bsb", "fp16"), ("dsb", "bf16"), ("asb", "fp16")])
@pytest.mark.parametrize("M", [1, 2, 3, 9])
def test_two_slots_and_more_equal_the_row_step(M, mode, prec):
    # 512 threads: two slots end at 1024 positions (spins x groups of two
    # agents), 1024 threads (split_n = 1): at 2048
    qs = [_qubo(n, 2.5, n) for n in (1, 2, 63, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049)]
    kw = dict(agents=M, steps=131, dt=0.1 if mode == "asb" else 0.5, c0=0.1, seed=5)
    for tuning in ({}, dict(split_n=1)):
        s = sbt.DeviceBatchSolver(qs, mode, prec, sbt.solve_params(energy_every=50, **kw), want_agent_energy=True,
                                  want_agent_state=True, want_trace=True, tuning=sbt.batch_tuning(**tuning))
        s.run()
        r = s.result()
        for e, q in enumerate(qs):
            ref = sbt.solve(q, mode, kernel="stream_rows", event=e, want_state=True, **kw)
            assert np.array_equal(r["agent_x"][e], ref["x"]), q.n
            assert np.array_equal(r["agent_T"][e], (ref["x"] >= 0).astype(np.int8)), q.n


def test_small_items_step_like_a_single_solve():
    """An event of a batch that fills two slots takes no more per step than
    three times the resident solve of the same event, which is one wave (five
    times before)."""
    q = _qubo(64, 3.0, 1)
    batch = (_ms([q], 16, 8000) - _ms([q], 16, 2000)) / 6000
    single = []
    for steps in (2000, 8000):
        s = sbt.DeviceSolver(q, "bsb", sbt.solve_params(agents=16, steps=steps))
        s.run()
        t = []
        for _ in range(5):
            b, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            b.record()
            s.run()
            e.record()
            torch.cuda.synchronize()
            t.append(b.elapsed_time(e))
        single.append(min(t))
    assert batch <= 3.0 * (single[1] - single[0]) / 6000
