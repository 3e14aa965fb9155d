"""Runs of matrix-core dSB steps with the state on the chip, against the same
steps one launch at a time (which a checkpoint after every step asks for):
the arithmetic is the same, so states and spins are equal to the bit."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2402_14718_amd as sbt  # noqa: E402


def _qubo(n, degree, seed):
    rng = np.random.default_rng(seed)
    m = n * degree // 2
    i, j = rng.integers(0, n, m), rng.integers(0, n, m)
    keep = i != j
    b = sp.csr_matrix((rng.uniform(-1, 1, keep.sum()), (i[keep], j[keep])), shape=(n, n))
    b = sp.csr_matrix(b + b.T)
    b.sort_indices()
    return sbt.Qubo(n, rng.uniform(-0.5, 0.7, n), b.indptr.astype(np.int64),
                    b.indices.astype(np.int32), b.data.copy(), np.zeros((n, 3), np.int64))


# one to three tiles a wave, ragged rows and agents, more groups than run at
# once, blocks without couplings, more listed columns than one chunk
@pytest.mark.parametrize("precision", ["fp32", "bf16x2", "fp8", "fp8_block", "bf16", "fp16"])
@pytest.mark.parametrize("n,M,degree", [(16, 1, 0), (95, 130, 3), (1480, 256, 4), (4111, 1030, 5), (8493, 1024, 3),
                                        (12288, 1000, 2), (3000, 128, 40)])
def test_run_on_the_chip_equals_single_steps(n, M, degree, precision):
    q = _qubo(n, degree, n)
    kw = dict(agents=M, steps=21, seed=7, kernel="stream_mfma", precision=precision, want_state=True)
    ref = sbt.solve(q, "dsb", energy_every=1, **kw)
    for every in (0, 8):
        got = sbt.solve(q, "dsb", energy_every=every, want_trace=every > 0, **kw)
        for k in ("x", "y", "T", "agent_energy", "best_agent"):
            assert np.array_equal(got[k], ref[k]), (every, k)


def test_runs_on_several_streams_at_once():
    q = _qubo(8493, 3, 4)
    kw = dict(agents=300, steps=40, kernel="stream_mfma")
    want = [sbt.solve(q, "dsb", seed=s, want_state=True, **kw) for s in range(4)]
    solvers = [sbt.DeviceSolver(q, "dsb", sbt.solve_params(seed=s, **kw), want_state=True) for s in range(4)]
    streams = [torch.cuda.Stream() for _ in solvers]
    torch.cuda.synchronize()
    for _ in range(3):
        for s, st in zip(solvers, streams):
            s.run(st)
    torch.cuda.synchronize()
    for s, w in zip(solvers, want):
        assert np.array_equal(s.x.cpu().numpy(), w["x"])
        assert np.array_equal(s.agent_energy.cpu().numpy(), w["agent_energy"])
