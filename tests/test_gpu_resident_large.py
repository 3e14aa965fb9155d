"""The LDS-row resident kernel (on request, events past the step loop's shapes):
equal to the row streaming step to the bit at the ends of its range, with the
couplings in LDS and in memory."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2402_14718_amd as sbt  # noqa: E402


@pytest.mark.parametrize("mode", ["bsb", "dsb", "asb"])
@pytest.mark.parametrize("n,pairs", [(9217, 2000), (9217, 30000), (16383, 500), (16384, 20000)])
def test_equals_the_row_step(n, pairs, mode):
    rng = np.random.default_rng(n + pairs)
    i, j = rng.integers(0, n, pairs), rng.integers(0, n, pairs)
    b = sp.csr_matrix((rng.uniform(-1, 1, pairs), (i, j)), shape=(n, n))
    b = sp.csr_matrix(sp.triu(b + b.T, 1))
    b = sp.csr_matrix(b + b.T)
    b.sort_indices()
    q = sbt.Qubo(n, rng.uniform(-0.5, 0.5, n), b.indptr.astype(np.int64), b.indices.astype(np.int32), b.data.copy(),
                 np.zeros((n, 3), np.int64))
    kw = dict(agents=3, steps=50, dt=0.1 if mode == "asb" else 0.5, c0=0.2, seed=n, energy_every=25, want_state=True)
    got = sbt.solve(q, mode, kernel="resident", **kw)
    ref = sbt.solve(q, mode, kernel="stream_rows", **kw)
    assert got["kernel"] == "resident"
    for k in ("x", "y", "T", "agent_energy", "best_agent"):
        assert np.array_equal(got[k], ref[k]), k
