"""Runs of matrix-core dSB steps on the chip where blocks of 16 rows have no
couplings: the K-steps of the blocks after them take their own operands."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2402_14718_amd as sbt  # noqa: E402


def _qubo(n, degree, seed, without=0.0):
    """Random couplings; a share `without` of the 16-row blocks has none."""
    rng = np.random.default_rng(seed)
    m = n * degree // 2
    i, j = rng.integers(0, n, m), rng.integers(0, n, m)
    empty = rng.random((n + 15) // 16) < without
    keep = (i != j) & ~empty[i // 16] & ~empty[j // 16]
    b = sp.csr_matrix((rng.uniform(-1, 1, keep.sum()), (i[keep], j[keep])), shape=(n, n))
    b = sp.csr_matrix(b + b.T)
    b.sort_indices()
    return sbt.Qubo(n, rng.uniform(-0.5, 0.7, n), b.indptr.astype(np.int64),
                    b.indices.astype(np.int32), b.data.copy(), np.zeros((n, 3), np.int64))


# 768 blocks on 32 workgroups of eight waves: three blocks a wave, and with
# four in ten of them without couplings every pattern of the three occurs
@pytest.mark.parametrize("precision", ["fp32", "bf16x2", "fp8", "fp8_block", "bf16", "fp16"])
@pytest.mark.parametrize("n,M,without", [(12288, 130, 0.4), (8000, 64, 0.5), (12288, 8, 0.95)])
def test_blocks_without_couplings(n, M, without, precision):
    q = _qubo(n, 4, n, without)
    kw = dict(agents=M, steps=9, seed=7, c0=0.3, kernel="stream_mfma", precision=precision, want_state=True)
    ref = sbt.solve(q, "dsb", energy_every=1, **kw)  # a launch per step
    got = sbt.solve(q, "dsb", **kw)
    for k in ("x", "y", "T", "agent_energy", "best_agent"):
        assert np.array_equal(got[k], ref[k]), k
