"""Runs of matrix-core dSB steps on the chip where blocks of 16 rows have no
couplings (the K-steps of the blocks after them take their own operands), and
where a gang's workgroups never run at once."""
import ctypes as C

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


def _masked_stream():
    """A stream for 16 compute units, two of each XCD however the mask's bits
    go round them."""
    lib = sbt.load()
    mask = (C.c_uint32 * 8)(*[3 << (2 * (w % 4)) for w in range(8)])
    s = C.c_void_p()
    assert lib.hipExtStreamCreateWithCUMask(C.byref(s), C.c_uint32(8), mask) == 0
    return lib, s


@pytest.mark.parametrize("precision", ["fp32", "fp8"])
def test_solve_captured_for_the_device_and_replayed_on_sixteen_units(precision):
    """A gang of 32 workgroups never runs at once there: its wait ends, and
    every output is still that of the solve on the whole device."""
    q = _qubo(8493, 3, 4)
    p = sbt.solve_params(agents=300, steps=30, energy_every=12, kernel="stream_mfma", precision=precision, seed=2)
    ds = sbt.DeviceSolver(q, "dsb", p, want_state=True, want_trace=True)
    keys = ("x", "y", "T", "agent_energy", "best_agent", "energy", "trace", "agent_trace")
    ds.run()
    ref = ds.result()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ds.run()
    lib, s = _masked_stream()
    try:
        st = torch.cuda.ExternalStream(s.value)
        for replay in (False, True, True):
            for v in (ds.x, ds.y, ds.T, ds.agent_energy, ds.trace, ds.agent_trace):
                v.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(st):
                g.replay() if replay else ds.run()
            torch.cuda.synchronize()
            got = ds.result()
            for k in keys:
                assert np.array_equal(got[k], ref[k]), (replay, k)
    finally:
        torch.cuda.synchronize()
        lib.hipStreamDestroy(s)
