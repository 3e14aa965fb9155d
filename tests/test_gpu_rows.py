"""The on-chip step loop (single solves and batches) where its layout
changes: slot and workgroup sizes, classes of row length, tails, odd agents.

The loop sums a row as the row streaming step does (one FP32 fused
multiply-add per coupling in CSR order, from the field), so states, spins
and checkpointed energies' spins have to be equal to the bit, for the batch
kernel too when the couplings are exact in its 16-bit form."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2402_14718_amd as sbt  # noqa: E402


def _qubo(n, hubs, seed, scale=1.0):
    """A path of n spins (rows of one or two couplings) and, per entry of
    `hubs`, one spin coupled to about that many others; couplings and biases
    are multiples of 1/8 up to 2, exact in every form."""
    rng = np.random.default_rng(seed)
    b = sp.lil_matrix((n, n))
    value = lambda: float(rng.integers(-16, 17)) / 8.0 or 0.5
    order = rng.permutation(n)
    for i, j in zip(order[:-1:1], order[1::1]):
        if rng.random() < 0.8:
            b[i, j] = value()
    for k, d in enumerate(hubs):
        i = order[(k * 7) % n]
        for j in rng.choice(n, size=min(d, n - 1), replace=False):
            if j != i:
                b[i, j] = value()
    b = sp.csr_matrix(b)
    b = sp.csr_matrix(sp.triu(b + b.T, 1))
    b = sp.csr_matrix(b + b.T)
    b.sort_indices()
    return sbt.Qubo(n, scale * (rng.integers(-8, 9, n) / 8.0), b.indptr.astype(np.int64),
                    b.indices.astype(np.int32), scale * b.data, np.zeros((n, 3), np.int64))


SHAPES = [(1, 3, []), (20, 32, []), (64, 1, [1, 2, 3]), (65, 100, [4, 5]), (128, 33, [8, 9]),
          (129, 257, [12, 13]), (512, 300, [16, 17, 3]), (513, 31, [2]), (1024, 257, [5, 4, 16]),
          (1025, 258, [14, 9, 5]), (2048, 3, [15, 15, 15]), (2049, 257, [18, 6]), (4096, 10, [48, 7]),
          (4097, 9, [12] * 40), (4097, 257, [12] * 40), (6144, 300, [22, 9]), (6145, 259, [30, 13, 7]),
          (8484, 300, [24, 12] + [7] * 90), (9216, 5, [70, 25] + [9] * 30), (9216, 257, [50] * 3)]


@pytest.mark.parametrize("mode", ["bsb", "dsb", "asb"])
@pytest.mark.parametrize("n,M,hubs", SHAPES)
def test_resident_rows_equal_the_row_streaming_step(n, M, hubs, mode):
    q = _qubo(n, hubs, n)
    kw = dict(agents=M, steps=131, dt=0.1 if mode == "asb" else 0.5, c0=0.15, seed=n + M, energy_every=13, want_state=True,
              want_trace=True)
    got = sbt.solve(q, mode, kernel="resident", **kw)
    ref = sbt.solve(q, mode, kernel="stream_rows", **kw)
    assert got["kernel"] == "resident" and ref["kernel"] != "resident"
    for k in ("x", "y", "T", "agent_energy", "best_agent", "energy"):
        assert np.array_equal(got[k], ref[k]), k
    # a checkpoint's energy is the same FP64 terms in another order
    scale = np.abs(q.a).sum() + np.abs(q.b).sum()
    assert np.max(np.abs(got["trace"] - ref["trace"])) <= (n + q.nnz) * 2.0 ** -53 * scale


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("mode", ["bsb", "dsb"])
def test_batch_rows_equal_single_solves_with_exact_couplings(mode, prec):
    M, kw = 100, dict(dt=0.5, c0=0.15, seed=5)
    qs = [_qubo(n, hubs, n) for n, _, hubs in SHAPES]
    states = []
    for tuning in ({}, dict(fill=0.25), dict(split_n=1), dict(split_n=4608, tail_words=0)):
        s = sbt.DeviceBatchSolver(qs, mode, prec, sbt.solve_params(agents=M, steps=64, **kw),
                                  want_agent_energy=True, want_agent_state=True,
                                  tuning=sbt.batch_tuning(**tuning))
        s.run()
        states.append(s.result())
    for e, q in enumerate(qs):
        ref = sbt.solve(q, mode, kernel="stream_rows", agents=M, steps=64, event=e, want_state=True,
                        **kw)
        for r in states:
            assert np.array_equal(r["agent_x"][e], ref["x"]), e
            # agents with the same spins have the same energy, whatever
            # workgroup they ran in, so a tie falls to the lowest
            T, E = np.asarray(r["agent_T"][e]), np.asarray(r["agent_energy"][e])
            _, which = np.unique(T, axis=1, return_inverse=True)
            for g in range(which.max() + 1):
                assert np.unique(E[which.ravel() == g]).size == 1
            assert np.array_equal(E, states[0]["agent_energy"][e])
            assert r["best_agent"][e] == np.argmin(E)


@pytest.mark.parametrize("n,per_spin,kernel", [(128, 100, "resident"), (1000, 12, "resident"),
                                               (1000, 40, "stream"), (4096, 7, "resident"),
                                               (4096, 10, "stream"), (9216, 3, "resident"),
                                               (9216, 6, "stream"), (9217, 2, "stream")])
def test_auto_takes_the_loop_while_couplings_fit_and_equals_the_row_step(n, per_spin, kernel):
    hubs = [min(250, n - 1)] * max(0, int((per_spin - 2) * n / 2 / min(250, n - 1)))
    q = _qubo(n, hubs, n)
    kw = dict(agents=40, steps=40, dt=0.5, c0=0.15, seed=n, want_state=True)
    got = sbt.solve(q, "bsb", **kw)
    ref = sbt.solve(q, "bsb", kernel="stream_rows", **kw)
    assert got["kernel"] == kernel, q.nnz / n
    for k in ("x", "y", "T", "agent_energy", "best_agent"):
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("scale", [2.0 ** -18, 2.0 ** 20])
@pytest.mark.parametrize("mode", ["bsb", "dsb"])
def test_batch_bf16_couplings_that_are_no_fp16_values(mode, scale):
    # BF16 values below or above the range of FP16, beside an event within it
    qs = [_qubo(300, [20], 1, scale), _qubo(300, [20], 1), _qubo(5000, [18, 6], 2, scale)]
    M, kw = 24, dict(steps=64, dt=0.5, seed=5)
    for k, q in enumerate(qs):
        c0 = 0.15 / (1.0 if k == 1 else scale)
        s = sbt.DeviceBatchSolver(qs, mode, "bf16", sbt.solve_params(agents=M, c0=c0, **kw),
                                  want_agent_energy=True, want_agent_state=True)
        s.run()
        got = s.result()["agent_x"][k]
        ref = sbt.solve(q, mode, kernel="stream_rows", agents=M, event=k, c0=c0, want_state=True, **kw)
        assert np.array_equal(got, ref["x"])


@pytest.mark.parametrize("kernel,mode,steps", [("stream", "bsb", 20), ("stream", "bsb", 21), ("stream", "dsb", 20),
                                               ("stream_mfma", "dsb", 20), ("resident", "bsb", 20)])
def test_final_state_in_arrays_aligned_to_four_bytes(kernel, mode, steps):
    q = _qubo(513, [9], 3)
    s = sbt.DeviceSolver(q, mode, sbt.solve_params(agents=72, steps=steps, kernel=kernel, seed=2), want_state=True)
    s.run()
    torch.cuda.synchronize()
    x, y = s.x.clone(), s.y.clone()
    n = x.numel()
    bx, by = torch.zeros(n + 2, device="cuda"), torch.zeros(n + 2, device="cuda")
    s._dr.x_final, s._dr.y_final = bx.data_ptr() + 4, by.data_ptr() + 4
    s.run()
    torch.cuda.synchronize()
    for base, want in ((bx, x), (by, y)):
        assert torch.equal(base[1:n + 1], want.reshape(-1))
        assert base[0] == 0 and base[n + 1] == 0
