"""Choices made on the host.  AUTO on shapes of half the LDS (a hint of 256 or
512 threads): the on-chip loop while registers and the list hold the couplings,
as many words as the kernel's own LDS leaves.  The tuner: splits that plan
different items."""
import pytest

import paper_2402_14718_amd as sbt


# list: (81920 - 1024 - 16 threads - 12 x 9 x threads) / 4 words, two a coupling
@pytest.mark.parametrize("n,tpb,mode,held,words", [
    (1500, 256, "bsb", 256 * (16 + 8 + 5 + 4 + 3 + 2), 12288), (1500, 256, "dsb", 256 * (12 + 6 + 4 + 3 + 2 + 2), 12288),
    (3000, 512, "bsb", 512 * (16 + 8 + 5 + 4 + 3 + 2), 4352), (3000, 512, "asb", 512 * (16 + 8 + 5 + 4 + 3 + 2), 4352)])
def test_hinted_shapes_leave_the_chip_where_their_list_ends(n, tpb, mode, held, words):
    kernel = lambda nnz: sbt.select_kernel(n, nnz, 40, mode, sbt.solve_params(agents=32, steps=10, tpb=tpb))
    assert kernel(held + words // 2) == "resident"
    assert kernel(held + words // 2 + 1) == "stream"
    assert kernel(4 * n) == "resident"


def test_the_tuner_tries_schedules_that_differ():
    """Each split of the shapes plans another number of items (seen in the
    workspace that they take)."""
    import ctypes as C

    import numpy as np

    from paper_2402_14718_amd import autotune
    n = np.array([90, 300, 800, 1500, 3000, 6000] * 60, np.int32)
    nnz = (2 * n).astype(np.int64)
    p = sbt.solve_params(agents=128, steps=10)
    sizes = []
    for split in autotune.SPLITS:
        t = sbt.batch_tuning(split_n=split)
        sizes.append(sbt.load().sbt_batch_workspace_bytes_tuned(
            n.ctypes.data_as(C.POINTER(C.c_int32)), nnz.ctypes.data_as(C.POINTER(C.c_int64)), n.size, C.byref(p), C.byref(t)))
    assert len(set(sizes)) == len(autotune.SPLITS), dict(zip(autotune.SPLITS, sizes))
