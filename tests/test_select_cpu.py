"""AUTO's choice on shapes of half the LDS (a hint of 256 or 512 threads): the
on-chip loop while registers and the list hold the couplings, as many words as
the kernel's own LDS leaves."""
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
