"""Rules of the built-in launch shapes at their edges.  Host code: no GPU needed."""
import os

import pytest

from paper_1709_02410_amd import rpywall


@pytest.fixture(scope="module")
def rp():
    if not os.path.exists(rpywall.LIB_PATH):
        pytest.skip("librpywall.so not built")
    rpywall.lib()
    return rpywall


@pytest.mark.parametrize("k", [5, 6])
def test_five_and_six_fp64_right_hand_sides(rp, k):
    """One block of 8 where that is the faster form, a block of 4 and the rest
    above; the rest of five over groups of 64 like one right-hand side."""
    for N in (300, 600, 1537, 2000, 2049, 3000, 3328):
        assert rp.get_shape(0, N, k)["kblk"] == 8, N
    for N in (3329, 3583, 3584, 20000, 32768):
        s = rp.get_shape(0, N, k)
        assert (s["kblk"], s["sym"]) == (4, 2), N
    assert rp.get_shape(0, 131072, k)["kblk"] == 4 and rp.get_shape(0, 131073, k)["kblk"] == 8
    assert all(rp.get_shape(0, N, 7)["kblk"] == 8 for N in (2000, 5000, 50000))


def test_workspace_holds_no_partials_of_kernels_that_cannot_run(rp):
    """FP64 blocks of two and four right-hand sides have one symmetric kernel, up
    to 131072 blobs; beyond it what is left of the bound is that of one."""
    ws = lambda N, k: rp.workspace_bytes(rp.OP_MATVEC, N, k, precision=0)  # noqa: E731
    for N in (131073, 200000, 400000):
        for k in (2, 4, 8, 16):
            assert ws(N, k) < 1.1 * ws(N, 1), (N, k)
    assert ws(131072, 4) > 4 * ws(131073, 4)
