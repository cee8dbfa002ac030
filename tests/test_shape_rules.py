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
