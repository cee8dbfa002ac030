"""The batched products' work list (batched_plan.h), compiled for the CPU: every
(target, source) of every system is covered once, and small systems beside a
large one do not multiply the items.  Runs without a GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HARNESS = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_harness")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("bp") / "batched_plan_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC",
                    os.path.join(HARNESS, "batched_plan_host.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.host_batched_plan.restype = ctypes.c_int64
    lib.host_batched_plan.argtypes = [ctypes.POINTER(ctypes.c_int64), ctypes.c_int, ctypes.c_int, ctypes.c_int,
                                      ctypes.c_int, ctypes.c_int64, ctypes.POINTER(ctypes.c_int),
                                      ctypes.POINTER(ctypes.c_int), ctypes.c_int64]

    def run(sizes, span, tile, mat):
        offs = np.r_[0, np.cumsum(np.asarray(sizes, dtype=np.int64))]
        whole = int(max(offs[-1] // span + 1, sum(-(-int(n) // span) for n in sizes)))
        parts = ctypes.c_int()
        buf = np.zeros((whole + 2 * 8192, 4), dtype=np.int32)
        n = lib.host_batched_plan(offs.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), len(sizes), span, tile, mat,
                                  whole, ctypes.byref(parts), buf.ctypes.data_as(ctypes.POINTER(ctypes.c_int)),
                                  buf.size)
        assert n <= buf.shape[0]
        return offs, whole, parts.value, buf[:n]
    run.lib = lib
    return run


CASES = [[1], [3, 700], [513, 64, 1, 2000, 129], [2000] * 16, [5000] + [20] * 1000, [2000] + [3] * 20000,
         [80] * 5000, [80] * 2000, [300] * 300, [1000] + [2] * 100000, [17000, 16000, 65, 64, 63]]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("span,tile,mat", [(256, 64, 0), (512, 64, 0), (256, 256, 0), (64, 64, 1), (64, 128, 1)])
def test_items_cover_every_share_once(plan, case, span, tile, mat):
    sizes = CASES[case]
    offs, whole, parts, items = plan(sizes, span, tile, mat)
    assert 1 <= parts <= 64 and len(items) <= whole + 8192
    assert np.unique(items[:, [2, 3]], axis=0).shape[0] == len(items)
    targets = {}
    for b, e, t, w in items[:30000].tolist():
        p, used = w % 256, w // 256
        length = plan.lib.host_share_tiles(-(-(e - b) // tile), used) * tile
        s0 = b + p * length
        assert p < used <= parts and (t - b) % span == 0 and b <= t < e
        assert s0 < e  # no empty shares
        assert (p + 1 == used) == (s0 + length >= e)  # the last one ends the system
        targets.setdefault(b, {}).setdefault((p, used), []).append(t)
    if len(items) <= 30000:
        for b, e in zip(offs, offs[1:]):
            got = targets[int(b)]
            used = next(iter(got))[1]
            assert sorted(got) == [(p, used) for p in range(used)]
            assert all(sorted(t) == list(range(int(b), int(e), span)) for t in got.values())


@pytest.mark.parametrize("parts", [1, 2, 3, 5, 8, 63, 64])
def test_shares_of_the_used_parts(plan, parts):
    """The kernels form a share's length from the number of shares used."""
    for tiles in range(1, 400):
        used = plan.lib.host_used_parts(tiles, parts)
        assert plan.lib.host_share_tiles(tiles, used) == plan.lib.host_share_tiles(tiles, parts)


def test_small_systems_stay_whole(plan):
    """Systems of one tile are one item to a span, whatever the largest one has;
    once the items fill the GPU, systems of few blobs stay whole."""
    _, _, parts, items = plan([5000] + [20] * 100, 256, 64, 0)
    assert parts > 16 and (items[items[:, 1] - items[:, 0] == 20][:, 3] == 256).all()
    for sizes in ([2000] + [3] * 20000, [80] * 5000, [80] * 2000, [280] * 250):
        _, _, parts, _ = plan(sizes, 256, 64, 0)
        assert parts == 1
    _, _, parts, items = plan([1000] + [80] * 2000, 256, 64, 0)
    assert parts > 1 and (items[items[:, 1] - items[:, 0] == 80][:, 3] == 256).all()
    _, _, parts, _ = plan([300] * 300, 64, 128, 1)
    assert parts == 1
    _, _, parts, _ = plan([2000] * 16, 256, 64, 0)
    assert parts == 32
