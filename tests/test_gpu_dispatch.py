"""Which kernel a call takes: rules of the dispatch at their edges, against the
FP64 oracle or against the same call through a fixed launch shape.  Bars: those
of the two precisions (FP64 1e-12, FP32C 1e-5, relative L2 and largest entry)."""
import numpy as np
import pytest

from parity_util import check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: 1e-5}


@pytest.fixture(scope="module")
def rp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_02410_amd import rpywall
    rpywall.lib()
    return rpywall


def _t(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _mixed(n, seed):
    """Blobs above and below z = a, overlapping pairs, one coincident pair."""
    rng = np.random.default_rng(seed)
    box = max(2.0, 2.0 * np.sqrt(n))
    pos = np.column_stack([rng.uniform(0, box, n), rng.uniform(0, box, n), rng.uniform(0.3, 4.0, n)])
    if n >= 3:
        pos[2] = pos[1]
    return pos


@pytest.mark.parametrize("N,k", [(1, 1), (300, 1), (300, 9), (1000, 1), (1280, 16), (2000, 4), (2048, 1)])
@pytest.mark.parametrize("prec", [0, 1])
def test_velocities_on_top_of_forces(rp, orc, N, k, prec):
    """out = F: all forces are read before the first velocity is written, also
    at the sizes of the one-launch products."""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + k).standard_normal((k, N, 3))
    U = _t(F)
    rp.matvec_multi(_t(pos), U, 0.9, 1.3, precision=prec, out=U)
    for j in {0, k // 2, k - 1}:
        check(U[j].cpu().numpy(), orc.matvec(pos, F[j], 0.9, 1.3), TOL[prec], f"in place N={N} k={k} rhs {j}")
    if k == 1:
        u = _t(F[0])
        rp.matvec_noalloc(_t(pos), u, 0.9, 1.3, precision=prec, out=u)
        check(u.cpu().numpy(), orc.matvec(pos, F[0], 0.9, 1.3), TOL[prec], f"in place, noalloc N={N}")


@pytest.mark.parametrize("prec,k", [(0, 1), (0, 8), (0, 16), (1, 1), (1, 16)])
def test_batched_small_systems_beside_a_large_one(rp, orc, prec, k):
    """Systems of fewer shares than the largest one's parts: the sums of the
    parts that they do not use are zero whatever the workspace held."""
    sizes = [2500] + [1, 5, 64, 65, 130, 700] * 4
    offs = np.r_[0, np.cumsum(sizes)]
    pos = np.concatenate([0.9 * _mixed(n, n) for n in sizes])
    F = np.random.default_rng(k).standard_normal((k, offs[-1], 3))
    junk = torch.full((1 << 26,), float("nan"), dtype=torch.float64, device="cuda")
    del junk  # the allocator hands this memory to the call's workspace
    U = rp.matvec_batched(_t(pos), offs, _t(F), 0.9, 1.3, precision=prec).cpu().numpy()
    for a, b in zip(offs, offs[1:8]):
        for j in {0, k - 1}:
            check(U[j, a:b], orc.matvec(pos[a:b], F[j, a:b], 0.9, 1.3), TOL[prec], f"system of {b - a} k={k} rhs {j}")


@pytest.mark.parametrize("sizes", [(700, 40), (3000, 1, 520)])
@pytest.mark.parametrize("prec,k", [(0, 5), (0, 6), (0, 7), (1, 5)])
def test_batched_five_and_six_right_hand_sides(rp, orc, sizes, prec, k):
    """One pass over the pairs, as for 7 and 8, in a block of 8."""
    offs = np.r_[0, np.cumsum(sizes)]
    pos = np.concatenate([0.9 * _mixed(n, n) for n in sizes])
    F = np.random.default_rng(k).standard_normal((k, offs[-1], 3))
    rp.profile_enable(True)
    try:
        rp.profile_read(reset=True)
        U = rp.matvec_batched(_t(pos), offs, _t(F), 0.9, 1.3, precision=prec).cpu().numpy()
        launches = rp.profile_read(reset=True)[1]
    finally:
        rp.profile_enable(False)
    assert launches == 1
    for a, b in zip(offs, offs[1:]):
        for j in (0, 3, k - 1):
            check(U[j, a:b], orc.matvec(pos[a:b], F[j, a:b], 0.9, 1.3), TOL[prec], f"system of {b - a} k={k} rhs {j}")


@pytest.mark.parametrize("N", [1537, 2049, 3328, 3329, 3583, 3584])
@pytest.mark.parametrize("k", [5, 6])
def test_five_and_six_right_hand_sides(rp, orc, N, k):
    """FP64, both sides of the line between one block of 8 and 4 + the rest,
    whose single right-hand side takes groups of 64 and of 128."""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + k).standard_normal((k, N, 3))
    U = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=0).cpu().numpy()
    for j in (0, 3, k - 1):
        check(U[j], orc.matvec(pos, F[j], 0.9, 1.3), TOL[0], f"N={N} k={k} rhs {j}")


TUNED_PROBE = """
import sys
sys.path.insert(0, {root!r})
import numpy as np, torch
from paper_1709_02410_amd import rpywall as rp
def t(x): return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
def cloud(n):
    rng = np.random.default_rng(n)
    b = 2.0 * np.sqrt(n)
    return t(np.column_stack([rng.uniform(0, b, n), rng.uniform(0, b, n), rng.uniform(0.3, 4.0, n)]))
{body}
"""


def _tuned_probe(body, env=None):
    """body in a process of its own: tuned shapes last as long as the process."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    e = {k: v for k, v in os.environ.items() if not k.startswith("RPYW_")}
    r = subprocess.run([sys.executable, "-c", TUNED_PROBE.format(root=root, body=body)], env={**e, **(env or {})},
                       capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], flush=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return r


def test_tuned_fp64_shapes_keep_the_other_calls_on_groups_of_64(rp):
    """The tuner at a size where every symmetric FP64 product is the kernel over
    groups of 128: what else reads the shape stays over groups of 64."""
    _tuned_probe('''
for n, k in ((3840, 1), (20000, 1), (3400, 5)):
    p = cloud(n)
    rp.autotune(p, torch.ones((k, n, 3), dtype=torch.float64, device="cuda"), precision=0)
    s = rp.get_shape(0, n, k)
    print(n, k, s, flush=True)
    assert s["sym"] != 1, s
''')


def test_small_fp64_products_obey_tuned_and_environment_shapes(rp, tmp_path):
    """The one-launch products are the built-in choice and a candidate of the
    tuner; a tuned shape without them, and RPYW_TILE or RPYW_RHS_WIDTH, are the
    shape that runs: to the bit the product with that shape fixed."""
    import json
    path = tmp_path / "shapes.json"
    body = '''
import json, os
out = {{}}
for n, k in ((300, 1), (1000, 1), (1000, 2)):
    f = torch.ones((k, n, 3), dtype=torch.float64, device="cuda")
    out[n, k] = rp.matvec_multi(cloud(n), f)
    s = rp.get_shape(0, n, k)
    rp.set_shape(0, n, k, **s)
    fixed = rp.matvec_multi(cloud(n), f)
    rp.reset_shape(0, n, k)
    assert torch.equal(out[n, k], fixed) == {obeys}, (n, k, s)
vjp = rp.matvec_vjp(cloud(300), out[300, 1][0], out[300, 1][0])
rp.set_shape(0, 300, 1, tpl=1, tile=64, kblk=1, sym=0, ipw=4)
assert torch.equal(vjp[0], rp.matvec_vjp(cloud(300), out[300, 1][0], out[300, 1][0])[0]) == {obeys}
rp.reset_shape(0, 300, 1)
if {tune}:
    for n, k in out: rp.autotune(cloud(n), torch.ones((k, n, 3), dtype=torch.float64, device="cuda"), precision=0)
    for n, k in out:  # far faster than the other kernels here
        assert torch.equal(out[n, k], rp.matvec_multi(cloud(n), torch.ones((k, n, 3), dtype=torch.float64, device="cuda")))
'''
    cache = {"RPYW_AUTOTUNE_CACHE": str(path)}
    _tuned_probe(body.format(obeys=False, tune=True), cache)  # the default, then tuned
    entries = json.loads(path.read_text())["entries"]
    assert len(entries) == 3 and all(e["direct"] == 1 for e in entries)
    _tuned_probe(body.format(obeys=False, tune=False), cache)  # from the file
    for e in entries:
        e.update(direct=0, sym=0, tpl=1, tile=64, ipw=4, kblk=1)
    path.write_text(json.dumps({"version": 1, "entries": entries}))
    _tuned_probe(body.format(obeys=True, tune=False), cache)
    for e in entries:
        del e["direct"], e["ipw2"]  # a file of an earlier version
    path.write_text(json.dumps({"version": 1, "entries": entries}))
    _tuned_probe(body.format(obeys=True, tune=False), cache)
    _tuned_probe(body.format(obeys=True, tune=False), {"RPYW_TILE": "256"})


def _other_calls(rp, n):
    """What else reads the FP64 shape of one right-hand side: VJP, periodic
    product, and the product of a smaller problem of the size class."""
    pos, f = _t(_mixed(n, n)), _t(np.random.default_rng(n).standard_normal((n, 3)))
    return (*rp.matvec_vjp(pos, f, f), rp.matvec_periodic(pos, f[None], (250.0, 260.0)))


@pytest.mark.parametrize("N", [8300, 16500])
def test_source_groups_of_the_128_kernel_are_its_own(rp, N):
    """FP64 products over groups of 128 take two source groups to a workgroup
    here, VJPs and periodic products over groups of 64 one: their sums are to
    the bit those of that shape."""
    assert rp.get_shape(0, N, 1)["ipw"] == 2
    got = _other_calls(rp, N)
    rp.set_shape(0, N, 1, tpl=1, tile=256, kblk=1, sym=2, ipw=1)
    try:
        ref = _other_calls(rp, N)
    finally:
        rp.reset_shape(0, N, 1)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


def test_tuning_leaves_the_other_calls_alone(rp, tmp_path):
    """... also after a tuning (of the groups of 128), and from its cache file."""
    body = '''
def other(n):
    p, f = cloud(n), torch.ones((n, 3), dtype=torch.float64, device="cuda")
    return (*rp.matvec_vjp(p, f, f), rp.matvec_periodic(p, f[None], (250.0, 260.0)))
before = other(3840), other(9000), rp.matvec(cloud(3000), torch.ones((3000, 3), dtype=torch.float64, device="cuda"))
if {tune}:
    for n in (3840, 9000):
        rp.autotune(cloud(n), torch.ones((1, n, 3), dtype=torch.float64, device="cuda"), precision=0)
for n in (3840, 9000): print(n, rp.get_shape(0, n, 1), flush=True)
after = other(3840), other(9000), rp.matvec(cloud(3000), torch.ones((3000, 3), dtype=torch.float64, device="cuda"))
flat = lambda x: [z for y in x for z in (y if isinstance(y, tuple) else (y,))]
if {tune}: torch.save(flat(before), {file!r})
assert all(torch.equal(a, b) for a, b in zip(flat(after), torch.load({file!r})))
'''
    env = {"RPYW_AUTOTUNE_CACHE": str(tmp_path / "shapes.json")}
    first = _tuned_probe(body.format(tune=True, file=str(tmp_path / "ref.pt")), env)
    again = _tuned_probe(body.format(tune=False, file=str(tmp_path / "ref.pt")), env)
    assert first.stdout == again.stdout


@pytest.mark.parametrize("N", [500, 3000, 3400, 9000, 33000])
@pytest.mark.parametrize("k", [2, 4, 5, 9])
def test_calls_fit_the_workspace_that_they_ask_for(rp, N, k):
    """FP64, every symmetric shape (the binding passes exactly the bytes of the
    query; too few would raise), with the sums of single products."""
    pos, F = _t(_mixed(N, N)), _t(np.random.default_rng(N).standard_normal((k, N, 3)))
    ref = rp.matvec(pos, F[k - 1].contiguous(), precision=0).cpu().numpy()
    check(rp.matvec_multi(pos, F, precision=0)[k - 1].cpu().numpy(), ref, 1e-12, f"N={N} k={k}")
    for kblk in (1, 2, 4):
        for sym in (1, 2):
            rp.set_shape(0, N, k, tpl=1, tile=256, kblk=kblk, sym=sym, ipw=1)
            try:
                U = rp.matvec_multi(pos, F, precision=0)
            finally:
                rp.reset_shape(0, N, k)
            check(U[k - 1].cpu().numpy(), ref, 1e-12, f"N={N} k={k} kblk={kblk} sym={sym}")


@pytest.mark.parametrize("N,pairs", [(30001, True), (32768, True), (32769, False)])
@pytest.mark.parametrize("prec", [0, 1])
def test_periodic_pairs_of_right_hand_sides_at_their_largest(rp, N, pairs, prec):
    """Two right-hand sides to a pass up to 32768 blobs, with the workspace of
    two and without one, and single passes beyond or with the workspace of one;
    the same sums, to the last bit in FP32C.  Beyond, the memory that the call
    takes is that of one."""
    import ctypes
    rng = np.random.default_rng(N)
    cell = (300.0, 310.0)
    pos = _t(np.column_stack([rng.uniform(0, cell[0], N), rng.uniform(0, cell[1], N), rng.uniform(0.4, 30.0, N)]))
    F = _t(rng.standard_normal((2, N, 3)))
    torch.cuda.reset_peak_memory_stats()
    held = torch.cuda.memory_allocated()

    def passes(fn):
        rp.profile_enable(True)
        rp.profile_read(reset=True)
        try:
            U = fn()
            return U, rp.profile_read(reset=True)[1]
        finally:
            rp.profile_enable(False)

    def raw(ws):
        U = torch.empty_like(F)
        rp._check(rp.lib().rpy_wall_matvec_periodic(
            pos.data_ptr(), F.data_ptr(), U.data_ptr(), N, 2, 1.0, 1.0, *cell, prec,
            ws.data_ptr() if ws is not None else None, ctypes.c_size_t(ws.numel() if ws is not None else 0),
            rp._stream(pos.device)), "periodic")
        return U
    got, n = passes(lambda: rp.matvec_periodic(pos, F, cell, precision=prec))
    assert n == (1 if pairs else 2)
    one = rp.workspace_bytes(rp.OP_MATVEC, N, 1, precision=prec)
    if not pairs:
        assert torch.cuda.max_memory_allocated() - held < 1.2 * one + (64 << 20)
    own, n = passes(lambda: raw(None))
    assert n == (1 if pairs else 2) and torch.equal(own, got)
    single, n = passes(lambda: raw(torch.empty(one, dtype=torch.uint8, device="cuda")))
    assert n == 2
    if prec == 1:
        assert torch.equal(single, got)
    else:
        check(single.cpu().numpy(), got.cpu().numpy(), 1e-13, f"N={N} single passes")


@pytest.mark.parametrize("N,groups_of_128", [(3583, False), (3584, True), (3968, True), (3969, False), (4096, False),
                                             (4480, False), (4481, True), (32768, True), (32769, False)])
def test_sizes_of_the_groups_of_128(rp, orc, N, groups_of_128):
    """FP64, one right-hand side: where both symmetric shapes are the kernel over
    groups of 128, their sums are the same to the bit."""
    pos, f = 0.9 * _mixed(N, N), np.random.default_rng(N).standard_normal((N, 3))
    U = [rp.matvec(_t(pos), _t(f), 0.9, 1.3, precision=0)]
    for sym in (1, 2):
        rp.set_shape(0, N, 1, tpl=1, tile=256, kblk=1, sym=sym, ipw=1)
        try:
            U.append(rp.matvec(_t(pos), _t(f), 0.9, 1.3, precision=0))
        finally:
            rp.reset_shape(0, N, 1)
    assert torch.equal(U[1], U[2]) == (groups_of_128 or N > 32768)
    rows = np.r_[0:8, N - 8:N]
    ref = orc.matvec(pos, f, 0.9, 1.3, rows=rows)
    for u in U:
        check(u.cpu().numpy()[rows], ref, TOL[0], f"N={N}")


def test_fp32c_calls_whose_target_partials_bound_the_kernel(rp, orc):
    """FP32C products above 605000 blobs and VJPs above 349000 run on the
    symmetric kernel with several items to a workgroup only; the workspace of the
    query holds that (it did not, and the calls were refused)."""
    N = 610000
    rng = np.random.default_rng(N)
    pos = np.column_stack([rng.uniform(0, 2000, N), rng.uniform(0, 2000, N), rng.uniform(0.4, 6.0, N)])
    f, g = rng.standard_normal((2, N, 3))
    rows = np.r_[0:4, N - 4:N]
    U = rp.matvec_multi(_t(pos), _t(f[None]), precision=1)[0]
    check(U.cpu().numpy()[rows], orc.matvec(pos, f, rows=rows), TOL[1], f"product N={N}")
    N = 352000
    gp, gf = rp.matvec_vjp(_t(pos[:N]), _t(f[:N]), _t(g[:N]), precision=1)
    rows = np.r_[0:4, N - 4:N]
    gp_ref, gf_ref = orc.vjp(pos[:N], f[:N], g[:N], rows=rows)
    check(gp.cpu().numpy()[rows], gp_ref, TOL[1], f"vjp N={N} grad_pos")
    check(gf.cpu().numpy()[rows], gf_ref, TOL[1], f"vjp N={N} grad_f")
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N,k", [(1, 2), (64, 3), (65, 4), (129, 7), (575, 5), (1025, 2), (1025, 8)])
@pytest.mark.parametrize("prec", [0, 1])
def test_plain_chunk_epilogue(rp, orc, N, k, prec):
    """The plain kernel at the sizes of the chunk epilogue's edges: one chunk,
    fewer than its shares, several rounds, a last wave of one blob."""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + 1).standard_normal((k, N, 3))
    rp.set_shape(prec, N, k, tpl=1, tile=64, kblk=2 if k == 2 else 4 if k <= 4 else 8, sym=0)
    try:
        U = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=prec).cpu().numpy()
    finally:
        rp.reset_shape(prec, N, k)
    for j in range(k):
        check(U[j], orc.matvec(pos, F[j], 0.9, 1.3), TOL[prec], f"plain N={N} k={k} rhs {j} prec={prec}")
