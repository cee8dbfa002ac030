"""The kernels of the products and derivatives at the sizes where their
splits, tiles and remainders change, against the FP64 oracle.  Bars: those of
the two precisions (FP64 1e-12, FP32C 1e-5, relative L2 and largest entry)."""
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


@pytest.mark.parametrize("N,k", [(1, 2), (64, 3), (65, 4), (129, 7), (575, 5), (1025, 2)])
@pytest.mark.parametrize("prec", [0, 1])
def test_chunk_epilogue(rp, orc, N, k, prec):
    """One chunk, fewer chunks than the epilogue's shares, and several rounds
    of them; a last wave of one blob."""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + 1).standard_normal((k, N, 3))
    U = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=prec).cpu().numpy()
    for j in range(k):
        check(U[j], orc.matvec(pos, F[j], 0.9, 1.3), TOL[prec], f"multi N={N} k={k} rhs {j} prec={prec}")


@pytest.mark.parametrize("N", [1, 2, 64, 65, 300, 511, 512, 513, 1500, 1985, 4033, 5000, 33000])
@pytest.mark.parametrize("prec", [0, 1])
def test_vjp_splits(rp, orc, N, prec):
    """FP64 passes split 16, 8 and 4 ways and not at all, records formed by the
    pair kernel and packed before it, groups of 64 and of 256, odd and even
    numbers of groups, a last wave of one blob."""
    pos = 0.9 * _mixed(N, N)
    f, g = np.random.default_rng(N + 1).standard_normal((2, N, 3))
    gp, gf = rp.matvec_vjp(_t(pos), _t(f), _t(g), 0.9, 1.3, precision=prec)
    rows = None if N < 4000 else np.r_[0:8, N - 8:N]
    gp_ref, gf_ref = orc.vjp(pos, f, g, 0.9, 1.3, rows=rows)
    at = slice(None) if rows is None else rows
    check(gp.cpu().numpy()[at], gp_ref, TOL[prec], f"vjp N={N} prec={prec} grad_pos")
    check(gf.cpu().numpy()[at], gf_ref, TOL[prec], f"vjp N={N} prec={prec} grad_f")


@pytest.mark.parametrize("N", [1, 2, 255, 256, 257, 513, 1281, 2047])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 9])
def test_one_launch_products(rp, orc, N, k):
    """FP64 products in one launch: a workgroup with one target of its two,
    fewer sources than threads, every block width and its remainder, two
    blocks.  (Above 1280 and 1536 blobs the wider ones take other kernels.)"""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + k).standard_normal((k, N, 3))
    U = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=0).cpu().numpy()
    for j in {0, k // 2, k - 1}:
        check(U[j], orc.matvec(pos, F[j], 0.9, 1.3), TOL[0], f"one launch N={N} k={k} rhs {j}")


@pytest.mark.parametrize("N,k,ipw", [(N, k, ipw) for N in (1, 64, 65, 128, 129, 257, 1500, 2049, 2305)
                                     for k, ipw in ((2, 1), (3, 4), (4, 2))]
                         + [(3584, 1, 1), (3649, 1, 3), (3713, 1, 2), (5000, 1, 1)])
def test_two_targets_per_lane(rp, orc, N, k, ipw):
    """The FP64 symmetric kernel over groups of 128: one group (diagonal items
    alone), half-filled and nearly empty last groups, odd and even numbers of
    groups, passes split 4 and 2 ways and not at all, chunks of several items
    and a last chunk of fewer."""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + k).standard_normal((k, N, 3))
    rp.set_shape(0, N, k, kblk=1 if k == 1 else 2 if k == 2 else 4, sym=1, ipw=ipw)
    try:
        U = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=0)
        again = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=0)
    finally:
        rp.reset_shape(0, N, k)
    assert torch.equal(U, again)
    for j in range(k):
        check(U[j].cpu().numpy(), orc.matvec(pos, F[j], 0.9, 1.3), TOL[0], f"two targets N={N} k={k} rhs {j}")


def test_repeated_solves_are_bitwise_equal(rp):
    """Roots and rigid solves repeat bit for bit when calls of different sizes
    alternate: no coefficient that the host reads may be one that an earlier
    call left in its pinned memory."""
    from paper_1709_02410_amd import workloads as wl
    cfg, runs = wl.config1(seed=0), []
    for bodies in (40, 60):
        offs = cfg.body_offsets[:bodies + 1]
        pos = cfg.pos[:offs[-1]]
        runs.append((_t(pos), _t(pos[offs[:-1]]), offs, _t(wl.gaussian(pos.shape, bodies))))
    first = [None, None]
    for _ in range(100):
        for i, (pos, q, offs, w) in enumerate(runs):
            root, it, _, _ = rp.lanczos_sqrt(pos, w, body_offsets=offs, tol=1e-9)
            _, U, its, _, _ = rp.rigid_solve(pos, q, offs, w, None, tol=1e-9)
            first[i] = first[i] or (root, U, it, its)
            assert (it, its) == first[i][2:]
            assert torch.equal(root, first[i][0]) and torch.equal(U, first[i][1])


@pytest.mark.parametrize("blobs,bodies", [(4, 300), (8, 30), (12, 12), (15, 9), (16, 9), (21, 9), (25, 6), (42, 5)])
def test_krylov_vector_kernels(rp, orc, blobs, bodies):
    """More than 256 groups of partials; 12 to 126 entries to a body (four, two
    and one thread per entry, every size of the factor kernels); 90 to 200 basis vectors, in
    registers (16 and 32 to a thread) and read again.  Bars: the tolerance
    1e-12 times the root of the condition number (1e3), and times it (1e5)."""
    from parity_util import krylov_path
    from paper_1709_02410_amd import workloads as wl
    N = blobs * bodies
    side = (2.8 * N) ** (1 / 3)  # overlapping blobs, so that many steps are needed
    pos = np.random.default_rng(blobs).uniform(0, side, (N, 3)) + [0, 0, 0.6]
    offs = np.arange(0, N + 1, blobs)
    W, q = wl.gaussian(pos.shape, blobs), pos[offs[:-1]]
    with krylov_path(rp, N, True):
        root, it, _, ok = rp.lanczos_sqrt(_t(pos), _t(W), body_offsets=offs, tol=1e-12, max_iter=250)
        _, U, its, _, ok2 = rp.rigid_solve(_t(pos), _t(q), offs, _t(W), None, tol=1e-12, max_iter=250)
    assert ok and ok2 and it > 80 and its > 80
    check(root.cpu().numpy(), orc.dense_sqrt(pos, W, offs), 1e-9, f"root {blobs}x{bodies}")
    check(U.cpu().numpy(), orc.rigid_solve(pos, q, offs, W, None)[1], 1e-7, f"U {blobs}x{bodies}")


@pytest.mark.parametrize("N,prec", [(5100, 1), (5160, 1), (10245, 0)])
def test_presummed_krylov_steps(rp, N, prec):
    """Fused steps below and above the number of groups from which the
    product's partials are summed first, against the steps on plain products
    (pair terms in FP32: 1e-5; FP64: 1e-11, a few steps of 1e-12 each)."""
    rng = np.random.default_rng(N)
    side = int(np.ceil((N / 5) ** 0.5))
    b = np.arange(N // 5)
    at = np.stack([4.5 * (b % side), 4.5 * (b // side), np.full(b.size, 1.4)], -1)
    arm = np.array([[0, 0, 0], [1.9, 0, 0], [0, 1.9, 0], [0, 0, 1.9], [1.9, 1.9, 0]])
    pos = (at[:, None] + arm + 0.05 * rng.standard_normal((b.size, 5, 3))).reshape(-1, 3)
    offs, W, q = np.arange(0, N + 1, 5), rng.standard_normal((N, 3)), pos[::5]

    def run():
        root = rp.lanczos_sqrt(_t(pos), _t(W), body_offsets=offs, tol=1e-30, max_iter=4, precision=prec)[0]
        U = rp.rigid_solve(_t(pos), _t(q), offs, _t(W), None, tol=1e-30, max_iter=4, precision=prec)[1]
        return root.cpu().numpy(), U.cpu().numpy()
    got = run()
    rp.set_shape(prec, N, 1, tpl=1, tile=256, kblk=1, sym=0)
    try:
        ref = run()
    finally:
        rp.reset_shape(prec, N, 1)
    for g, r, what in zip(got, ref, ("root", "U")):
        check(g, r, 1e-11 if prec == 0 else 1e-5, f"{what} N={N} prec={prec}")


@pytest.mark.parametrize("N", [300, 16100, 16400, 16900, 20000])
@pytest.mark.parametrize("prec", [0, 1])
def test_tail_chunks(rp, N, prec):
    """Groups of 256: rows of tail chunks alone (up to 63 groups), and of main
    chunks with remainders and a tail, for odd and even numbers of groups; one
    item to a chunk gives the same sums up to the order of FP64 additions."""
    pos = 0.9 * _mixed(N, N)
    f, g = np.random.default_rng(N + 1).standard_normal((2, N, 3))
    runs = []
    for ipw in (1, 2, 3, 6):
        rp.set_shape(prec, N, 1, tpl=1, tile=256, kblk=1, sym=1, ipw=ipw)
        u = rp.matvec(_t(pos), _t(f), 0.9, 1.3, precision=prec)
        runs.append([x.cpu().numpy() for x in (u, *rp.matvec_vjp(_t(pos), _t(f), _t(g), 0.9, 1.3, precision=prec))])
    rp.reset_shape(prec, N, 1)
    for ipw, r in zip((2, 3, 6), runs[1:]):
        for x, ref, what in zip(r, runs[0], ("u", "grad_pos", "grad_f")):
            check(x, ref, 1e-12, f"{what} N={N} prec={prec} ipw={ipw}")


@pytest.mark.parametrize("N", [1, 3, 127, 129, 300, 1000, 1300])
@pytest.mark.parametrize("prec,k", [(1, 1), (1, 3), (1, 8), (1, 13), (0, 12)])
def test_small_plain_products(rp, orc, N, prec, k):
    """Plain and matrix-core kernels of small problems: odd numbers of sources
    (two are taken at a time), chunks shared out at tiles with remainders, and
    shares without sources."""
    pos = 0.9 * _mixed(N, N)
    F = np.random.default_rng(N + k).standard_normal((k, N, 3))
    rp.set_shape(prec, N, k, tpl=1, tile=64, kblk={1: 1, 3: 4, 8: 8}.get(k, 16), sym=0, mat=1 if k >= 8 else 0)
    try:
        U = rp.matvec_multi(_t(pos), _t(F), 0.9, 1.3, precision=prec).cpu().numpy()
    finally:
        rp.reset_shape(prec, N, k)
    for j in {0, k // 2, k - 1}:
        check(U[j], orc.matvec(pos, F[j], 0.9, 1.3), TOL[prec], f"plain N={N} k={k} rhs {j} prec={prec}")


@pytest.mark.parametrize("blobs,bodies", [(3, 1), (4, 1), (5, 12), (7, 9), (15, 34)])
def test_small_krylov_steps(rp, orc, blobs, bodies):
    """Fused FP64 steps of problems below 512 blobs (default shape), down to
    one body in one group.  Bars: as for the vector kernels."""
    from paper_1709_02410_amd import workloads as wl
    N = blobs * bodies
    side = (2.8 * N) ** (1 / 3)
    pos = np.random.default_rng(N).uniform(0, side, (N, 3)) + [0, 0, 0.6]
    offs = np.arange(0, N + 1, blobs)
    W, q = wl.gaussian(pos.shape, blobs), pos[offs[:-1]]
    root, _, _, ok = rp.lanczos_sqrt(_t(pos), _t(W), body_offsets=offs, tol=1e-12, max_iter=250)
    free, _, _, ok1 = rp.lanczos_sqrt(_t(pos), _t(W), tol=1e-12, max_iter=250)
    _, U, _, _, ok2 = rp.rigid_solve(_t(pos), _t(q), offs, _t(W), None, tol=1e-12, max_iter=250)
    assert ok and ok1 and ok2
    check(root.cpu().numpy(), orc.dense_sqrt(pos, W, offs), 1e-9, f"root {blobs}x{bodies}")
    check(free.cpu().numpy(), orc.dense_sqrt(pos, W, None), 1e-9, f"root without bodies N={N}")
    check(U.cpu().numpy(), orc.rigid_solve(pos, q, offs, W, None)[1], 1e-7, f"U {blobs}x{bodies}")


@pytest.mark.parametrize("sizes", [(1,), (3, 700), (513, 64, 1, 2000, 129), (1500, 1400)])
@pytest.mark.parametrize("prec,k", [(1, 1), (1, 3), (1, 16), (0, 1), (0, 8), (0, 16)])
def test_batched_parts(rp, orc, sizes, prec, k):
    """Batched systems whose sources are split into parts: more parts than a
    small system has tiles, a last tile of one blob, one part (one blob)."""
    offs = np.r_[0, np.cumsum(sizes)]
    pos = np.concatenate([0.9 * _mixed(n, n) for n in sizes])
    F = np.random.default_rng(k).standard_normal((k, offs[-1], 3))
    U = rp.matvec_batched(_t(pos), offs, _t(F), 0.9, 1.3, precision=prec)
    assert torch.equal(U, rp.matvec_batched(_t(pos), offs, _t(F), 0.9, 1.3, precision=prec))
    for a, b in zip(offs, offs[1:]):
        for j in {0, k - 1}:
            check(U[j, a:b].cpu().numpy(), orc.matvec(pos[a:b], F[j, a:b], 0.9, 1.3), TOL[prec],
                  f"system {b - a} of {sizes} k={k} rhs {j} prec={prec}")


@pytest.mark.parametrize("N", [1, 64, 130, 700, 2000])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("cell", [(40.0, 37.0), (4.2, 4.3)])
def test_periodic_pairs_of_right_hand_sides(rp, orc, N, prec, cell):
    """Two right-hand sides to a pass (and the odd one alone), in wide cells and
    in one below 4.5 a: the sums of single products, FP32C to the last bit,
    FP64 up to the order of additions."""
    rng = np.random.default_rng(N)
    pos = np.column_stack([rng.uniform(0, cell[0], N), rng.uniform(0, cell[1], N), rng.uniform(0.4, 30.0, N)])
    F = rng.standard_normal((3, N, 3))
    U = rp.matvec_periodic(_t(pos), _t(F), cell, 1.0, 1.3, precision=prec).cpu().numpy()
    for j in range(3):
        one = rp.matvec_periodic(_t(pos), _t(F[j:j + 1]), cell, 1.0, 1.3, precision=prec).cpu().numpy()[0]
        if prec == 1:
            assert np.array_equal(U[j], one)
        else:
            check(U[j], one, 1e-13, f"periodic N={N} rhs {j}")


@pytest.mark.parametrize("N", [8128, 8129, 8192, 8193])
def test_periodic_fp32c_records(rp, N):
    """Both sides of the line between FP32C records formed in the kernel (127
    groups of 64) and packed ones (128 and more), full and ragged last groups,
    one and two right-hand sides: the FP32C products over groups of 256.  (FP64
    is no reference at this size: some pairs are half a cell apart up to FP32
    rounding, and precisions may differ in the images that they take.)"""
    rng = np.random.default_rng(N)
    cell = (150.0, 140.0)
    pos = np.column_stack([rng.uniform(-200, 300, N), rng.uniform(-200, 300, N), rng.uniform(0.4, 30.0, N)])
    F = rng.standard_normal((3, N, 3))
    U = rp.matvec_periodic(_t(pos), _t(F), cell, 1.0, 1.3, precision=1).cpu().numpy()
    rp.set_shape(1, N, 1, tpl=1, tile=256, kblk=1, sym=1, ipw=1)
    try:
        for j in range(3):
            ref = rp.matvec(_t(pos), _t(F[j]), 1.0, 1.3, precision=1, box=cell).cpu().numpy()
            check(U[j], ref, TOL[1], f"periodic N={N} rhs {j}")
    finally:
        rp.reset_shape(1, N, 1)
