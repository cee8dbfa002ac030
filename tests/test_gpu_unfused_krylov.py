"""The unfused Lanczos and GMRES drivers in FP64 at small sizes: the cases of the
two solvers' tests under a fixed plain shape.  (Their own fused=False runs take
the built-in shape, whose FP64 steps are fused at every size up to 2048 blobs.)"""
import pytest

import test_gpu_lanczos as lanczos
import test_gpu_rigid as rigid
from paper_1709_02410_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_02410_amd import rpywall
    rpywall.lib()
    return rpywall


@pytest.fixture
def plain(rp):
    """Size classes of 1 to 511 blobs."""
    for c in range(9):
        rp.set_shape(0, 1 << c, 1, tpl=1, tile=256, kblk=1, sym=0)
    yield
    for c in range(9):
        rp.reset_shape(0, 1 << c, 1)


def test_the_fixed_plain_shape_takes_the_other_driver(rp, plain):
    """Same root, other order of the sums."""
    pos, offs = wl.boomerang_suspension(12, 25.0, 1.5, 4.0, seed=3)
    W = lanczos._t(wl.gaussian(pos.shape, 4))
    run = lambda: rp.lanczos_sqrt(lanczos._t(pos), W, body_offsets=offs, tol=1e-10)[0]  # noqa: E731
    unfused = run()
    for c in range(9):
        rp.reset_shape(0, 1 << c, 1)
    fused = run()
    assert not torch.equal(unfused, fused)
    lanczos.check(unfused.cpu().numpy(), fused.cpu().numpy(), 1e-9, "unfused against fused")


@pytest.mark.parametrize("bodies", [True, False])
def test_small_against_dense_root(rp, orc, plain, bodies):
    lanczos.test_small_against_dense_root(rp, orc, bodies, False)


@pytest.mark.parametrize("N,bodies", [(1, False), (2, False), (15, True)])
def test_exhausted_krylov_space(rp, orc, plain, N, bodies):
    lanczos.test_exhausted_krylov_space(rp, orc, N, bodies, False)


@pytest.mark.parametrize("case", [lanczos.test_not_converged_returns_best_iterate, lanczos.test_largest_bodies_42_blobs,
                                  lanczos.test_back_to_back_calls_and_two_streams, rigid.test_iterations_match_oracle_gmres,
                                  rigid.test_single_body_is_solved_by_the_preconditioner,
                                  rigid.test_random_slip_gives_brownian_body_velocities])
def test_against_the_oracle(rp, orc, plain, case):
    case(rp, orc, False)


@pytest.mark.parametrize("case", [lanczos.test_non_spd_block_is_reported, lanczos.test_zero_vector,
                                  rigid.test_zero_rhs_and_not_converged_and_rod])
def test_end_cases(rp, plain, case):
    case(rp, False)


def test_rigid_solve_matches_dense_saddle_point(rp, orc, plain):
    rigid.test_rigid_solve_matches_dense_saddle_point(rp, orc, 0, 1e-11, 1e-8, False)
