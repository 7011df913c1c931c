"""Which problems the scaled solve holds on chip, and the horizons at the ends of that form.

``onchip_problems`` says for a batch's state size how many of its problems (the
shortest ones) the next solve holds on chip, so that the comparisons of the
two forms are known to compare two forms.  A mapping other than the default
one streams everything; both forms return the same bits.
"""
import numpy as np
import pytest

from paper_2309_06427_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def pack(nx, Ns, seed=1):
    rng = np.random.default_rng(seed)
    return inputs.pack([inputs.draw_problem(rng, int(n), nx, nx // 2) for n in Ns])


def streaming(db):
    db.solver.set_scaled_mapping(256, db.solver.scaled_mapping()[1] + 16)


def both(b, pc="sym"):
    """(results, on-chip problems per state size) of the default form and of the streaming one."""
    from paper_2309_06427_amd import solver
    out = []
    for forced in (False, True):
        with solver.DeviceBatch(b) as db:
            db.build(pc, "fp32_refine64")
            if forced:
                streaming(db)
            n = {int(x): db.solver.onchip_problems(int(x)) for x in np.unique(b.nx)}
            db.solve(1e-6)
            out.append((db.results(), n))
    return out


def assert_same(a, c):
    for k in ("iters", "outer", "status", "relres", "lam"):
        assert np.array_equal(a[k], c[k], equal_nan=True), k


# the longest horizon that fits and shorter ones; nx 6 also where p, s and x leave the LDS (from 1065 knots on)
ENDS = {6: (2128, 2127, 1070, 1064, 300), 14: (768, 767, 500), 26: (360, 359, 200)}


@pytest.mark.parametrize("pc", ["sym", "bj", "poly3"])
@pytest.mark.parametrize("nx", sorted(ENDS))
def test_horizons_at_the_ends(nx, pc):
    (a, on), (c, off) = both(pack(nx, ENDS[nx]), pc)
    assert on == {nx: len(ENDS[nx])} and off == {nx: 0}
    assert ((a["status"] & ~16) == 0).all()
    assert_same(a, c)


@pytest.mark.parametrize("nx", sorted(ENDS))
def test_few_problems_stream_beside_one_that_is_too_long(nx):
    (a, on), (c, _) = both(pack(nx, (ENDS[nx][0] + 1,) + ENDS[nx]))
    assert on == {nx: 0}
    assert_same(a, c)


def test_what_else_streams():
    from paper_2309_06427_amd import solver
    b = inputs.pack([inputs.draw_problem(np.random.default_rng(2), n, x, x // 2) for n, x in ((60, 6), (50, 26), (40, 36))])
    with solver.DeviceBatch(b) as db:
        with pytest.raises(RuntimeError):
            db.solver.onchip_problems(6)  # before a build
        db.build("sym", "fp32_refine64")
        chip = lambda: [db.solver.onchip_problems(x) for x in (6, 26, 36)]
        assert chip() == [1, 1, 0]
        with pytest.raises(RuntimeError):
            db.solver.onchip_problems(14)
        db.solver.set_reduction_fp64(True)
        assert chip() == [0, 0, 0]
        db.solver.set_reduction_fp64(False)
        streaming(db)
        assert chip() == [0, 0, 0]
        db.solver.set_scaled_mapping(0, 0)
        assert chip() == [1, 1, 0]
        db.build("jacobi", "fp32_refine64")  # the fused solve
        assert chip() == [0, 0, 0]
        db.build("sym", "fp64")
        assert chip() == [0, 0, 0]


def test_many_problems_of_state_size_6_stream():
    rng = np.random.default_rng(9)
    ns = rng.integers(1, 20, size=700)
    (a, on), _ = both(pack(6, ns))
    assert on == {6: 0}
    assert (a["status"] == 0).all()


@pytest.mark.parametrize("pc", ["bj", "add", "sym", "poly2", "poly3"])
@pytest.mark.parametrize("nx", sorted(ENDS))
def test_the_edge_batches_are_on_chip(nx, pc):
    """The horizons of test_gpu_chip_solve that fit, known to run on chip in one arm and to stream in the other."""
    from .test_gpu_chip_solve import EDGES
    ns = [n for n in EDGES[nx] if n <= ENDS[nx][0]]
    (a, on), (c, off) = both(pack(nx, ns, 100 + nx), pc)
    assert on == {nx: len(ns)} and off == {nx: 0}
    assert_same(a, c)


@pytest.mark.parametrize("nx", [14, 26])
def test_many_short_problems_stream(nx):
    """The same problems few on chip and many streaming: the same bits."""
    ns = np.random.default_rng(nx).integers(1, 9, size=1200)
    (a, on), _ = both(pack(nx, ns))
    (few, fon), (fs, _) = both(pack(nx, ns[:100]))
    assert on == {nx: 0} and fon == {nx: 100}
    assert_same(few, fs)
    n = few["lam"].shape[0]
    assert np.array_equal(a["lam"][:n], few["lam"]) and np.array_equal(a["iters"][:100], few["iters"])
