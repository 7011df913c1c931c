"""The on-chip form of the scaled solve against the streaming one.

Both run the same float arithmetic term by term and the same sums in the same
order, so every output has the same bits: lambda, iterations, refinement
steps, the reported residual and the statuses.  A mapping other than the
default one (here the default LDS budget plus 16 bytes, which leaves the
streaming solve's steps as they are) selects the streaming form.  The sizes
sit at the edges of the on-chip solve: horizons below, at and above a set of
four knots and of one set per wave, where the sets held in registers end,
where p, s and x leave the LDS (nx 26: 180, nx 14: 384 knots), the longest
horizon that fits (nx 26: 360) and the first that does not.  The oracle
comparisons of the default mapping are those of the other scaled-solve tests.
"""
import numpy as np
import pytest

from paper_2309_06427_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGES = {
    6: (1, 2, 3, 4, 5, 31, 32, 33, 36, 160, 161, 256, 400),
    14: (1, 3, 4, 5, 8, 31, 33, 64, 128, 129, 132, 255, 256, 384, 385),
    26: (1, 2, 4, 5, 7, 31, 32, 33, 35, 36, 37, 64, 96, 144, 180, 181, 233, 256, 360, 361),
}


def both(b, pc, precision="fp32_refine64", tol=1e-6, max_iter=0, warm=False):
    from paper_2309_06427_amd import solver
    out = []
    for streaming in (False, True):
        with solver.DeviceBatch(b) as db:
            db.build(pc, precision)
            lds = db.solver.scaled_mapping()[1]
            if streaming:
                db.solver.set_scaled_mapping(256, lds + 16)
            lam0 = None
            if warm:
                g = torch.Generator(device="cuda").manual_seed(3)
                lam0 = 0.1 * torch.randn(db.lam.shape, generator=g, dtype=torch.float64, device="cuda")
            db.solve(tol, max_iter, lam0=lam0, fallback=warm)
            out.append(db.results())
            assert db.solver.solve_kernel()[0] == 4
    return out


def batch(nx, Ns, seed, qmode="wishart", qcond_max=1e4):
    rng = np.random.default_rng(seed)
    return inputs.pack([inputs.draw_problem(rng, n, nx, nx // 2, qmode, qcond_max) for n in Ns])


def assert_same(out):
    a, c = out
    for k in ("iters", "outer", "status", "relres", "lam"):
        assert np.array_equal(a[k], c[k], equal_nan=True), (k, a[k], c[k])


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("pc", ["bj", "add", "sym", "poly2", "poly3"])
@pytest.mark.parametrize("nx", sorted(EDGES))
def test_same_bits_as_the_streaming_solve(nx, pc):
    out = both(batch(nx, EDGES[nx], 100 + nx), pc)
    assert ((out[0]["status"] & ~16) == 0).all()
    assert_same(out)


@pytest.mark.parametrize("case", ["tight", "fp32", "limit", "warm", "cond", "nonfinite"])
def test_same_bits_on_every_exit(case):
    if case == "cond":  # several refinement steps, block-Jacobi beside the stair
        b = batch(26, (40, 97, 128), 7, "logcond", 1e6)
        for pc in ("sym", "bj"):
            assert_same(both(b, pc))
        return
    b = inputs.batch(18, 8, N_range=(1, 150), nx_choices=(6, 14, 26))
    if case == "nonfinite":
        b.gamma[int(b.off_v[3])] = np.inf
        b.gamma[int(b.off_v[5]):int(b.off_v[6])] = 0.0
    out = both(b, "sym", "fp32" if case == "fp32" else "fp32_refine64", 1e-10 if case == "tight" else 1e-6,
               7 if case == "limit" else 0, case == "warm")
    assert_same(out)
    if case == "nonfinite":
        assert out[0]["status"][3] == 3 and out[0]["iters"][5] == 0


def test_many_small_state_problems_stream():
    """At nx 6 the choice also depends on the number of problems: the same bits on both sides of it."""
    rng = np.random.default_rng(9)
    probs = [inputs.draw_problem(rng, int(n), 6, 3) for n in rng.integers(1, 20, size=700)]
    many, few = inputs.pack(probs), inputs.pack(probs[:40])
    a, c = both(many, "sym")[0], both(few, "sym")[0]
    n = c["lam"].shape[0]
    assert np.array_equal(a["lam"][:n], c["lam"]) and np.array_equal(a["iters"][:40], c["iters"])
