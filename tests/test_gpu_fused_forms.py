"""The two forms of the fused solve's small workgroups (loads in parts or at once) at the horizon between them.

A group whose problems have at most three steps runs one form, a longer one the
other.  The same problems are solved alone and beside one problem of a knot
more than three steps hold; both runs meet the tolerance of 1e-10, so they agree
to the condition number (below 1e3) times twice that, 2e-7.  Under FP64 they do
the same sums in the same order: iterations equal, lambda to 1e-9.
"""
import numpy as np
import pytest

from paper_2309_06427_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,pc", [("fp64", "sym"), ("fp64", "bj"), ("fp32_refine64", "sym"), ("fp32_refine64", "jacobi")])
@pytest.mark.parametrize("threads", [128, 256])
@pytest.mark.parametrize("nx", [6, 14, 26, 36])
def test_both_forms_agree(nx, threads, precision, pc):
    from paper_2309_06427_amd import _lib, solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L, fp32 = _lib.load(), precision != "fp64"
    lds = L._ZN3ssp8pcg2_ldsEibi(nx, fp32, threads)
    if lds == 0:
        pytest.skip("the mapping holds no knot of this state size")
    c = L._ZN3ssp14pcg2_steps_forEibii(nx, fp32, threads, lds)
    rng = np.random.default_rng(nx + threads)
    ns = sorted({1, 2, c - 1, c, c + 1, 2 * c, 3 * c - 1, 3 * c} - {0})
    probs = [inputs.draw_problem(rng, n, nx, nx // 2) for n in ns]
    out = []
    for more in ([], [inputs.draw_problem(rng, 3 * c + 1, nx, nx // 2)]):
        with solver.DeviceBatch(inputs.pack(probs + more)) as db:
            db.solver.set_mapping(threads, 0, 2)
            db.build(pc, precision)
            db.solve(1e-10)
            out.append(db.results())
            assert db.solver.solve_kernel()[0] == 2 and db.solver.mapping()[0][1] == threads
    a, b = out
    assert (a["status"] == 0).all() and (b["status"] == 0).all()
    n = a["lam"].shape[0]
    bound = 1e-9 if precision == "fp64" else 2e-7
    assert np.linalg.norm(a["lam"] - b["lam"][:n]) <= bound * np.linalg.norm(a["lam"])
    if precision == "fp64":
        assert np.array_equal(a["iters"], b["iters"][:len(ns)])
