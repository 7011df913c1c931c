"""Mappings of the fused solve read back, set again, stored and given up.

A mapping that the library reports can be set, on the same handle or another,
and gives the same bits; the library's own choice can be restored after any
ssp_set_mapping; 512 threads are for FP64 storage alone.
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


def batch():
    """Longest horizons that make the FP64 default 512 (nx 14, 26, 48), 256 (nx 36) and 128 threads (nx 6)."""
    rng = np.random.default_rng(3)
    return inputs.pack([inputs.draw_problem(rng, n, x, x // 2)
                        for n, x in ((60, 14), (33, 14), (40, 26), (9, 26), (12, 48), (1, 36), (15, 6), (7, 6))])


def solved(db):
    db.solve(1e-9)
    r = db.results()
    assert (r["status"] == 0).all() and db.solver.solve_kernel()[0] == 2
    return r


def test_reported_mapping_can_be_set():
    from paper_2309_06427_amd import solver
    b = batch()
    with solver.DeviceBatch(b) as db:
        db.build("sym", "fp64")
        own = [m[:3] for m in db.solver.mapping()]
        assert {m[0]: m[1] for m in own} == {14: 512, 26: 512, 48: 512, 36: 256, 6: 128}
        ref = solved(db)
        for m in own:
            db.solver.set_group_mapping(*m)
        assert [m[:3] for m in db.solver.mapping()] == own
        assert np.array_equal(solved(db)["lam"], ref["lam"])
    with solver.DeviceBatch(b) as db:  # on a handle whose mapping is another
        db.solver.set_mapping(256, 0, 2)
        db.build("sym", "fp64")
        for m in own:
            db.solver.set_group_mapping(*m)
        assert np.array_equal(solved(db)["lam"], ref["lam"])


def test_own_mapping_comes_back():
    from paper_2309_06427_amd import solver
    with solver.DeviceBatch(batch()) as db:
        db.build("sym", "fp64")
        own, ref = db.solver.mapping(), solved(db)
        for t, l in ((128, 0), (256, 60000)):
            db.solver.set_mapping(t, l, 2)
            assert {m[1] for m in db.solver.mapping()} == {t}
            db.solver.set_mapping(0, 0, 2)
            assert db.solver.mapping() == own
            assert np.array_equal(solved(db)["lam"], ref["lam"])
        with pytest.raises(RuntimeError):
            db.solver.set_mapping(0, 60000, 2)
        with pytest.raises(RuntimeError):
            db.solver.set_mapping(96, 0, 2)
        db.solver.set_mapping(512, 0, 0)  # for the whole handle: the explicit kernel
        db.build("sym", "fp64")
        db.solve(1e-9)
        assert db.solver.solve_kernel()[0] == 1


def test_512_threads_are_for_fp64_storage():
    from paper_2309_06427_amd import solver
    rng = np.random.default_rng(4)
    b = inputs.pack([inputs.draw_problem(rng, n, 20, 10) for n in (30, 44)])  # nx 20: the fused solve under FP32 too
    with solver.DeviceBatch(b) as db:
        db.build("sym", "fp64")
        (nx, t, lds, _), = db.solver.mapping()
        assert t == 512
        db.solver.set_group_mapping(nx, t, lds)
        db.build("sym", "fp32_refine64")
        assert db.solver.mapping()[0][1] == 128
        db.solve(1e-6)
        assert db.solver.solve_kernel()[0] == 2 and (db.results()["status"] == 0).all()
        with pytest.raises(RuntimeError):
            db.solver.set_group_mapping(nx, 512, lds)
        db.build("sym", "fp64")
        assert db.solver.mapping()[0][:3] == (nx, t, lds)


def test_tuned_mapping_is_stored_and_found(tmp_path):
    """The tuner's choice, 512 threads among its candidates, comes back from the file as it was."""
    from paper_2309_06427_amd import solver
    path, b = str(tmp_path / "tune.json"), batch()
    with solver.DeviceBatch(b) as db:
        db.build("sym", "fp64")
        tuned = [m[:3] for m in db.autotune(1e-9, cache=path)]
        ref = db.results()
    assert 512 in {m[1] for m in tuned}
    with solver.DeviceBatch(b) as db:
        db.build("sym", "fp64")
        again = db.autotune(1e-9, cache=path)
        assert [m[:3] for m in again] == tuned and all(m[3] == 0.0 for m in again)  # not timed again
        assert np.array_equal(db.results()["lam"], ref["lam"])
