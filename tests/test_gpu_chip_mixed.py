"""Batches whose state size has problems on chip and problems that are too long for it.

The two forms run side by side on streams of their own.  Their results are
those of the streaming form alone, also from a replayed graph, and a solve of
both takes less than the two parts one after the other: 16 problems of 400
knots (one workgroup each) beside 480 of 300 knots (nx 26) take about as long
as the slower part, against its sum with the other where they run in turn; the
bound of 0.85 of the sum leaves a fifth of the expected gain for noise.
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


def pack(sizes, seed=4):
    rng = np.random.default_rng(seed)
    return inputs.pack([inputs.draw_problem(rng, n, nx, nx // 2) for n, nx in sizes])


MIXES = {"one size": [(400, 26), (361, 26), (360, 26), (30, 26), (5, 26)] + [(20, 26)] * 3,
         "three sizes": [(380, 26), (100, 26), (800, 14), (768, 14), (50, 14), (2200, 6), (900, 6), (40, 6), (30, 36)]}


@pytest.mark.parametrize("mix", sorted(MIXES))
def test_results_are_those_of_the_streaming_form(mix):
    from paper_2309_06427_amd import solver
    b = pack(MIXES[mix])
    out = []
    for forced in (False, True):
        with solver.DeviceBatch(b) as db:
            db.build("sym", "fp32_refine64")
            if forced:
                db.solver.set_scaled_mapping(256, db.solver.scaled_mapping()[1] + 16)
            else:
                assert 0 < db.solver.onchip_problems(26) < int((b.nx == 26).sum())
            db.solve(1e-6)
            out.append(db.results())
            if not forced:  # the same solve from a graph, replayed with other work between the replays
                g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
                torch.cuda.synchronize()
                with torch.cuda.graph(g, stream=s):
                    db.solve(1e-6)
                for k in range(3):
                    db.lam.fill_(float(k))
                    db.iters.zero_()
                    g.replay()
                    r = db.results()
                    assert np.array_equal(r["lam"], out[0]["lam"]) and np.array_equal(r["iters"], out[0]["iters"]), k
    assert (out[0]["status"] == 0).all()
    for k in ("iters", "outer", "status", "relres", "lam"):
        assert np.array_equal(out[0][k], out[1][k]), k


def test_long_and_short_problems_overlap():
    from paper_2309_06427_amd import solver
    long_, short = pack([(400, 26)] * 2), pack([(300, 26)] * 5)

    def ms(b, idx):
        with solver.DeviceBatch(b.subset(idx)) as db:
            db.build("sym", "fp32_refine64")
            t = []
            for _ in range(6):
                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                e[0].record()
                db.solve(1e-6)
                e[1].record()
                torch.cuda.synchronize()
                t.append(e[0].elapsed_time(e[1]))
            return float(np.median(t[1:]))

    both = pack([(400, 26)] * 2 + [(300, 26)] * 5)
    a = ms(long_, [0, 1] * 8)
    c = ms(short, [k % 5 for k in range(480)])
    t = ms(both, [0, 1] * 8 + [2 + k % 5 for k in range(480)])
    print(f"16 of 400 knots {a:.3f} ms, 480 of 300 {c:.3f} ms, together {t:.3f} ms")
    assert t < 0.85 * (a + c), (a, c, t)
