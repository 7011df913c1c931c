"""bench.py counts as held on chip what the library says it holds on chip."""
import os
import sys

import numpy as np

from paper_2309_06427_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Says:
    def __init__(self, **n):
        self.n = n

    def onchip_problems(self, nx):
        return self.n[f"nx{nx}"]


def test_chip_mask_follows_the_library(monkeypatch):
    """The shortest n problems of each state size, later ones first among equals, whatever n the library reports."""
    monkeypatch.syspath_prepend(ROOT)
    import bench
    rng = np.random.default_rng(0)
    b = inputs.pack([inputs.draw_problem(rng, n, x, x // 2) for n, x in ((9, 6), (3, 14), (5, 6), (5, 6), (8, 14), (2, 6))])
    assert bench.chip_mask(b, Says(nx6=0, nx14=0)).tolist() == [False] * 6
    assert bench.chip_mask(b, Says(nx6=2, nx14=1)).tolist() == [False, True, False, True, False, True]
    assert bench.chip_mask(b, Says(nx6=4, nx14=2)).all()
