"""The rules that choose between the forms of a solve, against measured times.

Each row is a batch of one state size that was timed in both forms; the rule,
a host function of the horizons and the CU count, has to take the faster one
wherever they differ by more than a tenth.
"""
import ctypes as C

import numpy as np
import pytest

CUS = 256

# state size, horizons (one, or a range drawn uniformly), problems, on-chip ms, streaming ms
SCALED = [
    (14, 1, 16, 0.0315, 0.0261), (14, 1, 4096, 0.2992, 0.1039), (14, 4, 128, 0.0860, 0.0922), (14, 4, 1024, 0.2672, 0.1673),
    (14, 8, 256, 0.1017, 0.1184), (14, 8, 4096, 1.0735, 0.5364), (14, 16, 256, 0.1038, 0.1278), (14, 16, 300, 0.1710, 0.1380),
    (14, 16, 512, 0.1741, 0.1396), (14, 20, 1024, 0.3397, 0.3653), (14, 20, 4096, 1.2347, 1.0036),
    (14, 64, 4096, 1.7121, 2.2748), (14, 128, 512, 0.3256, 0.7541), (14, 256, 1024, 1.3694, 2.9087),
    (14, 768, 16, 0.9976, 3.7127), (14, (1, 9), 100, 0.0937, 0.1082), (14, (1, 9), 4096, 0.8539, 0.3831),
    (14, (1, 32), 1365, 0.3964, 0.2944), (14, (1, 32), 300, 0.1439, 0.2046), (14, (32, 256), 4096, 2.9338, 4.5994),
    (26, 1, 128, 0.0368, 0.0282), (26, 1, 4096, 0.3699, 0.1301), (26, 2, 512, 0.1231, 0.0828), (26, 4, 16, 0.0849, 0.0995),
    (26, 4, 4096, 1.2211, 0.6476), (26, 8, 256, 0.1247, 0.1608), (26, 8, 512, 0.2248, 0.1860), (26, 8, 4096, 1.4439, 0.8718),
    (26, 16, 512, 0.2483, 0.3407), (26, 24, 4096, 2.1505, 2.4373), (26, 64, 1024, 1.0995, 1.9952),
    (26, 360, 256, 1.9299, 5.5498), (26, (1, 12), 4096, 1.2739, 0.8103), (26, (1, 40), 300, 0.2053, 0.5491),
    (26, (32, 256), 1365, 3.3381, 5.0505),
    (6, 1, 16, 0.0279, 0.0222), (6, 8, 640, 0.1996, 0.0863), (6, 32, 16, 0.0963, 0.0860), (6, 32, 256, 0.1130, 0.1000),
    (6, 64, 256, 0.1288, 0.1594), (6, 64, 512, 0.2355, 0.1727), (6, 128, 256, 0.1769, 0.2715), (6, 128, 512, 0.3212, 0.2860),
    (6, 256, 256, 0.3025, 0.4533), (6, 256, 640, 0.7361, 0.5370), (6, 985, 64, 0.966, 1.343), (6, 985, 512, 2.245, 1.599),
    (6, (1, 40), 256, 0.1165, 0.0975), (6, (1, 64), 640, 0.2510, 0.1621), (6, (32, 256), 512, 0.3639, 0.4569),
    (6, (32, 256), 1365, 0.781, 0.513),
]


def chip_pays(nx, N, too_long=0, cus=CUS):
    from paper_2309_06427_amd import _lib
    f = _lib.load()._ZN3ssp9chip_paysEiPKiiii
    f.restype = C.c_bool
    N = np.ascontiguousarray(np.sort(np.asarray(N, dtype=np.int32))[::-1])
    return f(nx, N.ctypes.data_as(C.c_void_p), len(N), too_long, cus)


def horizons(n, P):
    return np.full(P, n) if np.isscalar(n) else np.random.default_rng(P).integers(n[0], n[1] + 1, size=P)


@pytest.mark.parametrize("nx,n,P,chip,stream", SCALED)
def test_scaled_form_is_the_faster_one(nx, n, P, chip, stream):
    pays = chip_pays(nx, horizons(n, P))
    if chip <= stream / 1.1:
        assert pays
    elif stream <= chip / 1.1:
        assert not pays


def test_scaled_form_with_problems_that_are_too_long():
    """nx 26, the rest on chip after the long ones and all streaming, ms: 256 of 400 knots and 256 of 300 7.72 and 6.23,
    one of 400 and 1000 of 100 7.02 and 5.47, 600 of 400 and 600 of 200 10.16 and 10.43; nx 14, one of 800 and 1000 of
    100 4.07 and 3.81.  All of them too long: streaming."""
    assert not chip_pays(26, [400] * 256 + [300] * 256, 256)
    assert not chip_pays(26, [400] * 16 + [300] * 480, 16)
    assert not chip_pays(26, [400] + [100] * 1000, 1)
    assert not chip_pays(14, [800] + [100] * 1000, 1)
    assert chip_pays(26, [400] * 600 + [200] * 600, 600)
    assert chip_pays(26, [400] + [100] * 12000, 1)
    assert not chip_pays(26, [400] * 16, 16)


def test_scaled_form_of_other_state_sizes_streams():
    assert not any(chip_pays(nx, [50]) for nx in range(1, 65) if nx not in (6, 14, 26))
    assert chip_pays(14, [50], cus=1)


# state size, horizon, problems, ms with 128, 256 and 512 threads
FUSED64 = [
    (4, 1, 16, 0.0199, 0.0210, 0.0238), (4, 16, 512, 0.1359, 0.1455, 0.3248), (4, 128, 16, 0.6151, 0.3814, 0.2542),
    (6, 8, 256, 0.0886, 0.0935, 0.1077), (6, 32, 512, 0.2661, 0.1718, 0.3124), (6, 128, 16, 0.7287, 0.4712, 0.3213),
    (6, 128, 512, 0.8983, 0.5967, 0.6917), (9, 16, 256, 0.3349, 0.1991, 0.2511), (9, 64, 512, 1.2822, 0.6905, 1.0342),
    (12, 2, 512, 0.0934, 0.0970, 0.2147), (12, 16, 16, 0.5064, 0.3577, 0.2531), (12, 16, 512, 0.5907, 0.4177, 0.5223),
    (14, 4, 4096, 0.5220, 0.9069, 1.9643), (14, 8, 512, 0.2639, 0.1709, 0.3335), (14, 16, 4096, 2.3045, 2.2709, 2.7656),
    (14, 128, 16, 2.9646, 1.5888, 0.8137), (14, 64, 512, 1.8698, 1.0765, 0.9837), (20, 2, 4096, 0.5227, 0.7828, 2.4258),
    (20, 4, 256, 0.3080, 0.2183, 0.2662), (20, 32, 1024, 3.7489, 3.7964, 2.7684), (26, 2, 4096, 0.5842, 0.7967, 1.7290),
    (26, 4, 512, 0.4178, 0.2670, 0.3764), (26, 8, 4096, 4.8723, 4.6218, 3.3787), (26, 128, 512, 20.45, 10.87, 5.806),
    (31, 2, 512, 0.2625, 0.2103, 0.4444), (31, 8, 4096, 12.8155, 9.5538, 12.0855), (31, 64, 256, 19.28, 9.881, 3.997),
]


def fp64_threads(nx, N, resident):
    from paper_2309_06427_amd import _lib
    f = _lib.load()._ZN3ssp18fused_fp64_threadsEiPKiiiS1_
    N = np.ascontiguousarray(N, dtype=np.int32)
    return f(nx, N.ctypes.data_as(C.c_void_p), len(N), CUS, (C.c_int32 * 3)(*resident))


@pytest.mark.parametrize("nx,n,P,t128,t256,t512", FUSED64)
def test_fp64_workgroup_is_close_to_the_fastest(nx, n, P, t128, t256, t512):
    """Within a seventh of the fastest workgroup size."""
    N = np.full(P, n, dtype=np.int32)
    ms = {128: t128, 256: t256, 512: t512}
    assert ms[fp64_threads(nx, N, (4, 2, 1) if nx in (6, 14, 26) else (5, 3, 1))] <= min(ms.values()) * 8 / 7


def test_fp64_workgroup_of_sizes_that_few_hold():
    """From state size 45 on only 512 threads hold a knot, from 58 on none does (the explicit kernel's 128)."""
    N = np.full(3, 1, dtype=np.int32)
    got = [fp64_threads(nx, N, (1, 1, 1)) for nx in (44, 45, 57, 58, 64)]
    assert got == [256, 512, 512, 128, 128]
