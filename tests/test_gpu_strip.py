"""Launches of K steps with the intermediate states in registers, the default of
D1Q3 rows and D2Q9 domains: strips, and blocks for small D2Q9 domains.  Every run is bitwise the one-step-per-launch run (time_block = 1): the
same per-node code, and float storage rounds after every step in both."""
import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu


def _lbm():
    from paper_2303_08163_amd import lbm
    return lbm


def _compare(shape, dtype, corr, eq, chunks, seed, umax=0.1):
    lbm = _lbm()
    rho0, u0 = workloads.random_field(shape, seed=seed, umax=umax)
    kw = dict(dtype=dtype, bulk_correction=corr, equilibrium=eq)
    with lbm.Domain(rho0, u0, 0.55, **kw) as a, \
            lbm.Domain(rho0, u0, 0.55, tuning=lbm.make_tuning(time_block=1), **kw) as b:
        for n in chunks:
            a.step(n)
            b.step(n)
            ra, ua, da = a.moments()
            rb, ub, db = b.moments()
            assert da["steps"] == db["steps"]
            assert np.array_equal(ra, rb) and np.array_equal(ua, ub), (shape, n)
        assert np.array_equal(a.populations(), b.populations()), shape


D2_CASES = [  # (ny, nx), dtype, correction, equilibrium, step chunks
    ((2500, 512), "fp32_dev", False, "entropic", (4, 5, 6, 7, 100)),
    ((2500, 512), "fp64", True, "entropic", (6, 7, 8, 9, 10, 11, 100)),
    # widths one off a multiple of the own columns (58 and 54), odd heights
    ((3001, 349), "fp32_dev", True, "entropic", (4, 67)),
    ((1801, 1081), "fp64", False, "entropic", (6, 71)),
    ((1703, 1079), "fp64", True, "product", (12, 4)),
    ((2011, 971), "fp64", False, "poly2", (13,)),
    ((1201, 1045), "fp32_dev", False, "poly2", (9,)),
    ((1999, 811), "fp32_dev", True, "product", (8,)),
    # the narrowest rows, and fewer rows than a sweep's halo (wrapped several times)
    ((30049, 64), "fp32_dev", False, "entropic", (12, 3)),
    ((30017, 65), "fp64", False, "entropic", (14,)),
    ((1, 1048576), "fp64", True, "entropic", (14, 3)),
    ((2, 655361), "fp32_dev", True, "entropic", (8, 5)),
    ((5, 300001), "fp64", False, "entropic", (18,)),
    # non-temporal stores (the two buffers exceed the last-level cache)
    ((2050, 2049), "fp32_dev", False, "entropic", (10,)),
    ((1500, 1501), "fp64", True, "entropic", (12,)),
]


@pytest.mark.parametrize("case", range(len(D2_CASES)))
def test_d2q9_strips_equal_one_step_bitwise(case):
    shape, dtype, corr, eq, chunks = D2_CASES[case]
    _compare(shape, dtype, corr, eq, chunks, seed=300 + case)


BLOCK_CASES = [  # (ny, nx), dtype, correction, equilibrium, step chunks
    ((64, 64), "fp64", False, "entropic", (1, 2, 3, 4, 5, 100)),
    ((64, 64), "fp32_dev", True, "entropic", (3, 7, 64)),
    # extents one off the own columns (58) and rows, and of one or two workgroups
    ((2, 58), "fp64", True, "entropic", (4, 3)),
    ((3, 59), "fp32_dev", False, "product", (6,)),
    ((10, 57), "fp64", False, "poly2", (9,)),
    ((11, 116), "fp32_dev", True, "poly2", (66,)),
    ((61, 117), "fp64", True, "product", (13,)),
    # fewer columns or rows than the halo (wrapped onto the domain itself)
    ((1, 1), "fp64", False, "entropic", (6,)),
    ((1, 70), "fp32_dev", False, "entropic", (4, 2)),
    ((70, 1), "fp64", True, "entropic", (5,)),
    ((5, 3), "fp32_dev", True, "entropic", (8, 64)),
    ((300, 17), "fp64", False, "entropic", (10,)),
    # two rows per wavefront, several workgroups per compute unit
    ((333, 500), "fp32_dev", True, "entropic", (6, 64)),
    ((300, 300), "fp64", False, "entropic", (7,)),
    ((512, 509), "fp64", True, "entropic", (11,)),
    # five steps: 56 own columns and one off, every remainder, rows the later steps leave out
    ((64, 64), "fp64", True, "entropic", (5, 6, 7, 8, 9, 105)),
    ((2, 56), "fp32_dev", False, "entropic", (10, 4)),
    ((9, 57), "fp64", False, "product", (15,)),
    ((17, 113), "fp32_dev", True, "poly2", (11, 3)),
    ((41, 167), "fp64", True, "entropic", (10, 2)),
    ((640, 601), "fp64", False, "entropic", (5, 9)),
    # several workgroups per compute unit: four steps with float storage
    ((509, 512), "fp32_dev", False, "entropic", (9, 2)),
]


@pytest.mark.parametrize("case", range(len(BLOCK_CASES)))
def test_d2q9_blocks_equal_one_step_bitwise(case):
    shape, dtype, corr, eq, chunks = BLOCK_CASES[case]
    _compare(shape, dtype, corr, eq, chunks, seed=600 + case)


D1_CASES = [  # nx, dtype, correction, equilibrium, step chunks
    (16, "fp64", True, "entropic", (1, 2, 15, 16, 17, 100)),
    (17, "fp32_dev", False, "entropic", (3, 16, 33)),
    (95, "fp32_dev", True, "entropic", (9, 16, 70)),
    (96, "fp64", False, "product", (10, 10, 64)),
    (97, "fp64", True, "poly2", (31,)),
    (113, "fp32_dev", True, "product", (8, 24)),
    (5003, "fp64", False, "entropic", (13, 100)),
    ((1 << 22) - 1, "fp32_dev", True, "entropic", (16, 5)),
    (1 << 22, "fp32_dev", True, "entropic", (8, 7, 9)),
    ((1 << 22) + 5, "fp64", True, "entropic", (8, 3)),
    ((1 << 22) + 3, "fp32_dev", False, "poly2", (11,)),
    ((1 << 23) + 2, "fp64", False, "product", (8, 1)),
    ((1 << 24) + 9, "fp32_dev", False, "entropic", (17,)),
    # 32, 24 and 16 steps per launch, and one node beyond each
    (600, "fp64", True, "entropic", (31, 32, 33, 100)),
    (1 << 17, "fp32_dev", False, "entropic", (32, 3)),
    ((1 << 17) + 1, "fp64", True, "product", (24, 25)),
    (400000, "fp32_dev", True, "poly2", (50,)),
    (400001, "fp64", False, "entropic", (33,)),
]


@pytest.mark.parametrize("case", range(len(D1_CASES)))
def test_d1q3_strips_equal_one_step_bitwise(case):
    nx, dtype, corr, eq, chunks = D1_CASES[case]
    _compare((nx,), dtype, corr, eq, chunks, seed=400 + case)


@pytest.mark.parametrize("shape,dtype", [((64, 64), "fp64"), ((1100, 900), "fp64"), ((400, 400), "fp32_dev"), ((3000,), "fp64")])
def test_strips_raise_the_domain_flag_as_one_step(shape, dtype):
    """A state about to leave the domain raises the flag in the same call, and
    the halo columns' and rows' unused values raise none in a healthy one."""
    lbm = _lbm()
    for umax in (0.97, 0.99, 0.3):
        rho0, u0 = workloads.random_field(shape, seed=7, umax=umax, rho_lo=0.3 if umax > 0.5 else 0.9,
                                          rho_hi=2.0 if umax > 0.5 else 1.1)
        with lbm.Domain(rho0, u0, 0.5001, dtype=dtype) as a, \
                lbm.Domain(rho0, u0, 0.5001, dtype=dtype, tuning=lbm.make_tuning(time_block=1)) as b:
            for n in (4, 6, 12):
                a.step(n)
                b.step(n)
                fa = a.moments(fields=False, raise_on_domain=False)[2]["domain_error"]
                fb = b.moments(fields=False, raise_on_domain=False)[2]["domain_error"]
                assert fa == fb, (umax, n)
