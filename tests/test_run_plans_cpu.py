"""Which launches a domain's runs take, by the rules that weigh launches of
several steps against one step per launch: the domains on both sides of each
rule that were timed in both forms (us per step: several steps / one)."""
import pytest

from paper_2303_08163_amd import lbm


def _steps(shape, dtype):
    return lbm.lbm_get_run_info(lbm.make_config(3 ** len(shape), shape, 0.6, dtype))["steps"]


# D2Q9, shape (x first)
@pytest.mark.parametrize("shape,dtype,several", [
    ((1, 300000), "fp32_dev", False),    # 78.7 / 11.8
    ((2, 1500000), "fp64", False),       # 320 / 107
    ((4, 7500), "fp32_dev", False),      # 3.9 / 2.9
    ((4, 7500), "fp64", False),          # 3.3 / 3.0
    ((8, 375000), "fp32_dev", False),    # 98 / 32
    ((8, 37500), "fp64", False),         # 11.1 / 8.3
    ((8, 1500000), "fp64", False),       # 323 / 299
    ((12, 1000000), "fp32_dev", False),  # 256 / 198
    ((16, 187500), "fp32_dev", False),   # 50 / 31
    ((300000, 1), "fp32_dev", False),    # 9.5 / 5.6
    ((300000, 1), "fp64", False),        # 9.5 / 8.0
    ((150000, 2), "fp64", False),        # 9.8 / 8.7
    ((1500000, 2), "fp32_dev", False),   # 46 / 33
    ((8, 3750), "fp32_dev", True),       # 2.2 / 2.8
    ((12, 250000), "fp64", True),        # 57 / 85
    ((16, 18750), "fp64", True),         # 6.8 / 8.0
    ((16, 750000), "fp64", True),        # 165 / 290
    ((24, 125000), "fp32_dev", True),    # 35 / 44
    ((32, 9375), "fp32_dev", True),      # 5.0 / 5.3
    ((64, 46875), "fp32_dev", True),     # 28 / 31
    ((600000, 5), "fp32_dev", True),     # 26 / 33
    ((60000, 5), "fp64", True),          # 6.1 / 8.3
    ((1, 3000), "fp64", True),           # 1.8 / 3.5
    ((3000, 1), "fp32_dev", True),       # 1.2 / 2.6
    ((333, 500), "fp32_dev", True),
    ((1024, 1024), "fp64", True),
    ((3000, 2001), "fp64", True),
    ((4096, 4096), "fp32_dev", True),
])
def test_d2q9(shape, dtype, several):
    assert (_steps(shape, dtype) > 2) == several


# D3Q27 domains large enough for sweeps
@pytest.mark.parametrize("shape,dtype,several", [
    ((16, 4, 25000), "fp32_dev", False),    # 129 / 74
    ((16, 8, 12500), "fp32_dev", False),    # 95 / 76
    ((16, 256, 256), "fp32_dev", False),    # 43 / 34
    ((1000, 1000, 1), "fp32_dev", False),   # 45 / 32
    ((600, 600, 2), "fp32_dev", False),     # 28 / 24
    ((1024, 512, 1), "fp32_dev", False),    # 26 / 22
    ((128, 64, 64), "fp32_dev", False),     # 18.2 / 17.2
    ((16, 4, 25000), "fp64", False),        # 140 / 129
    ((35, 86, 57), "fp64", False),          # 18.7 / 16.2
    ((16, 128, 128), "fp64", False),        # 18.0 / 17.5
    ((16, 256, 256), "fp64", True),         # 70 / 88
    ((16, 8, 12500), "fp64", True),         # 108 / 130
    ((20, 256, 256), "fp32_dev", True),     # 65 / 86
    ((33, 128, 128), "fp32_dev", True),     # 22 / 27
    ((36, 200, 256), "fp64", True),
    ((33, 200, 200), "fp32_dev", True),
    ((512, 4, 512), "fp32_dev", True),      # 31 / 47
    ((100, 7, 1000), "fp32_dev", True),     # 22 / 26
    ((64, 64, 64), "fp64", True),           # 15.7 / 17.5
    ((128, 128, 128), "fp32_dev", True),
    ((256, 256, 256), "fp32_dev", True),
    ((256, 256, 256), "fp64", True),
    ((150, 131, 120), "fp64", True),
])
def test_d3q27_sweeps(shape, dtype, several):
    assert (_steps(shape, dtype) == 2) == several


# small D3Q27 domains
@pytest.mark.parametrize("shape,dtype,several", [
    ((147, 5, 40), "fp32_dev", False),    # 4.6 / 3.7
    ((108, 23, 19), "fp32_dev", False),   # 5.2 / 4.3
    ((108, 9, 49), "fp32_dev", False),    # 5.0 / 4.2
    ((111, 20, 22), "fp32_dev", False),   # 5.0 / 4.3
    ((115, 30, 15), "fp32_dev", False),   # 5.3 / 4.6
    ((101, 31, 14), "fp32_dev", False),   # 5.2 / 4.4
    ((16, 16, 16), "fp32_dev", True),     # 2.7 / 3.7
    ((32, 32, 32), "fp32_dev", True),
    ((40, 40, 40), "fp32_dev", True),
    ((256, 16, 16), "fp32_dev", True),    # 4.9 / 7.3
    ((48, 48, 48), "fp32_dev", True),     # 5.9 / 6.9
    ((48, 48, 48), "fp64", True),         # 8.1 / 9.9
    ((16, 16, 256), "fp64", True),
])
def test_d3q27_blocks(shape, dtype, several):
    assert (_steps(shape, dtype) == 2) == several
