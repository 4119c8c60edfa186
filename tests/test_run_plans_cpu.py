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
