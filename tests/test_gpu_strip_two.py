"""D1Q3 launches of two steps, named by the tuning or left at the end of a run,
on rows around the length where lanes take more columns (2^22 nodes; doubles do
so from four steps per launch on).  Bitwise the one-step-per-launch run."""
import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [16, 113, (1 << 22) - 1, 1 << 22, (1 << 22) + 37, (1 << 23) + 2])
@pytest.mark.parametrize("dtype", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("block", [2, 4, 0])
def test_short_launches_equal_one_step_bitwise(nx, dtype, block):
    from paper_2303_08163_amd import lbm
    rho0, u0 = workloads.random_field((nx,), seed=nx % 1000 + block, umax=0.1)
    kw = dict(dtype=dtype, bulk_correction=True)
    tun = lbm.make_tuning(time_block=block) if block else None
    with lbm.Domain(rho0, u0, 0.55, tuning=tun, **kw) as a, \
            lbm.Domain(rho0, u0, 0.55, tuning=lbm.make_tuning(time_block=1), **kw) as b:
        for n in (2, 3, 4, 11):
            a.step(n)
            for _ in range(n):
                b.step(1)
            assert np.array_equal(a.populations(), b.populations()), n
