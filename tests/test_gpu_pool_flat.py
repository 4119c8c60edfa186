"""Two-step classes of flat slots: blocks of 14 rows only where the slots fill
more than half of them (1.9 times the nodes at most), else one step per launch
or, from 2^22 (FP32) and 2^20 (FP64) nodes on, sweeps.  The number of launches
tells one step per launch from two; every slot is bitwise its single-domain run."""
import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,shapes,steps,launches", [
    ("fp32_dev", [(1, 30001)], 4, 4),
    ("fp64", [(3, 9000), (2, 5000)], 5, 5),
    ("fp32_dev", [(7, 4000)], 4, 4),              # 2.0 times the nodes
    ("fp64", [(8, 4000)], 4, 2),                  # 1.75
    ("fp32_dev", [(15, 3001)], 4, 2),             # 1.87
    ("fp64", [(16, 301)], 4, 2),
    ("fp32_dev", [(3, 1000), (28, 1000)], 6, 3),  # the class as a whole: 1.36
    ("fp32_dev", [(1, 9000), (14, 200)], 6, 6),   # 10.9
    ("fp64", [(2, 600001)], 5, 3),                # sweeps and one step
    ("fp32_dev", [(2, 2100001)], 4, 2),
])
def test_flat_classes_equal_alone(dtype, shapes, steps, launches):
    from paper_2303_08163_amd import lbm
    fields = [workloads.random_field(s, seed=900 + k, umax=0.1) for k, s in enumerate(shapes)]
    with lbm.Pool(3 << 30, max_slots=8, tuning=lbm.make_pool_tuning(64, 4, time_block=2)) as pool:
        slots = [pool.admit(r, u, 0.55, steps, dtype=dtype) for r, u in fields]
        pool.run(steps)
        assert sorted(pool.poll()) == sorted(slots)
        assert pool.stats()["launches"] == launches
        for s, (r, u) in zip(slots, fields):
            with lbm.Domain(r, u, 0.55, dtype=dtype, tuning=lbm.make_tuning(time_block=1)) as d:
                d.step(steps)
                assert np.array_equal(d.populations(), pool.populations(s))
