"""Pools whose two-step launches work in blocks: from the smallest class that
takes them to one beyond the last-level cache (where every second launch walks
its blocks in reverse and fewer workgroups share a compute unit).  Every slot
is bitwise its single-domain run of one step per launch."""
import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu
GiB = 1 << 30


@pytest.mark.parametrize("dtype,corr,shapes,runs,launches", [
    # 4095 and 4096 nodes in slots of at least two steps: one step per launch below, blocks from there
    ("fp64", False, [(63, 65)], (4,), 4),
    ("fp64", False, [(64, 64)], (4, 3), 2 + 2),
    ("fp32_dev", True, [(64, 63), (1, 64)], (6, 5), 3 + 3),
    # block edges: 62 columns and 14 rows, one off, narrower than the halo
    ("fp32_dev", False, [(14, 62), (15, 63), (13, 61), (28, 124), (1, 300), (300, 1), (29, 125)], (7,), 4),
    ("fp64", True, [(43, 187), (2, 2), (14, 63)], (8, 2), 4 + 1),
    # both buffers beyond 256 MiB: reverse walks; beyond 768 MiB: forward again
    ("fp32_dev", False, [(2003, 1999), (77, 33)], (6, 3), 3 + 2),
    ("fp64", True, [(1403, 1399), (77, 33)], (4, 5), 2 + 3),
    ("fp64", False, [(2401, 2399)], (5,), 3),
])
def test_block_launches_equal_alone(dtype, corr, shapes, runs, launches):
    from paper_2303_08163_amd import lbm
    fields = [workloads.random_field(s, seed=700 + k, umax=0.1) for k, s in enumerate(shapes)]
    total = sum(runs)
    with lbm.Pool(4 * GiB, max_slots=8, tuning=lbm.make_pool_tuning(64, 4, time_block=2)) as pool:
        slots = [pool.admit(r, u, 0.55, total, dtype=dtype, bulk_correction=corr) for r, u in fields]
        for k in runs:
            pool.run(k)
        assert sorted(pool.poll()) == sorted(slots)
        assert pool.stats()["launches"] == launches
        for s, (r, u) in zip(slots, fields):
            with lbm.Domain(r, u, 0.55, dtype=dtype, bulk_correction=corr,
                            tuning=lbm.make_tuning(time_block=1)) as d:
                d.step(total)
                assert np.array_equal(d.populations(), pool.populations(s))
            pool.release(s)
