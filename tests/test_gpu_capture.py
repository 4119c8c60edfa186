"""Runs recorded into the caller's own HIP graph: a replay goes on from the state
that the one before left when the run's launches of time_block steps, as
lbm_get_launch_info states them, are even in number, however many steps the
library puts into one launch.  Each replay is checked bitwise against one-step
launches, with moments (eager work and a wait) between the replays."""
import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu

CASES = [  # shape (nx last), dtype, steps per replay (even numbers of time_block launches)
    ((64, 64), "fp64", (2, 4, 6, 20, 32)),         # D2Q9 blocks
    ((300, 257), "fp32_dev", (2, 4, 12)),
    ((1100, 900), "fp64", (2, 4, 6, 10, 14)),      # D2Q9 strips of six and four
    ((1300, 1800), "fp32_dev", (4, 12)),           # of four
    ((2048, 2048), "fp32_dev", (4, 8, 7)),         # time_block 2
    ((64,), "fp64", (2, 16, 9)),                   # one row in one workgroup, time_block 8
    ((9,), "fp32_dev", (2, 10)),
    ((3000,), "fp64", (2, 16, 9, 32)),             # D1Q3 strips
    ((5000000,), "fp32_dev", (16, 11)),
    ((16, 16, 16), "fp32_dev", (2, 6, 10)),        # D3Q27 blocks
    ((80, 80, 80), "fp32_dev", (2, 6)),            # D3Q27 sweeps
]


def _launches(info, steps):
    return steps // info["time_block"] + steps % info["time_block"]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_replays_go_on_from_the_last_state(case):
    import torch
    from paper_2303_08163_amd import lbm
    shape, dtype, counts = CASES[case]
    rho0, u0 = workloads.random_field(shape, seed=800 + case, umax=0.1)
    for steps in counts:
        stream = torch.cuda.Stream()
        with lbm.Domain(rho0, u0, 0.57, dtype=dtype, stream=stream) as a, \
                lbm.Domain(rho0, u0, 0.57, dtype=dtype, tuning=lbm.make_tuning(time_block=1)) as b:
            assert _launches(a.launch_info(), steps) % 2 == 0
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
                a.step(steps)
            for _ in range(4):
                with torch.cuda.stream(stream):
                    g.replay()
                b.step(steps)
                ra, ua, _ = a.moments()
                rb, ub, _ = b.moments()
                assert np.array_equal(ra, rb) and np.array_equal(ua, ub), (shape, steps)
            assert np.array_equal(a.populations(), b.populations()), (shape, steps)


@pytest.mark.parametrize("nx,steps,every", [(64, 20, 10), (64, 48, 16), (300, 10, 5), (7, 6, 3)])
def test_replayed_histories_go_on_from_the_last_state(nx, steps, every):
    import torch
    from paper_2303_08163_amd import lbm
    rho0, u0 = workloads.random_field((nx,), seed=77, umax=0.1)
    n = steps // every + 1
    stream = torch.cuda.Stream()
    with lbm.Domain(rho0, u0, 0.57, dtype="fp64", stream=stream) as a, \
            lbm.Domain(rho0, u0, 0.57, dtype="fp64", tuning=lbm.make_tuning(time_block=1)) as b:
        assert steps // every * _launches(a.launch_info(), every) % 2 == 0
        out = torch.empty(n, dtype=torch.float64, device="cuda:0")
        ref = torch.empty_like(out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            a.energy_history(steps, every, None, 1.0, out=out)
        for k in range(4):
            with torch.cuda.stream(stream):
                g.replay()
            b.energy_history(steps, every, None, 1.0, out=ref)
            torch.cuda.synchronize()
            assert torch.equal(out, ref), k
            assert np.array_equal(a.populations(), b.populations()), k
