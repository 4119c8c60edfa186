"""The kernels that runs are made of, each named by the domain's plan
(lbm_get_run_info) or by an explicit time_block, so that the kernel meant is the
one that runs:

* the D3Q27 sweeps of the headline box (rows of 256 nodes, tiles of 64 own
  columns) against the oracle over the headline's 500 steps, and at 256^3 itself
  bitwise against one step per launch;
* the one-step vector kernels (time_block 1) against the oracle, 500 steps;
* the two-step LDS kernel (time_block 2) at 4096^2 and on a ragged 4000^2, bitwise;
* step graphs, where there are any, bitwise against calls of one step.

Oracle tolerances as for the box runs of 16 x 16 cross-sections: normwise over
the field FP64 1e-12, FP32 deviation storage 1e-5; wider cross-sections amplify
rounding differences less.
"""
import numpy as np
import pytest

import oracle
from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32_dev": 1e-5}
TAU, STEPS = 0.5005, 500


def _lbm():
    from paper_2303_08163_amd import lbm
    return lbm


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b))) / np.max(np.abs(b)))


def _against_oracle(d, box, corr, tol, what):
    rho0, u0 = workloads.taylor_green_3d_box(*box, u0=0.05)
    oracle.set_threads(16)
    r_ref, u_ref, bad = oracle.run(rho0, u0, TAU, STEPS, corr="min" if corr else "off")
    assert bad == 0
    d.step(STEPS)
    rho, u, diag = d.moments()
    er, eu = _rel(rho, r_ref), _rel(u, u_ref)
    print(f"[parity] D3Q27 {box} {STEPS} steps {what} corr={corr}: rel err rho {er:.3e} u {eu:.3e}", flush=True)
    assert diag["steps"] == STEPS and not diag["domain_error"]
    assert er < tol and eu < tol


@pytest.mark.parametrize("dtype,box", [("fp32_dev", (256, 64, 32)), ("fp64", (256, 32, 30))])
@pytest.mark.parametrize("corr", [False, True])
def test_sweep_full_steps_vs_oracle(dtype, box, corr):
    lbm = _lbm()
    rho0, u0 = workloads.taylor_green_3d_box(*box, u0=0.05)
    with lbm.Domain(rho0, u0, TAU, dtype=dtype, bulk_correction=corr) as d:
        run = d.run_info()
        assert (run["kernel"], run["steps"], run["cols"]) == ("sweep", 2, 64), run
        head = lbm.lbm_get_run_info(lbm.make_config(27, (256, 256, 256), TAU, dtype, corr))
        assert (head["kernel"], head["steps"], head["cols"]) == ("sweep", 2, 64), head
        _against_oracle(d, box, corr, TOL[dtype], f"{dtype} sweep")


@pytest.mark.parametrize("dtype", ["fp32_dev", "fp64"])
def test_headline_box_equals_one_step_bitwise(dtype):
    import torch
    lbm = _lbm()
    g = torch.Generator(device="cuda:0").manual_seed(256)
    shape = (256, 256, 256)
    rho = 0.8 + 0.4 * torch.rand(shape, generator=g, dtype=torch.float64, device="cuda:0")
    u = 0.1 * (2 * torch.rand((3,) + shape, generator=g, dtype=torch.float64, device="cuda:0") - 1)
    out = [torch.empty((27,) + shape, dtype=torch.float64, device="cuda:0") for _ in range(2)]
    with lbm.Domain(rho, u, TAU, dtype=dtype) as a, \
            lbm.Domain(rho, u, TAU, dtype=dtype, tuning=lbm.make_tuning(time_block=1)) as b:
        assert a.run_info()["kernel"] == "sweep" and b.run_info()["kernel"] == "vector"
        for n in (4, 3):
            a.step(n)
            b.step(n)
            for d, o in zip((a, b), out):
                lbm.lbm_get_populations(d.handle, o.data_ptr())
            assert torch.equal(*out), n


@pytest.mark.parametrize("dtype,nx", [("fp32_dev", 256), ("fp64", 256), ("fp64", 128)])
@pytest.mark.parametrize("corr", [False, True])
def test_one_step_vector_kernels_vs_oracle(dtype, nx, corr):
    lbm = _lbm()
    box = (nx, 16, 16)
    rho0, u0 = workloads.taylor_green_3d_box(*box, u0=0.05)
    with lbm.Domain(rho0, u0, TAU, dtype=dtype, bulk_correction=corr, tuning=lbm.make_tuning(time_block=1)) as d:
        run, info = d.run_info(), d.launch_info()
        assert (run["kernel"], run["steps"]) == ("vector", 1), run
        npt = 4 if dtype == "fp32_dev" else 2
        assert info["row_wave"] == (1 if nx == 64 * npt else 0) and info["graph_steps"] == 32
        _against_oracle(d, box, corr, TOL[dtype], f"{dtype} vector, row wave {info['row_wave']}")


@pytest.mark.parametrize("dtype,n,cols", [("fp32_dev", 4096, 1024), ("fp64", 4096, 128), ("fp32_dev", 4000, 1024)])
def test_two_step_kernel_full_size_bitwise(dtype, n, cols):
    lbm = _lbm()
    rho0, u0 = workloads.random_field((n, n), seed=50 + n, umax=0.1)
    with lbm.Domain(rho0, u0, 0.51, dtype=dtype, tuning=lbm.make_tuning(time_block=2)) as a:
        run = a.run_info()
        assert (run["kernel"], run["steps"], run["cols"]) == ("two_step", 2, cols), run
        a.step(5)
        fa = a.populations()
    with lbm.Domain(rho0, u0, 0.51, dtype=dtype, tuning=lbm.make_tuning(time_block=1)) as b:
        b.step(5)
        assert np.array_equal(fa, b.populations())


GRAPHS = [  # shape, dtype, time_block (0: the library's choice), steps per replay
    ((64, 64), "fp64", 1, 32),
    ((33, 70), "fp32_dev", 1, 32),
    ((256,), "fp64", 1, 32),
    ((2048,), "fp64", 8, 32),
    ((40, 128), "fp32_dev", 2, 32),
    ((16, 16, 16), "fp32_dev", 0, 32),
    ((7, 9, 13), "fp32_dev", 1, 32),
    ((64, 64), "fp64", 0, 0),
    ((256,), "fp64", 0, 0),
]


@pytest.mark.parametrize("case", range(len(GRAPHS)))
def test_step_graphs_equal_calls_of_one_step_bitwise(case):
    lbm = _lbm()
    shape, dtype, block, graph = GRAPHS[case]
    rho0, u0 = workloads.random_field(shape, seed=40 + case, umax=0.1)
    tun = lbm.make_tuning(time_block=block) if block else None
    with lbm.Domain(rho0, u0, 0.58, dtype=dtype, tuning=tun) as a, \
            lbm.Domain(rho0, u0, 0.58, dtype=dtype, tuning=lbm.make_tuning(time_block=1)) as b:
        assert a.launch_info()["graph_steps"] == graph
        for n in (1, 100, 64, 3, 257):  # from both buffers
            a.step(n)
            for _ in range(n):
                b.step(1)
            ra, ua, _ = a.moments()
            rb, ub, _ = b.moments()
            assert np.array_equal(ra, rb) and np.array_equal(ua, ub), n
        assert np.array_equal(a.populations(), b.populations())
