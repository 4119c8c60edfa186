"""Short D1Q3 rows, whole runs and energy histories in one workgroup and one
launch.  Steps are bitwise those of one-step launches (time_block = 1), float
storage rounding after each, and the energies those of lbm_energy."""
import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu


def _lbm():
    from paper_2303_08163_amd import lbm
    return lbm


# one wavefront, its edges, one and several wavefronts per SIMD, the longest
# row of plain runs (256) and of histories (1024), and one beyond each
SIZES = [1, 2, 3, 15, 63, 64, 65, 128, 255, 256, 257, 512, 513, 1000, 1024, 1025]


@pytest.mark.parametrize("k", range(len(SIZES)))
@pytest.mark.parametrize("dtype", ["fp64", "fp32_dev"])
def test_row_equals_one_step_launches_bitwise(k, dtype):
    import torch
    lbm = _lbm()
    nx = SIZES[k]
    eq = ("entropic", "poly2", "product")[k % 3]
    corr = k % 2 == 0
    rho0, u0 = workloads.random_field((nx,), seed=900 + k, umax=0.1)
    kw = dict(dtype=dtype, bulk_correction=corr, equilibrium=eq)
    U = [0.03]
    with lbm.Domain(rho0, u0, 0.55, **kw) as a, lbm.Domain(rho0, u0, 0.55, **kw) as c, \
            lbm.Domain(rho0, u0, 0.55, tuning=lbm.make_tuning(time_block=1), **kw) as b:
        hb = torch.empty(8, dtype=torch.float64, device=b.device)
        for steps, every in ((7, 1), (13, 13), (40, 8)):
            a.step(steps)
            hc = c.energy_history(steps, every, U, 1.02)
            b.energy(U, 1.02, out=hb[0:1])
            for r in range(1, steps // every + 1):
                b.step(every)
                b.energy(U, 1.02, out=hb[r:r + 1])
            torch.cuda.synchronize()
            assert torch.equal(hc, hb[:steps // every + 1]), (nx, steps)
            assert np.array_equal(a.populations(), b.populations()), (nx, steps)
            assert np.array_equal(c.populations(), b.populations()), (nx, steps)


@pytest.mark.parametrize("nx", [64, 100])
def test_row_runs_of_several_launches(nx):
    """More steps than one launch takes, with an interval that does not divide a launch's most."""
    import torch
    lbm = _lbm()
    rho0, u0 = workloads.random_field((nx,), seed=5, umax=0.1)
    with lbm.Domain(rho0, u0, 0.55) as a, lbm.Domain(rho0, u0, 0.55) as c, \
            lbm.Domain(rho0, u0, 0.55, tuning=lbm.make_tuning(time_block=1)) as b:
        a.step(35000)
        hc = c.energy_history(35000, 5000, [0.0], 1.0)
        hb = torch.empty(8, dtype=torch.float64, device=b.device)
        b.energy([0.0], 1.0, out=hb[0:1])
        for r in range(1, 8):
            b.step(5000)
            b.energy([0.0], 1.0, out=hb[r:r + 1])
        torch.cuda.synchronize()
        assert torch.equal(hc, hb)
        assert a.moments(fields=False)[2]["steps"] == c.moments(fields=False)[2]["steps"] == 35000
        assert np.array_equal(a.populations(), b.populations())
        assert np.array_equal(c.populations(), b.populations())


@pytest.mark.parametrize("nx", [60, 300])
def test_row_raises_the_domain_flag_as_one_step(nx):
    lbm = _lbm()
    for umax in (0.97, 0.99, 0.3):
        rho0, u0 = workloads.random_field((nx,), seed=7, umax=umax, rho_lo=0.3 if umax > 0.5 else 0.9,
                                          rho_hi=2.0 if umax > 0.5 else 1.1)
        with lbm.Domain(rho0, u0, 0.5001) as a, \
                lbm.Domain(rho0, u0, 0.5001, tuning=lbm.make_tuning(time_block=1)) as b:
            for n in (4, 6, 12):
                a.step(n)
                b.step(n)
                fa = a.moments(fields=False, raise_on_domain=False)[2]["domain_error"]
                fb = b.moments(fields=False, raise_on_domain=False)[2]["domain_error"]
                assert fa == fb, (umax, n)
