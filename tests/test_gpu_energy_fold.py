"""lbm_energy on both sides of the size where its partial sums are folded by a
second launch (100,000 nodes), and beyond one node per thread of 1024
workgroups.  Oracle: the same sum over the moment fields, by math.fsum.  The
terms are positive; a node's velocity is off by some 30 units of rounding of
populations of order one, 3e-14 of |u - U| ~ 0.1, and a thread's chain of
additions is at most 64 long: 1e-12 relative holds both with room."""
import math

import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(100000,), (100001,), (250, 400), (331, 303), (46, 46, 47), (47, 46, 47),
                                   (1025, 1024), (1500, 1201)])
@pytest.mark.parametrize("dtype", ["fp64", "fp32_dev"])
def test_energy_sum(shape, dtype):
    import torch
    from paper_2303_08163_amd import lbm
    rho0, u0 = workloads.random_field(shape, seed=sum(shape), umax=0.1)
    U, rho_ref = [0.03, -0.02, 0.01][:len(shape)], 1.05
    out = torch.full((3,), -1.0, dtype=torch.float64, device="cuda:0")
    with lbm.Domain(rho0, u0, 0.6, dtype=dtype) as d:
        d.step(3)
        for k in range(2):  # twice: the partials and the counter serve again
            d.energy(U, rho_ref, out=out[k:k + 1])
        rho, u, _ = d.moments()
        d.energy(U, rho_ref, out=out[2:3])
        torch.cuda.synchronize()
    du2 = sum((u[a] - U[a]) ** 2 for a in range(len(shape)))
    ref = math.fsum((0.5 * rho_ref * du2 + (rho - rho_ref) ** 2 / (6.0 * rho_ref)).ravel().tolist())
    e = out.cpu().numpy()
    assert e[0] == e[1] == e[2]
    assert abs(e[0] - ref) < 1e-12 * ref, (e[0], ref)
