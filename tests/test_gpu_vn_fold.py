"""GPU test of lbm_vn_max_radius where a wavefront of 64 matrices holds many
states, one whole state, or the end of one and the start of the next: the runs
of equal states that the kernel folds before its atomics.

Oracle: the largest LAPACK spectral radius over the same wave vectors; both
eigensolvers are backward stable and the matrices' entries are O(1), so the
bound is that of the other radius tests, 1e-10 relative.
"""
import numpy as np
import pytest

from oracle import stability as ost

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,nk,n", [(1, 1, 130), (1, 3, 50), (1, 63, 5), (1, 64, 4), (1, 65, 5),
                                      (2, 1, 65), (2, 2, 33), (2, 7, 5), (2, 8, 3), (2, 9, 4)])
def test_runs_of_states(dim, nk, n):
    from paper_2303_08163_amd import vonneumann as vn
    rng = np.random.default_rng(100 * dim + nk)
    # neighbours differ widely: slow, well-damped states next to fast, weakly damped ones
    nus = np.exp(rng.uniform(np.log(1e-6), np.log(1.2), n))
    sp = np.where(np.arange(n) % 2 == 0, 0.05, 0.9) * rng.uniform(0.5, 1.0, n)
    th = rng.uniform(0, np.pi / 2, n) if dim == 2 else np.zeros(n)
    states = np.stack([0.5 + 3 * nus, sp * np.cos(th), sp * np.sin(th)], axis=1)
    r, bad = vn.max_radius(states, dim=dim, nk=nk)
    assert bad == 0
    # one wave vector per axis means k = 0
    ks = ost.k_grid(nk, dim) if nk > 1 else np.zeros((1, dim))
    for s, st in enumerate(states):
        ref = np.max(ost.batch_spectral_radius(st[0], st[1:1 + dim], ks))
        assert abs(r[s] - ref) < 1e-10 * max(1.0, ref), (s, st, r[s], ref)
