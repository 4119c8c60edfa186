"""Handles come and go while others work: lbm_destroy waits for its own stream
alone, and the pinned result block that a handle gives back serves a later one,
in slabs of 64 up to 1024 blocks (handles beyond those copy their results)."""
import threading

import numpy as np
import pytest

from paper_2303_08163_amd import workloads

pytestmark = pytest.mark.gpu


def test_destroy_does_not_wait_for_other_streams():
    import torch
    from paper_2303_08163_amd import lbm
    rho0, u0 = workloads.taylor_green_2d(2048)
    rs, us = workloads.taylor_green_2d(64)
    busy, own = torch.cuda.Stream(), torch.cuda.Stream()
    with lbm.Domain(rho0, u0, 0.6, dtype="fp64", stream=busy) as big:
        small = lbm.Domain(rs, us, 0.6, dtype="fp64", stream=own)
        small.step(10)
        small.moments(fields=False)
        torch.cuda.synchronize()
        end = torch.cuda.Event()
        big.step(30000)  # half a second and more
        end.record(busy)
        small.close()
        assert not end.query(), "lbm_destroy waited for the other domain's steps"
        with lbm.Domain(rs, us, 0.6, dtype="fp64", stream=own) as again:
            assert again.moments(fields=False)[2]["steps"] == 0
        assert not end.query(), "lbm_destroy waited for the other domain's steps"
        big.moments(fields=False)


@pytest.mark.parametrize("count", [64, 65, 1024, 1026])
def test_many_handles_read_their_own_results(count):
    from paper_2303_08163_amd import lbm
    doms, mass = [], []
    try:
        for k in range(count):
            doms.append(lbm.Domain(np.full(8, 1.0 + k / 4096.0), np.zeros((1, 8)), 0.6, dtype="fp64"))
            mass.append(doms[k].moments(fields=False)[2]["mass"])
        assert [round((m / 8 - 1) * 4096) for m in mass] == list(range(count))
        for k in reversed(range(count)):
            assert doms[k].moments(fields=False)[2]["mass"] == mass[k]
    finally:
        for d in doms:
            d.close()


def test_threads_create_and_destroy():
    import torch
    from paper_2303_08163_amd import lbm
    errors = []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            for k in range(40):
                rho = 1.0 + (40 * i + k) / 1024.0
                with lbm.Domain(np.full(16, rho), np.zeros((1, 16)), 0.6, dtype="fp64", stream=stream) as d:
                    assert round((d.moments(fields=False)[2]["mass"] / 16 - 1) * 1024) == 40 * i + k
        except Exception as e:  # noqa: BLE001 -- reported by the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors, errors
