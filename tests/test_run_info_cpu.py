"""lbm_get_run_info: the launch that a domain's runs are made of, from the
configuration and tuning alone (host logic, no GPU)."""
import pytest

from paper_2303_08163_amd import lbm


def _info(shape, dtype="fp32_dev", eq="entropic", z_halo=False, **tun):
    lattice = 3 ** len(shape)
    cfg = lbm.make_config(lattice, shape, 0.6, dtype, equilibrium=eq, z_halo=z_halo)
    return lbm.lbm_get_run_info(cfg, lbm.make_tuning(**tun) if tun else None)


# shape (x first), dtype, kernel, steps, (cols, rows, planes)
@pytest.mark.parametrize("shape,dtype,kernel,steps,own", [
    ((256, 256, 256), "fp32_dev", "sweep", 2, (64, 8, 128)),  # the headline box
    ((256, 256, 256), "fp64", "sweep", 2, (64, 4, 256)),
    ((150, 131, 120), "fp64", "sweep", 2, None),
    ((48, 48, 48), "fp32_dev", "block", 2, (12, 6, 6)),
    ((256, 16, 16), "fp32_dev", "block", 2, None),
    ((64, 64, 64), "fp32_dev", "node", 1, (64, 4, 1)),
    ((4096, 4096), "fp32_dev", "strip", 4, None),
    ((4096, 4096), "fp64", "strip", 6, None),
    ((1024, 1024), "fp64", "strip", 6, None),
    ((64, 64), "fp64", "block", 5, None),
    ((500, 333), "fp32_dev", "block", 5, None),
    ((512, 512), "fp32_dev", "block", 4, None),
    ((1 << 27,), "fp32_dev", "strip", 8, (496, 1, 1)),
    ((3000,), "fp64", "strip", 32, (64, 1, 1)),
    ((64,), "fp64", "row", 16384, (64, 1, 1)),
    ((500,), "fp64", "strip", 32, (64, 1, 1)),
])
def test_default_runs(shape, dtype, kernel, steps, own):
    i = _info(shape, dtype)
    assert (i["kernel"], i["steps"]) == (kernel, steps), i
    if own:
        assert (i["cols"], i["rows"], i["planes"]) == own, i


def test_named_launches_and_other_forms():
    # a tuning that names the launch gets it
    assert _info((256, 256, 256), time_block=1)["kernel"] == "vector"
    assert _info((256, 256, 256), time_block=1)["steps"] == 1
    two = _info((4096, 4096), time_block=2)
    assert (two["kernel"], two["steps"], two["cols"]) == ("two_step", 2, 1024)
    assert _info((3000,), time_block=4)["kernel"] == "multi_step"
    assert _info((3000,), time_block=4)["steps"] == 4
    assert _info((64, 64, 64), block_x=64, block_y=1)["steps"] == 1
    # z-slabs and the other storage types keep one step per launch
    assert _info((256, 256, 256), z_halo=True)["steps"] == 1
    assert _info((256, 256, 256), "fp32_dev_mixed")["steps"] == 1
    assert _info((64,), "fp32_dev_f32")["steps"] == 1


def test_refusals_are_those_of_create():
    cfg = lbm.make_config(9, (64, 64), 0.5)
    with pytest.raises(lbm.LBMError) as e:
        lbm.lbm_get_run_info(cfg)
    assert e.value.status == lbm.LBM_EINVAL
    cfg = lbm.make_config(27, (64, 64, 64), 0.6)
    with pytest.raises(lbm.LBMError):
        lbm.lbm_get_run_info(cfg, lbm.make_tuning(time_block=2))
    lib = lbm.load_library()
    assert lib.lbm_get_run_info(None, None, None) == lbm.LBM_EINVAL
