"""The tile plans of the mass-transfer passes, as mtpt_plan states them (host
arithmetic: no GPU)."""
import ctypes as C

import pytest

from paper_2204_03756_amd import mtpt, workloads as W


def _cube(n, per_unit, ns, prec, d_mt, dt, **kw):
    """A 3-d sim of n particles, per_unit of them in a unit of volume."""
    side = (n / per_unit) ** (1.0 / 3.0)
    return W.Params(dim=3, n=n, lo=[0.0] * 3, hi=[side] * 3, d_rw=d_mt, d_mt=d_mt, dt=dt, n_species=ns, precision=prec,
                    **kw)


def test_plan_covers_the_grid_and_checks_its_arguments():
    p = _cube(100_003, 1.0, 3, W.FP64, 0.7, 0.05)
    plan = mtpt.mtpt_plan(p)
    nc = [int(p.hi[k] / (p.psi_eff * (1 + 1e-6))) for k in range(3)]
    for tile, tiles in ((plan["tile"], plan["tiles"]), (plan["ttile"], plan["ttiles"])):
        assert tiles == -(-nc[0] // tile[0]) * -(-nc[1] // tile[1]) * -(-nc[2] // tile[2])
    lib, q = mtpt.load(), mtpt.make_params(p)
    assert lib.mtpt_plan(C.byref(q), None) == mtpt.MTPT_E_ARG
    assert lib.mtpt_sim_plan(None, C.byref(mtpt.mtpt_plan_t())) == mtpt.MTPT_E_ARG
    q.dt = 0.0
    with pytest.raises(mtpt.MtptError):
        mtpt.mtpt_plan(q)


@pytest.mark.parametrize("n", [120_001, 175_693, 203_301, 224_999, 241_927, 282_953, 342_375])
def test_tiles_on_both_sides_of_the_rule_for_few_tiles(n):
    """FP64 walks of one particle in a unit of volume: tiles for every compute
    unit to spare, so none of less than half a workgroup.  (The rule for few
    tiles once priced shapes past its line in waves and the others in
    workgroups, and took tiles of 105 particles.)"""
    plan = mtpt.mtpt_plan(_cube(n, 1.0, 1, W.FP64, 1.0, 0.1))
    nc = int((n ** (1.0 / 3.0)) / (3.0 * 0.4 ** 0.5 * (1 + 1e-6)))
    for t in (plan["tile"], plan["ttile"]):
        assert t[0] * t[1] * t[2] * n / nc ** 3 >= 128, plan


@pytest.mark.parametrize("n,hi,ns", [(971, [6.1, 11.6, 15.8], 1), (1331, [16.3, 23.0, 3.4], 1), (1081, [17.8, 3.0, 18.9], 3)])
def test_list_tiles_are_doubled_inside_the_grid_only(n, hi, ns, monkeypatch):
    """Boxes as thin as their transfer tile: two of them make a list tile along
    an axis where the grid has two."""
    monkeypatch.setenv("MTPT_MIN_TILES", "1")
    plan = mtpt.mtpt_plan(W.Params(dim=3, n=n, lo=[0.0] * 3, hi=hi, d_rw=0.3, d_mt=1.1 ** 2 / 3.6, dt=0.1, psi=1.1,
                                   n_species=ns, precision=W.FP64))
    for axis in range(3):
        if plan["lists"] and plan["tile"][axis] != plan["ttile"][axis]:
            assert plan["ttile"][axis] < int(hi[axis] / (1.1 * (1 + 1e-6))), plan


@pytest.mark.parametrize("n", [200_003, 221_717, 443_990, 1_000_001, 1_727_426, 2_256_415, 8_000_000, 20_000_000, 32_000_000])
def test_reacting_sims_of_every_size_take_lists(n):
    """The reacting workload's density: also where the transfer pass's best tile
    is eight cells wide, whose double reaches past the mask variant's limit."""
    plan = mtpt.mtpt_plan(_cube(n, 32e6 / 318.0 ** 3, 3, W.FP64, 0.7, 0.05))
    assert plan["lists"], plan
    assert plan["tile"][0] * plan["tile"][1] * plan["tile"][2] <= 12 * 6 * 6


@pytest.mark.parametrize("n,neighbours,ns", [(200_003, 4.4, 3), (1_000_001, 5.0, 3), (4_000_003, 5.0, 3), (4_000_003, 5.9, 1)])
def test_list_tiles_fill_their_workgroup(n, neighbours, ns):
    """A workgroup of 512 threads takes about as long for half as many
    particles: where two transfer tiles or a larger one fill it, they do."""
    psi = 1.1
    per_unit = neighbours / (4.18879 * psi ** 3)
    plan = mtpt.mtpt_plan(_cube(n, per_unit, ns, W.FP64, psi * psi / 3.6, 0.1, psi=psi))
    nc = int((n / per_unit) ** (1.0 / 3.0) / (psi * (1 + 1e-6)))
    assert plan["lists"] and plan["tile"][0] * plan["tile"][1] * plan["tile"][2] * n / nc ** 3 >= 384, plan
