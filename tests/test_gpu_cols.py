"""The ILU(0) by lattice columns (one workgroup per subdomain of a block ILU0,
per small system, or per tile of a whole lattice) against the one-launch-per-
level shape: the same row arithmetic in the same order, so inverse pivots and
solutions are bitwise equal.  Boxes and tiles of one and several wavefronts,
ragged edges, masked grids, boxes shorter than the columns, grids of one tile
per axis, and repeated applications (the exchange arrays are refilled)."""
import pytest
import torch

from paper_1910_06059_amd import cases
from paper_1910_06059_amd.cases import DAY

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def opm():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1910_06059_amd import opm as _opm
    _opm.init()
    return _opm


def _masked():
    import numpy as np
    return cases.box_case(19, 13, 6, seed=6, wells=[], mask=cases.masked_mask(
        np.random.default_rng(9), (6, 13, 19), 900))


SHAPES = {
    "one_wave": (lambda: cases.box_case(12, 9, 11, seed=3), (4, 4, 11)),
    "ragged_two_waves": (lambda: cases.box_case(13, 11, 7, seed=3), (5, 6, 7)),
    "cut_columns": (lambda: cases.box_case(9, 10, 13, seed=3), (8, 8, 5)),
    "eight_waves": (lambda: cases.box_case(24, 13, 9, seed=3), (11, 11, 9)),
    "masked_blocks": (_masked, (7, 5, 6)),
    "one_box": (cases.config1, None),
    "tiles": (lambda: cases.box_case(17, 18, 10, seed=3), None),
    "tiles_one_row": (lambda: cases.box_case(40, 5, 6, seed=4), None),
    "tiles_one_column": (lambda: cases.box_case(3, 60, 9, seed=4), None),
    "tiles_tall": (lambda: cases.box_case(16, 9, 70, seed=4), None),
    "tiles_masked": (_masked, None),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(SHAPES))
def test_columns_bitwise_equal(opm, name, precision):
    make, blk = SHAPES[name]
    case = make()
    print(f"columns: {name} {case.name} precision {precision}", flush=True)
    g = opm.GpuModel(case, ilu_blocks=blk, amg=False)
    y = g.state(cases.random_state(case, 5))
    acc0 = g.accumulation(g.state(cases.random_state(case, 6)))
    R, J, _ = g.assemble(y, acc0, DAY)
    ns = (g.n + 63) // 64 * 64
    npiv = 8 * 9 * ns if precision == 0 else 12 * 9 * ns
    r2 = torch.flip(R, [0]).contiguous()
    out = []
    try:
        for mode in (-1, 1):
            opm.set_option(opm.OPT_SWEEP_MODE, mode)
            ilu, status = g.ilu0_factor(J, precision)
            assert int(status.item()) == 0
            out.append([ilu[:npiv].clone()] + [g.ilu0_apply(ilu, r, precision)
                                               for r in (R, r2, R, R)])
    finally:
        opm.set_option(opm.OPT_SWEEP_MODE, -1)
    assert torch.isfinite(out[1][1]).all()
    for q, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a, b), (name, precision, q)


def test_columns_without_lattice(opm):
    """Without the box of the block topology the position lists are used: the
    same factors and solution."""
    case = cases.config2()
    g = opm.GpuModel(case, ilu_blocks=(4, 4, 15), amg=False)
    assert g.pb.ilu_box == 4 | 4 << 10 | 15 << 20
    y = g.state(cases.random_state(case, 5))
    R, J, _ = g.assemble(y, g.accumulation(g.state(cases.random_state(case, 6))), DAY)
    ilu, _ = g.ilu0_factor(J)
    x = g.ilu0_apply(ilu, R)
    g.pb.ilu_box = 0
    ilu, _ = g.ilu0_factor(J)
    assert torch.equal(g.ilu0_apply(ilu, R), x)


def test_tiles_give_up_with_nan(opm):
    """A tile whose wait gives up (a spin limit of zero polls) takes NaN: the
    solve returns NaN instead of hanging, BiCGStab reports it, and the next
    application with the normal limit is exact again."""
    case = cases.box_case(20, 18, 6, seed=3)
    g = opm.GpuModel(case, amg=False)
    y = g.state(cases.random_state(case, 5))
    R, J, _ = g.assemble(y, g.accumulation(g.state(cases.random_state(case, 6))), DAY)
    ilu, _ = g.ilu0_factor(J)
    ref = g.ilu0_apply(ilu, R)
    try:
        opm.set_option(opm.OPT_PLANE_SPIN, 0)
        bad = g.ilu0_apply(ilu, R)
        assert torch.isnan(bad).all()
        x, rep = g.bicgstab(J, ilu, -R, rtol=1e-6)
        assert rep.status != 0
    finally:
        opm.set_option(opm.OPT_PLANE_SPIN, 1 << 18)
    assert torch.equal(g.ilu0_apply(ilu, R), ref)
