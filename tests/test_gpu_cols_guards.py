"""What the ILU(0) by columns does with a wait that gives up in its
factorisation and with a box that does not belong to the topology: no wrong
preconditioner passes for a right one."""
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


def _factor(opm, g, J, ilu, status, precision):
    """opm_ilu0_factor; status may be None (the entry point takes NULL)."""
    assert opm.lib().opm_ilu0_factor(g._pbp(), opm._ptr(J), opm._ptr(ilu), precision,
                                     opm._ptr(status) if status is not None else None,
                                     opm._stream()) == opm.OK


@pytest.mark.parametrize("precision", [0, 1])
def test_tile_factorisation_gives_up_with_nan(opm, precision):
    """Tiles whose factorisation gave up waiting (a spin limit of zero polls):
    OPM_EHIP where a status is given, and a solve with such factors returns NaN
    in every value also where none is; the next factorisation is exact again."""
    case = cases.box_case(20, 18, 6, seed=3)
    g = opm.GpuModel(case, amg=False)
    y = g.state(cases.random_state(case, 5))
    R, J, _ = g.assemble(y, g.accumulation(g.state(cases.random_state(case, 6))), DAY)
    ilu, status = g.ilu0_factor(J, precision)
    assert int(status.item()) == 0
    ref = g.ilu0_apply(ilu, R, precision)
    try:
        opm.set_option(opm.OPT_PLANE_SPIN, 0)
        _factor(opm, g, J, ilu, status, precision)
        assert int(status.item()) == opm.EHIP
        _factor(opm, g, J, ilu, None, precision)
    finally:
        opm.set_option(opm.OPT_PLANE_SPIN, 1 << 18)
    assert torch.isnan(g.ilu0_apply(ilu, R, precision)).all()
    _factor(opm, g, J, ilu, None, precision)
    assert torch.equal(g.ilu0_apply(ilu, R, precision), ref)
