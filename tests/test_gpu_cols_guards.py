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


def _blocks(opm, dims, blk):
    case = cases.box_case(*dims, seed=3)
    g = opm.GpuModel(case, ilu_blocks=blk, amg=False)
    y = g.state(cases.random_state(case, 5))
    R, J, _ = g.assemble(y, g.accumulation(g.state(cases.random_state(case, 6))), DAY)
    return g, R, J


@pytest.mark.parametrize("precision", [0, 1])
def test_box_that_was_never_set(opm, precision):
    """A box that the topology's counts contradict: factors and solution by
    position, bitwise those of the right box."""
    g, R, J = _blocks(opm, (24, 25, 15), (4, 4, 15))
    ilu, _ = g.ilu0_factor(J, precision)
    ref = g.ilu0_apply(ilu, R, precision)
    for box in (-1, 0x7fffffff, 2 | 2 << 10 | 15 << 20, 0x00cdcdcd):
        g.pb.ilu_box = box
        ilu, status = g.ilu0_factor(J, precision)
        assert int(status.item()) == 0
        assert torch.equal(g.ilu0_apply(ilu, R, precision), ref), hex(box)


@pytest.mark.parametrize("precision", [0, 1])
def test_transposed_box_is_refused(opm, precision):
    """A box with the counts of the topology's own but other subdomains:
    OPM_EINVAL where a status is given, and no finite solution; the Newton step
    returns OPM_EINVAL.  With the right box everything is as before."""
    g, R, J = _blocks(opm, (12, 12, 6), (2, 6, 6))
    right = g.pb.ilu_box
    ilu, status = g.ilu0_factor(J, precision)
    assert int(status.item()) == 0
    ref = g.ilu0_apply(ilu, R, precision)
    g.pb.ilu_box = 6 | 2 << 10 | 6 << 20
    ilu, status = g.ilu0_factor(J, precision)
    assert int(status.item()) == opm.EINVAL
    _factor(opm, g, J, ilu, None, precision)
    x = g.ilu0_apply(ilu, R, precision)
    assert torch.isnan(x).any() and not torch.isfinite(x.sum())
    y = g.initial_state()
    with pytest.raises(opm.OpmError):
        g.newton_step(y, g.initial_state(), DAY, opm.default_opts(g.case, precision=precision))
    g.pb.ilu_box = right
    ilu, status = g.ilu0_factor(J, precision)
    assert int(status.item()) == 0 and torch.equal(g.ilu0_apply(ilu, R, precision), ref)
