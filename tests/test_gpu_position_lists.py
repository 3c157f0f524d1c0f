"""The ILU(0) by position lists, which a lattice reaches only where the column shape
does not suit it (or with OPT_SWEEP_MODE): the one-workgroup ring kernels, and the
sweeps of one workgroup per subdomain, plain and fused with BiCGStab, at one and
two levels of loads in flight.  Every shape computes a row in the same order:
bitwise equal to one launch per level, and to the columns."""
import numpy as np
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


def _system(opm, case, blk):
    g = opm.GpuModel(case, ilu_blocks=blk, amg=False)
    y = g.state(cases.random_state(case, 5))
    R, J, _ = g.assemble(y, g.accumulation(g.state(cases.random_state(case, 6))), DAY)
    return g, R, J


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dims", [(24, 25, 15), (30, 30, 12)])
def test_ring_kernels(opm, dims, precision):
    """Kernels 1 to 6 and the automatic one, with one workgroup forced; levels
    wider than 256 and 128 threads."""
    case = cases.box_case(*dims, seed=9)
    g, R, J = _system(opm, case, None)
    assert g.max_level > 256
    ring = 1 << (g.sweep_span + g.max_level).bit_length()
    assert 8 * 3 * ring <= 128 * 1024   # (the sweep takes the ring)
    cols, _ = g.ilu0_factor(J, precision)
    ref = g.ilu0_apply(cols, R, precision)
    assert torch.isfinite(ref).all()
    try:
        opm.set_option(opm.OPT_SWEEP_MODE, 0)
        ilu, status = g.ilu0_factor(J, precision)
        assert int(status.item()) == 0
        for kind in range(7):
            opm.set_option(opm.OPT_SWEEP_KERNEL, kind)
            for r in (R, R):
                assert torch.equal(g.ilu0_apply(ilu, r, precision), ref), (kind, precision)
    finally:
        opm.set_option(opm.OPT_SWEEP_KERNEL, 0)
        opm.set_option(opm.OPT_SWEEP_MODE, -1)


# threads of a workgroup, bounds in registers (at most 64 levels) or not, levels
# wider than the workgroup
BLOCKS = {
    "one_wave": ((24, 25, 15), (4, 4, 15)),
    "one_wave_tall": ((8, 9, 70), (4, 4, 70)),
    "two_waves": ((13, 11, 9), (5, 6, 9)),
    "four_waves": ((17, 18, 12), (8, 8, 12)),
    "four_waves_tall": ((9, 16, 60), (8, 8, 60)),
    "wide": ((24, 23, 9), (12, 12, 9)),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("depth", [0, 1, 2])
@pytest.mark.parametrize("name", list(BLOCKS))
def test_subdomain_sweeps_and_fused_krylov(opm, name, depth, precision):
    dims, blk = BLOCKS[name]
    case = cases.box_case(*dims, seed=3)
    g, R, J = _system(opm, case, blk)
    print(f"position lists: {name} depth {depth} precision {precision}", flush=True)
    out = []
    try:
        opm.set_option(opm.OPT_BLOCK_DEPTH, depth)
        for mode in (2, 1):
            opm.set_option(opm.OPT_SWEEP_MODE, mode)
            ilu, status = g.ilu0_factor(J, precision)
            assert int(status.item()) == 0
            x, rep = g.bicgstab(J, ilu, -R, rtol=1e-6, precision=precision)
            assert rep.status == 0
            out.append((g.ilu0_apply(ilu, R, precision), x.cpu().numpy(), rep.its, rep.half))
    finally:
        opm.set_option(opm.OPT_SWEEP_MODE, -1)
        opm.set_option(opm.OPT_BLOCK_DEPTH, 0)
    assert torch.equal(out[0][0], out[1][0])
    assert out[0][2:] == out[1][2:]
    # only the order of the dot products differs; FP32 sweeps pass their last
    # bits on at their own rounding
    tol = 1e-9 if precision == 0 else 1e-7
    assert np.abs(out[0][1] - out[1][1]).max() <= tol * np.abs(out[1][1]).max()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["wide", "no_box", "short"])
def test_automatic_choice_by_position(opm, name, precision):
    """What the automatic mode gives the position lists: boxes of more than 128
    columns, a topology without its box, boxes with few rows per level."""
    dims, blk = {"wide": BLOCKS["wide"], "no_box": BLOCKS["one_wave"],
                 "short": ((20, 19, 3), (8, 8, 3))}[name]
    g, R, J = _system(opm, cases.box_case(*dims, seed=4), blk)
    if name == "no_box":
        g.pb.ilu_box = 0
    out = []
    try:
        for mode in (-1, 2, 1):
            opm.set_option(opm.OPT_SWEEP_MODE, mode)
            ilu, status = g.ilu0_factor(J, precision)
            assert int(status.item()) == 0
            x, rep = g.bicgstab(J, ilu, -R, rtol=1e-6, precision=precision)
            assert rep.status == 0
            out.append((g.ilu0_apply(ilu, R, precision), x))
    finally:
        opm.set_option(opm.OPT_SWEEP_MODE, -1)
    assert torch.equal(out[0][0], out[2][0])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
