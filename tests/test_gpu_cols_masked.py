"""The column kernels on masked lattices, where a column has holes and records of
inactive cells are neither written (whole groups of slots) nor read: bitwise the
results of one launch per level.  Single cells out at random, blobs, whole
columns and whole tiles out; boxes of one and four wavefronts, one box, tiles."""
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


def _cells(dims, share):
    return np.random.default_rng(4).random(dims[::-1]) < share


def _blobs(dims, share):
    from scipy import ndimage
    f = ndimage.uniform_filter(np.random.default_rng(5).standard_normal(dims[::-1]), size=(3, 5, 5))
    return f >= np.quantile(f, 1 - share)


def _outline(dims, share):
    m = np.zeros(dims[::-1], bool)
    m[:, : max(1, round(share * dims[1])), 1:dims[0] - 2] = True
    return m


SHAPES = {
    "one_wave_cells": ((13, 10, 11), (4, 4, 11), _cells, 0.5),
    "one_wave_outline": ((20, 20, 9), (4, 4, 9), _outline, 0.4),
    "four_waves_blobs": ((19, 17, 20), (8, 8, 20), _blobs, 0.6),
    "four_waves_cells": ((19, 17, 40), (8, 8, 40), _cells, 0.9),
    "by_position": ((19, 17, 20), (8, 8, 20), _cells, 0.1),
    "short_boxes": ((20, 20, 3), (8, 8, 3), _cells, 1.1),
    "one_box": ((10, 9, 12), None, _cells, 0.3),
    "tiles_cells": ((26, 19, 12), None, _cells, 0.4),
    "tiles_outline": ((40, 33, 7), None, _outline, 0.3),
    "tiles_one_cell": ((20, 20, 5), None, _cells, 0.002),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(SHAPES))
def test_masked_columns_bitwise_equal(opm, name, precision):
    dims, blk, make, share = SHAPES[name]
    mask = make(dims, share)
    case = cases.box_case(*dims, seed=3, wells=[], mask=mask)
    print(f"masked columns: {name} {int(mask.sum())} cells, precision {precision}", flush=True)
    g = opm.GpuModel(case, ilu_blocks=blk, amg=False)
    y = g.state(cases.random_state(case, 5))
    R, J, _ = g.assemble(y, g.accumulation(g.state(cases.random_state(case, 6))), DAY)
    out = []
    try:
        for mode, before in ((-1, 0xff), (1, 0)):
            opm.set_option(opm.OPT_SWEEP_MODE, mode)
            # (storage that held other values: nothing of it may be read)
            size = opm.lib().opm_ilu0_bytes(g._pbp(), precision)
            ilu = torch.full((size,), before, dtype=torch.uint8, device=g.dev)
            status = torch.zeros(1, dtype=torch.int32, device=g.dev)
            assert opm.lib().opm_ilu0_factor(g._pbp(), opm._ptr(J), opm._ptr(ilu), precision,
                                             opm._ptr(status), opm._stream()) == opm.OK
            assert int(status.item()) == 0
            x, rep = g.bicgstab(J, ilu, -R, rtol=1e-8, precision=precision)
            assert rep.status == 0
            out.append(([g.ilu0_apply(ilu, r, precision)
                         for r in (R, torch.flip(R, [0]).contiguous(), R)], x))
    finally:
        opm.set_option(opm.OPT_SWEEP_MODE, -1)
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.isfinite(b).all() and torch.equal(a, b), (name, precision)
    # the solutions: each meets ||r|| <= 1e-8 ||R|| on the same operator
    for _, x in out:
        r = -R - g.spmv(J, x)
        assert float(r.norm()) <= 1.01e-8 * float(R.norm())
