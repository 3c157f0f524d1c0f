"""The LDS of an ensemble with several workgroups per member: what is kept beside
the sweep window (cell marks, level bounds) never refuses a shape whose window
fits, and a configuration that has room for the window alone runs."""
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


@pytest.mark.parametrize("threads", [256, 128])
def test_shape_with_many_levels_is_accepted(opm, threads):
    """20,000 levels, one row each: their bounds would take 160 KB, the window
    takes 48 bytes."""
    ens = opm.Ensemble([cases.box_case(2, 1, 20000, seed=3, wells=[])], precision=opm.PREC_FP64,
                       member_split=(2, 1))
    ens.configure(threads, 0, 0, 2)
    assert ens.config.wgs == 2 and 48 <= ens.config.sweep_bytes <= 75 * 1024


@pytest.mark.parametrize("precision", [0, 1])
def test_window_alone(opm, precision):
    """A configuration of an earlier run that holds the size of the window alone:
    the sweeps read their level bounds from memory, with the same results."""
    ms = [cases.config1(), cases.box_case(9, 8, 5, seed=12, name="m1"),
          cases.box_case(6, 5, 3, seed=11, name="m0")]
    out = []
    for alone in (False, True):
        ens = opm.Ensemble(ms, precision=precision, member_split=(2, 2))
        ens.configure(256, 0, 0, 8)
        assert ens.config.wgs > len(ms)
        if alone:
            # (sizes in units of 256 bytes; two level bounds of 4 bytes per level)
            bounds = 8 * max(m.n_levels for m in ens.members)
            window = (ens.config.sweep_bytes - bounds) // 256 * 256
            assert 0 < bounds <= 256 and window == ens.config.sweep_bytes - 256
            ens.config.sweep_bytes = window
        ens.launch(10 * DAY, 2)
        torch.cuda.synchronize()
        reps = ens.read_reports()
        assert all(r["status"] == 0 and r["steps_done"] == 2 for r in reps), reps
        out.append((ens.states(), [r["lin_its"] for r in reps]))
    assert out[0][1] == out[1][1]
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)
