"""CPR cycle on a system whose first level takes four sets of rows per
wavefront (200,000 rows and more), with two coarse levels of their own and the
rest as one dense operator: 211,200, 26,880, 3,360 | 448, 64 unknowns.  And a
hierarchy of exactly two levels.  Reference: the oracle's cycle; the bound is
that of the smaller systems' tests (1e-8 of the largest entry: sums of at most a
few hundred terms per value, rounded in a different order)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1910_06059_amd import cases
from paper_1910_06059_amd.cases import DAY

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,levels", [((64, 60, 55), 5), ((9, 5, 3), 2)],
                         ids=["five_levels", "two_levels"])
def test_cpr_cycle(dims, levels):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1910_06059_amd import opm
    opm.init()
    c = cases.box_case(*dims, seed=3, wells=[])
    m = oracle.Model(c)
    m.set_ilu_blocks(4, 4, dims[2])
    st, R, J = m.assemble(cases.random_state(c, seed=4),
                          m.accumulation(cases.random_state(c, seed=5)), 2 * DAY)
    st, F = m.ilu0(J)
    assert st == 0
    cp = m.cpr(J)
    g = opm.GpuModel(c, ilu_blocks=(4, 4, dims[2]))
    assert g.amg.n_levels == cp.nl == levels
    Jd = torch.from_numpy(J).to(g.dev)
    cpr, status = g.cpr_setup(Jd)
    assert int(status.item()) == 0
    b = np.random.default_rng(6).standard_normal(m.n) * np.abs(R[:, 0]).max()
    x_o = cp.vcycle(b)
    x_g = g.cpr_vcycle(cpr, torch.from_numpy(b).to(g.dev)).cpu().numpy()
    assert np.abs(x_g - x_o).max() <= 1e-8 * np.abs(x_o).max()
    ilu, st = g.ilu0_factor(Jd)
    z_o = cp.apply(F, R)
    z_g = g.cpr_apply(Jd, ilu, cpr, torch.from_numpy(R).to(g.dev)).cpu().numpy()
    assert (np.abs(z_g - z_o) / (np.abs(z_o).max(axis=0) + 1e-300)).max() <= 1e-8
