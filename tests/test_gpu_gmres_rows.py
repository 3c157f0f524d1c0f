"""GMRes orthogonalisation kernels at the edges of their sizes: the number of
basis rows on both sides of each kernel variant (4, 8, 16, 32 rows), and a
system large enough that a thread takes several elements and a sum has more
partials than are asked for ahead.  Reference: the oracle's GMRes stopped at
the same iteration (modified Gram-Schmidt, 64 bits), the iterates equal to 1e-9
of the largest entry per variable: both are the minimum over the same Krylov
space, up to the rounding of at most 32 orthogonalised vectors.
"""
import numpy as np
import pytest
import torch

import oracle
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


@pytest.fixture(scope="module")
def systems():
    made = {}

    def get(dims):
        if dims not in made:
            case = cases.box_case(*dims, seed=8)
            m = oracle.Model(case)
            m.set_ilu_blocks(4, 4, dims[2])
            st, R, J = m.assemble(cases.random_state(case, seed=1),
                                  m.accumulation(cases.random_state(case, seed=2)), 30 * DAY)
            st, F = m.ilu0(J)
            assert st == 0
            made[dims] = case, m, R, J, F
        return made[dims]
    return get


@pytest.mark.parametrize("dims,its", [((25, 20, 6), k) for k in (1, 4, 5, 8, 9, 16, 17, 32)]
                         + [((62, 60, 13), 9), ((62, 60, 13), 20)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_gmres_rows(opm, systems, dims, its):
    case, m, R, J, F = systems(dims)
    st, xo, its_o, rr = m.gmres(J, F, -R, rtol=1e-14, maxit=its, restart=its)
    assert st == oracle.ENOTCONV and its_o == its
    g = opm.GpuModel(case, ilu_blocks=(4, 4, dims[2]), amg=False)
    Jg = torch.from_numpy(J).to(g.dev)
    ilu, _ = g.ilu0_factor(Jg)
    x, rep = g.gmres(Jg, ilu, g.state(-R), rtol=1e-14, maxit=its, restart=its)
    assert rep.status == opm.ENOTCONV and rep.its == its
    err = np.abs(x.cpu().numpy() - xo) / np.abs(xo).max(axis=0)[None, :]
    assert err.max() <= 1e-9
    assert abs(rep.rel_res - rr) <= 1e-9 * rr
