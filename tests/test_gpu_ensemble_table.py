"""Sharing out a member's subdomains takes time in proportion to their number."""
import time

import numpy as np
import pytest
import torch

from paper_1910_06059_amd import cases

pytestmark = pytest.mark.gpu


def test_many_uneven_subdomains():
    """2500 columns of 12 to 20 active cells for 256 workgroups: a few
    milliseconds, where a step for every sum of neighbouring columns took seconds."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1910_06059_amd import opm
    mask = np.random.default_rng(7).random((20, 50, 50)) < 0.85
    ens = opm.Ensemble([cases.box_case(50, 50, 20, seed=3, wells=[], mask=mask)],
                       precision=opm.PREC_MIXED, member_split=(50, 50))
    assert ens.members[0].pb.n_sub == 2500
    t = time.perf_counter()
    ens.configure(256, 0, 0, 256)
    t = time.perf_counter() - t
    assert 200 <= ens.config.wgs <= 256
    assert t < 1.0, t
