"""Which systems are factored by lattice columns (no GPU needed): the size of the
factor storage follows the active cells, not the lattice around them, and a
box whose widest level leaves wavefronts without a row goes by position."""
import numpy as np
import pytest

from paper_1910_06059_amd import opm


def _bytes(dims, blk, mask=None, precision=opm.PREC_FP64, lattice=True):
    """opm_ilu0_bytes of a system (host only: it reads none of the device arrays);
    lattice=False: as without the lattice maps and the box, by position."""
    mask = np.ones(dims[::-1], bool) if mask is None else mask
    n, nf, host, topo, b = opm.build_topology(*dims, mask, blk)
    there = host["row_ptr"].ctypes.data
    pb = opm.Problem(n_cells=n, n_faces=nf, nnzb=n + 2 * nf, n_levels=topo.n_levels,
                     max_level=topo.max_level, sweep_span=topo.sweep_span, row_ptr=there,
                     iperm=there, lo_blk=there, up_blk=there)
    if b is not None:
        pb.n_sub, pb.max_sub, pb.max_width = b.n_sub, b.max_sub, b.max_width
    if lattice:
        pb.nx, pb.ny, pb.nz = dims
        pb.box_cell = pb.cell_box = there
        if blk is not None:
            x, y, z = (min(q, m) for q, m in zip(blk, dims))
            pb.ilu_box = x | y << 10 | z << 20
    return opm.lib().opm_ilu0_bytes(pb, precision), n


def _some(dims, share):
    return np.random.default_rng(2).random(dims[::-1]) < share


# (lattice, box, active share, precision): by columns?
RULE = [
    ((24, 25, 15), (2, 2, 15), 1.0, 0, True),
    ((20, 20, 3), (8, 8, 3), 1.0, 0, False),           # 22 rows of 64 on the widest level
    ((30, 30, 30), (8, 8, 30), 0.05, 0, False),        # sparse: the same
    ((64, 64, 48), (4, 4, 48), 0.25, 0, True),         # 49,000 cells, 4.7 slots each
    ((128, 128, 48), (4, 4, 48), 0.25, 0, False),      # 197,000 cells: bound by bytes
    ((128, 128, 48), (4, 4, 48), 0.45, 0, False),
    ((128, 128, 48), (4, 4, 48), 0.45, 1, True),
    ((50, 50, 12), None, 1.0, 0, True),                # 2.7 slots per cell
    ((200, 200, 60), None, 0.01, 0, False),            # 123 slots per cell
]


@pytest.mark.parametrize("dims,blk,share,precision,columns", RULE)
def test_rule_follows_active_cells(dims, blk, share, precision, columns):
    mask = None if share == 1.0 else _some(dims, share)
    got, n = _bytes(dims, blk, mask, precision)
    plain, _ = _bytes(dims, blk, mask, precision, lattice=False)
    # (planes of a whole lattice: a table of two words per plane and diagonal)
    table = 8 * (dims[0] + dims[1]) * dims[2] + 100 * n if blk is None else 0
    assert (got > plain + table) == columns, (got, plain, n)


@pytest.mark.parametrize("share", [1.0, 0.5, 0.2, 0.05, 0.01])
@pytest.mark.parametrize("dims,blk", [((200, 200, 60), None), ((200, 200, 60), (8, 8, 60)),
                                      ((200, 200, 60), (4, 4, 60))])
def test_storage_in_proportion_to_cells(dims, blk, share):
    """Subdomains take at most two slots (604 bytes) per cell beyond 0.64 GB, the
    whole system at most 32."""
    got, n = _bytes(dims, blk, None if share == 1.0 else _some(dims, share))
    assert got <= max(1400 * n if blk else 32 * 640 * n, 640 << 20), (got / n, n)


@pytest.mark.parametrize("box", [
    -1, 0x7fffffff, 1 << 30 | 4 | 4 << 10 | 15 << 20, 4 | 4 << 10, 25 | 4 << 10 | 15 << 20,
    2 | 2 << 10 | 15 << 20, 4 | 4 << 10 | 14 << 20, 5 | 4 << 10 | 15 << 20, 8 | 2 << 10 | 15 << 20,
    0x00cdcdcd])
def test_box_of_another_topology_is_not_taken(box):
    """A box that the counts of the topology contradict (a field that was never
    set): by position, as without a box."""
    dims, blk = (24, 25, 15), (4, 4, 15)
    n, nf, host, topo, b = opm.build_topology(*dims, np.ones(dims[::-1], bool), blk)
    there = host["row_ptr"].ctypes.data
    pb = opm.Problem(n_cells=n, n_faces=nf, nnzb=n + 2 * nf, n_levels=topo.n_levels,
                     max_level=topo.max_level, sweep_span=topo.sweep_span, row_ptr=there,
                     iperm=there, lo_blk=there, up_blk=there, n_sub=b.n_sub, max_sub=b.max_sub,
                     max_width=b.max_width, nx=24, ny=25, nz=15, box_cell=there, cell_box=there)
    size = opm.lib().opm_ilu0_bytes
    plain = size(pb, opm.PREC_FP64)
    pb.ilu_box = 4 | 4 << 10 | 15 << 20
    # (63 doubles, an index and a 32-byte record for each of 42 x 21 x 16 slots)
    assert size(pb, opm.PREC_FP64) >= 42 * 21 * 16 * (63 * 8 + 36)
    pb.ilu_box = box
    assert size(pb, opm.PREC_FP64) == plain
