"""Convolution kernels of the learned guess at the edges of their tiles.

The kernels stage tiles of 16 x 4 x 4 cells and loop over them with a fixed
number of workgroups (768, weight gradients 512), so the shapes are one exact
tile, one cell more and less on each side, and a box of 867 tiles, where
workgroups take a second one.  Reference: oracle/convnet.py in 64 bits.

Operands are BF16 and products exact in FP32, so an output before rounding
differs by at most n 2^-24 S (S the sum of |terms|; n = 432 + 1 terms of a
forward or transposed product, 2.6e-5 S, the sums in any order); storing BF16
adds 2^-9 relative on each side.  A weight gradient adds one term per cell: in
a chain of matrix products within a tile and over a workgroup's tiles, then
over at most 512 partial sums, less than 1100 roundings in all: 6.6e-5 S.
Bounds: 1e-4 S (products) and 2e-4 S (weight gradients) plus 2^-8 relative for
BF16 results.
"""
import numpy as np
import pytest
import torch

import oracle.convnet as cn
from paper_1910_06059_amd import cases

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4, 16), (5, 5, 17), (3, 3, 15), (1, 9, 31), (9, 65, 257)]   # nz, ny, nx


@pytest.fixture(scope="module")
def opm():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1910_06059_amd import opm as _opm
    _opm.init()
    return _opm


def _to_dev(x):
    cells = int(np.prod(x.shape[:3]))
    b = np.zeros(((cells + 15) // 16 * 16, cn.CH), dtype=np.uint16)
    b[:cells] = cn.to_bf16_bits(x.reshape(-1, cn.CH))
    return torch.from_numpy(b.view(np.int16)).cuda()


def _to_box(t, shape, bf16=True):
    a = t.cpu().numpy()[:int(np.prod(shape))]
    v = cn.from_bf16_bits(a.view(np.uint16)) if bf16 else a.astype(np.float64)
    return v.reshape(*shape, cn.CH).astype(np.float64)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_tiles(opm, shape):
    p = cases.guess_init_params(5, last_scale=1.0)
    net = opm.GuessNet(p)
    W, b = cn.split(p)[1]
    Wr = cn.bf16(W)
    x = np.maximum(cases.guess_random_feats(shape, seed=31, channels=16), 0.0)
    d = cn.bf16(cases.guess_random_feats(shape, seed=32, channels=16) * np.float32(1e-3))
    x64, d64 = x.astype(np.float64), d.astype(np.float64)
    z, S = cn.conv(x64, Wr, b), cn.conv_abs(x64, Wr, b)
    for relu in (True, False):
        got = _to_box(opm.guess_conv(shape, _to_dev(x), net.w_fwd(1), net.bias(1), relu), shape, relu)
        ref = np.maximum(z, 0.0) if relu else z
        assert np.all(np.abs(got - ref) <= 1e-4 * S + (2.0 ** -8 * np.abs(ref) if relu else 0.0))
    grad, din = opm.guess_conv_backward(shape, _to_dev(x), _to_dev(d), net.w_bwd(1), _to_dev(x))
    ref = np.concatenate([v.ravel() for v in cn.conv_weight_grad(x64, d64)])
    S = np.concatenate([v.ravel() for v in cn.conv_weight_grad(np.abs(x64), np.abs(d64))])
    assert np.all(np.abs(grad.cpu().numpy() - ref) <= 2e-4 * S + 1e-30)
    ref = np.where(x64 > 0, cn.conv_transpose(d64, Wr), 0.0)
    S = cn.conv_transpose(np.abs(d64), np.abs(Wr))
    assert np.all(np.abs(_to_box(din, shape) - ref) <= 1e-4 * S + 2.0 ** -8 * np.abs(ref) + 1e-30)
