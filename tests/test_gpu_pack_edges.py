"""Edges of the register-resident MWQ pack: weights that start at a 4-byte
aligned address, row and group counts that do not fill a workgroup (64 rows,
4 groups), and groups that hold infinities or NaN (whose residual signs are
taken by comparison)."""
import numpy as np
import pytest
import torch

from layer_cases import DEV
from oracle import oracle as O
from paper_2504_15299_amd import api

pytestmark = pytest.mark.gpu


def _pack(W, group, b_min=2, b_max=8):
    m = api.MWQ.empty(W.shape[0], W.shape[1], W.shape[2], group, b_min, b_max, device=DEV)
    api.pack_mwq(W, m)
    torch.cuda.synchronize()
    return m


@pytest.mark.parametrize("group,rows,cols", [(128, 16, 128), (128, 80, 640), (64, 32, 64),
                                             (64, 96, 576)])
def test_unaligned_weights_and_ragged_tiles(group, rows, cols):
    rng = np.random.default_rng(rows + cols)
    W = (rng.standard_normal((rows, cols)) * 0.02).astype(np.float32)
    buf = torch.zeros(rows * cols + 1, dtype=torch.float32, device=DEV)
    buf[1:] = torch.from_numpy(W).to(DEV).reshape(-1)
    view = buf[1:].view(1, rows, cols)
    assert view.is_contiguous() and view.data_ptr() % 16 == 4
    m = _pack(view, group)
    rp, rs, rz = O.mwq_pack(O.mwq_quantize(W, group, 2, 8))
    assert np.array_equal(m.planes.cpu().numpy().view(np.uint32), rp)
    assert np.array_equal(m.scales.cpu().numpy().view(np.uint16), rs)
    assert np.array_equal(m.zeros.cpu().numpy(), rz)


@pytest.mark.parametrize("group", [64, 128])
def test_non_finite_weights(group):
    """A NaN takes base code 0, and its sign is never 'v >= 0'; the other
    groups of the matrix are not touched by it.  An infinite weight makes the
    range infinite (base scale 1), so its residual is infinite at the first
    level and NaN (bit clear) from then on, like every other residual of its
    group."""
    rows, cols = 2048 // group, 2 * group
    W = (np.random.default_rng(5).standard_normal((rows, cols)) * 0.02).astype(np.float32)
    clean = _pack(torch.from_numpy(W[None]).to(DEV), group)
    W[1, 3] = np.nan
    W[2, 5] = np.inf
    m = _pack(torch.from_numpy(W[None]).to(DEV), group)
    # signs [levels][row][col] and base codes
    q1, signs = api.debug_unpack(m, 0, 8)
    c1, csigns = api.debug_unpack(clean, 0, 8)
    torch.cuda.synchronize()
    q1, signs, c1, csigns = (t.cpu().numpy() for t in (q1, signs, c1, csigns))
    assert q1[1, 3] == 0 and q1[2, 5] == 3
    assert (signs[:, 1, 3] == -1).all()
    assert (signs[1:, 1, :group] == -1).all()       # the first scale is NaN
    assert signs[0, 2, 5] == 1 and (signs[2:, 2, :group] == -1).all()
    keep = np.ones((rows, cols), bool)
    keep[1:3, :group] = False
    assert np.array_equal(q1[keep], c1[keep])
    assert np.array_equal(signs[:, keep], csigns[:, keep])
