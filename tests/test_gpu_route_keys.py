"""The routing histogram's scan takes as few (expert, bit-width) keys per lane
of one wave as hold them: numbers of keys at and beside the multiples of 64,
the smallest and the largest, with the selections made in the histogram
workgroup and before it.  Counts, offsets and positions must be exactly those
that the call's own selections give."""
import numpy as np
import pytest
import torch

from layer_cases import DEV
from paper_2504_15299_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [3, 64, 300])
@pytest.mark.parametrize("E,b_min,b_max", [(1, 8, 8), (8, 2, 8), (21, 2, 4), (64, 4, 4), (13, 1, 5),
                                           (16, 1, 8), (43, 6, 8), (64, 2, 8), (64, 1, 8)])
def test_counts_offsets_and_positions(T, E, b_min, b_max):
    d, k, L = 64, min(E, 3), b_max - b_min + 1
    g = torch.Generator(device=DEV).manual_seed(T * 1000 + E * 10 + L)
    x = torch.randn((T, d), generator=g, device=DEV)
    Wg = torch.randn((E, d), generator=g, device=DEV)
    table = torch.randint(b_min, b_max + 1, (T, E), generator=g, device=DEV).to(torch.uint8)
    req = torch.arange(T, dtype=torch.int32, device=DEV)
    r = api.route(x, Wg, None, k, req, table, b_min, b_max)
    torch.cuda.synchronize()
    idx, bits = r.topk_idx.cpu().numpy().reshape(-1), r.topk_bits.cpu().numpy().reshape(-1)
    key = idx.astype(np.int64) * L + bits - b_min
    count = np.bincount(key, minlength=E * L)
    assert np.array_equal(r.hist.cpu().numpy().reshape(-1), count)
    assert np.array_equal(r.offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(count)]))
    perm = r.perm.cpu().numpy()
    assert np.array_equal(perm, np.argsort(key, kind="stable"))
    slot_of = r.slot_of.cpu().numpy().reshape(-1)
    assert np.array_equal(slot_of[perm], np.arange(T * k))
