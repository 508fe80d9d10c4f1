"""The register GEMM cuts an expert's positions into blocks of at most 16 per
bit-width and chunks of at most 8 blocks; large buckets take the tile GEMM.  One-expert layers with chosen
numbers of positions per width put runs at the edges of a block and of a
chunk, in every nest start, with a reduction dimension that ends in half a
128-column step and row tiles that are partly past the matrix edge, against
the oracle (bf16 operands, fp32 sums: per-row max-abs-rel 2e-2)."""
import numpy as np
import pytest
import torch

from layer_cases import FWD_TOL, Layer, row_max_abs_rel
from oracle import oracle as O
from paper_2504_15299_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (b_min, b_max, group, d, f, positions per width)
CASES = {
    "one": (2, 8, 64, 192, 64, {2: 1}),
    "edges_15_17": (2, 8, 64, 320, 192, {2: 15, 8: 17}),
    "full_blocks": (2, 8, 64, 192, 64, {2: 16, 3: 16, 4: 16, 8: 16}),
    "every_width": (1, 8, 64, 192, 64, {b: 1 for b in range(1, 9)}),
    "nine_blocks": (5, 8, 64, 320, 64, {5: 33, 6: 17, 7: 16, 8: 33}),
    "chunk_edge_128": (2, 8, 128, 256, 128, {4: 128}),
    "chunk_edge_129": (2, 4, 128, 384, 256, {2: 113, 4: 16}),
    "ks2_long_reduction": (2, 8, 64, 128, 1088, {2: 20, 8: 3}),
    "two_chunks_mixed": (3, 8, 128, 256, 128, {3: 100, 5: 1, 8: 150}),
    "long_run": (8, 8, 64, 64, 64, {8: 257}),
    "one_width_200": (2, 8, 64, 320, 64, {4: 200}),
    # 384 positions per expert and more take the LDS-tile GEMM (chunks of 256
    # positions of one width)
    "tile_two_widths": (5, 8, 128, 256, 128, {5: 420, 8: 1}),
    # every width on it, for each way of grouping the planes, from b_min 2 and not
    "tile_widths_from_1": (1, 8, 64, 320, 64, {b: 47 + b for b in range(1, 9)}),
    "tile_widths_from_2": (2, 8, 128, 256, 128, {b: 53 + b for b in range(2, 9)}),
}


@pytest.mark.parametrize("name", list(CASES))
def test_blocks_and_chunks(name):
    b_min, b_max, group, d, f, counts = CASES[name]
    T = sum(counts.values())
    spec = wl.scaled(wl.tiny(seed=21), d=d, f=f, E=1, k=1, T=T, group=group, x_dtype="bf16",
                     b_min=b_min, b_max=b_max, n_requests=T, bits_choices=(b_min, b_max))
    L = Layer(spec)
    widths = np.repeat(np.array(list(counts), np.uint8), list(counts.values()))
    np.random.default_rng(3).shuffle(widths)
    L.table = widths[:, None].copy()
    L.ref_route = O.route_from_logits(L.ref_logits, 1, L.req, L.table, b_min, b_max)
    L.pack()
    r = L.route()
    got = L.forward()
    hist = r.hist.cpu().numpy()[0]
    assert {b_min + i: int(n) for i, n in enumerate(hist) if n} == counts
    rel = row_max_abs_rel(got, L.reference())
    assert np.isfinite(got).all() and rel.max() <= FWD_TOL, rel.max()
    # a second call on the same buffers gives the same bits
    again = L.forward()
    assert np.array_equal(got, again)
    torch.cuda.synchronize()
