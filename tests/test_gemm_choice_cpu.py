"""Which kernels a layer takes, read off the launches without a GPU."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def _kernels(fake, c):
    return [op for _, op, _, _ in fake_hip.calls(fake, [c]) if op.startswith("launch:")]


def _streamed(counts, bits, f, d):
    """Counts of positions per expert, all at `bits`, one expert per token."""
    E = len(counts)
    hist = [[n if b == bits else 0 for b in range(2, 9)] for n in counts]
    return dict(kind="streamed", T=sum(counts), d=d, f=f, E=E, k=1, b_min=2, b_max=8, group=128,
                hist=hist, units=[(e, bits, 0, bits) for e in range(E) if counts[e]], pinned=1 << 39)


@pytest.mark.parametrize("counts,bits,d,f,want", [
    # large and small experts in one layer: one GEMM for all of them (the two
    # in a row, each with its own tail, are slower than either)
    ((200, 200, 30, 30), 4, 256, 512, "bgemm"),
    ((250, 250, 250, 30), 8, 4096, 14336, "tile_gemm"),
    # few workgroups, of W1/W3 or of W2: the register GEMM's shorter ones; many:
    # the tile GEMM's fewer ones
    ((250, 250, 250, 250), 8, 256, 512, "bgemm"),
    ((250, 250, 250, 250), 8, 256, 14336, "bgemm"),
    ((250, 250, 250, 250), 8, 4096, 14336, "tile_gemm"),
    # wide chunks cost the register GEMM more than narrow ones
    ((250, 250, 250, 250), 2, 4096, 14336, "bgemm"),
    # from 384 positions per expert on average
    ((700, 70), 2, 256, 512, "tile_gemm"),
    # at most 128 positions per expert, and few positions per chunk
    ((128, 128, 100, 1), 8, 4096, 14336, "bgemm"),
    ((129,) + (1,) * 63, 8, 4096, 14336, "bgemm"),
])
def test_a_layer_takes_one_gemm(fake, counts, bits, d, f, want):
    gemms = [op for op in _kernels(fake, _streamed(counts, bits, f, d)) if "gemm_kernel" in op]
    assert len(gemms) == 2 * sum(n > 0 for n in counts)
    other = "tile_gemm" if want == "bgemm" else "bgemm"
    assert all(want in op for op in gemms) and not any(other in op for op in gemms), gemms


@pytest.mark.parametrize("E,k,T,d,f,b_max,pairs", [
    # one column block: 5120 waves
    (8, 2, 16, 4096, 14336, 8, True), (8, 2, 4, 4096, 14336, 8, False),
    # two: 2560 (2816 here and 2304, 1536 below), and not over a multiple of 128 KiB
    (8, 2, 20, 2048, 13824, 8, True), (8, 2, 20, 2048, 8192, 8, False),
    (8, 2, 20, 2048, 8192, 7, True), (4, 2, 16, 3072, 7168, 8, False),
    (8, 2, 32, 1024, 8192, 7, False),
    # three: 1280 up to 4 bits, else 2048 for one expert and 3072 for several
    (1, 1, 16, 5120, 13824, 4, True), (1, 1, 16, 5120, 13824, 8, False),
    (1, 1, 16, 4096, 13824, 4, False), (1, 1, 64, 4096, 8192, 8, True),
    (8, 2, 64, 2048, 8192, 8, True), (8, 2, 64, 1536, 8192, 8, False),
])
def test_decode_w2_takes_row_block_pairs(fake, E, k, T, d, f, b_max, pairs):
    ops = _kernels(fake, dict(kind="forward", T=T, d=d, f=f, E=E, k=k, b_min=2, b_max=b_max,
                              group=128))
    # activation prep, W1/W3, prep, W2, combine
    assert len(ops) == 5 and "decode13_kernel" in ops[1], ops
    assert ("decode13_kernel" if pairs else "13decode_kernel") in ops[3], ops[3]
