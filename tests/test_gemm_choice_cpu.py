"""Which kernels a layer takes, read off the launches without a GPU."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def _kernels(fake, c):
    return [op for _, op, _, _ in fake_hip.calls(fake, [c]) if op.startswith("launch:")]


def _streamed(counts, bits, f, d=256):
    """Counts of positions per expert, all at `bits`, one expert per token."""
    E = len(counts)
    hist = [[n if b == bits else 0 for b in range(2, 9)] for n in counts]
    return dict(kind="streamed", T=sum(counts), d=d, f=f, E=E, k=1, b_min=2, b_max=8, group=128,
                hist=hist, units=[(e, bits, 0, bits) for e in range(E) if counts[e]], pinned=1 << 39)


@pytest.mark.parametrize("counts,bits,f,want", [
    # large and small experts in one layer: one GEMM for all of them (the two
    # in a row, each with its own tail, are slower than either)
    ((200, 200, 30, 30), 4, 512, "bgemm"),
    ((250, 250, 250, 30), 8, 14336, "tile_gemm"),
    # few workgroups: the register GEMM's shorter ones; many: the tile GEMM's
    # fewer ones
    ((250, 250, 250, 250), 8, 512, "bgemm"),
    ((250, 250, 250, 250), 8, 14336, "tile_gemm"),
    # from 384 positions per expert on average
    ((700, 70), 2, 512, "tile_gemm"),
    # at most 128 positions per expert
    ((128, 128, 100, 1), 8, 14336, "bgemm"),
])
def test_a_layer_takes_one_gemm(fake, counts, bits, f, want):
    gemms = [op for op in _kernels(fake, _streamed(counts, bits, f)) if "gemm_kernel" in op]
    assert len(gemms) == 2 * sum(n > 0 for n in counts)
    other = "tile_gemm" if want == "bgemm" else "bgemm"
    assert all(want in op for op in gemms) and not any(other in op for op in gemms), gemms
