"""The combine takes four columns per thread and eight rows of a token at a
time: numbers of selected experts at and past that count, widths that end
inside a workgroup, an output that is aligned to its elements only, with and
without the shared expert's partial sums, against the oracle (bf16 operands,
fp32 sums: per-row max-abs-rel 2e-2)."""
import pytest
import torch

from layer_cases import DEV, FWD_TOL, Layer, row_max_abs_rel
from paper_2504_15299_amd import api, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,d,dtype,shared_f", [(1, 64, "bf16", 0), (8, 576, "f32", 0),
                                                (9, 576, "bf16", 64), (17, 320, "f32", 1088)])
def test_rows_widths_and_alignment(k, d, dtype, shared_f):
    T, E = 5, 18
    spec = wl.scaled(wl.tiny(seed=33), d=d, f=64, E=E, k=k, T=T, group=64, x_dtype=dtype,
                     shared_f=shared_f)
    L = Layer(spec).pack()
    L.route()
    want = L.reference()
    buf = torch.full((T * d + 2,), 7.0, dtype=L.xt.dtype, device=DEV)
    out = buf[1:-1].view(T, d)
    api.moe_forward(L.xt, L.w13, L.w2, L.r, k, shared=L.shared, out=out)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    assert float(buf[0]) == 7.0 and float(buf[-1]) == 7.0
    assert row_max_abs_rel(got, want).max() <= FWD_TOL
    # the aligned output of another call holds the same values
    assert (L.forward() == got).all()
