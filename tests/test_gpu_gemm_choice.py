"""The layer takes the register GEMM or the LDS-tile GEMM for all of its
routed experts, chosen on the device from the routing's counts (on the host
for the streamed forward, whose sums are the same bit for bit only if it
chooses the same); the shared expert takes the tile GEMM from 768 tokens on.
Layers of either choice with several experts, uneven loads, one to three
widths and less than 384 positions per expert, against the oracle and the
streamed forward.  Which GEMM a case means to reach is checked first, on a
stand-in for the runtime, from the same counts."""
import numpy as np
import pytest
import torch

import fake_hip
from layer_cases import DEV, FWD_TOL, Layer, ambiguous_tokens, logit_error_bound, row_max_abs_rel
from oracle import oracle as O
from paper_2504_15299_amd import api
from paper_2504_15299_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def _spec(**kw):
    c = dict(d=2048, f=768, E=16, k=2, T=1200, group=64, x_dtype="bf16", n_requests=1, shared_f=0)
    c.update(kw)
    return wl.scaled(wl.tiny(seed=41), **c)


def _gemms(fake, s, **kw):
    call = dict(T=s.T, d=s.d, f=s.f, E=s.E, k=s.k, b_min=s.b_min, b_max=s.b_max, group=s.group)
    call.update(kw)
    return [(op, stream) for _, op, stream, _ in fake_hip.calls(fake, [call])
            if "gemm_kernel" in op]


def _check(L, got):
    """Every 17th token that is not ambiguous against the oracle."""
    amb = ambiguous_tokens(L.ref_logits, L.spec.k, logit_error_bound(L.x, L.Wg, L.bias))
    tokens = [t for t in range(0, L.spec.T, 17) if not amb[t]]
    ref = L.reference(tokens=tokens)
    err = row_max_abs_rel(got[tokens], ref)
    assert np.isfinite(got).all() and err.max() <= FWD_TOL, err.max()


def _pinned(m):
    return api.MWQ(m.n_experts, m.rows, m.cols, m.group, m.b_min, m.b_max,
                   *[torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t)
                     for t in (m.planes, m.scales, m.zeros)])


# name: (spec, widths of the experts, the GEMM that the layer takes)
CASES = {
    "tile_8_bits": (dict(), [8] * 16, "tile_gemm"),
    "tile_zipf": (dict(T=1400, zipf_s=1.1), [8, 8, 4, 4, 8, 2, 2, 3] * 2, "tile_gemm"),
    "tile_two_widths": (dict(T=2400, n_requests=2), [[8] * 16, [4] * 16], "tile_gemm"),
    "tile_group_128": (dict(group=128), [8, 7, 6, 5] * 4, "tile_gemm"),
    # the same loads in a layer of few workgroups, and loads of which some
    # experts alone would take the tile GEMM
    "register_small_layer": (dict(f=128, d=192), [8] * 16, "bgemm"),
    "register_zipf": (dict(T=700, zipf_s=1.1, d=192, f=320), [2, 3, 4, 8] * 4, "bgemm"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_resident_and_streamed_take_the_same_gemm(fake, name):
    kw, widths, want = CASES[name]
    L = Layer(_spec(**kw))
    s = L.spec
    L.table = np.array(widths, np.uint8).reshape(s.n_requests, s.E)
    L.ref_route = O.route_from_logits(L.ref_logits, s.k, L.req, L.table, s.b_min, s.b_max)
    L.pack()
    r = L.route()
    hist = r.hist.cpu().numpy()
    assert s.T * s.k < 384 * s.E and hist.sum(1).min() < hist.sum(1).max()
    units = api.hebf_order(hist, s.b_min, s.b_max)
    gemms = _gemms(fake, s, kind="streamed", hist=hist.tolist(), pinned=1 << 39,
                   units=[u[:4] for u in units])
    assert len(gemms) == 2 * len(units) and all(want in op for op, _ in gemms), (name, hist)
    got = L.forward()
    _check(L, got)
    d13, d2 = (api.MWQ.empty(m.n_experts, m.rows, m.cols, m.group, m.b_min, m.b_max, device=DEV)
               for m in (L.w13, L.w2))
    resident = np.zeros(s.E, np.uint8)
    st = api.moe_forward_streamed(L.xt, _pinned(L.w13), _pinned(L.w2), d13, d2, resident, r, s.k,
                                  hist, units, [torch.cuda.Event() for _ in units],
                                  torch.cuda.Stream())
    torch.cuda.synchronize()
    assert np.array_equal(st.float().cpu().numpy(), got)
    assert np.array_equal(L.forward(), got)


@pytest.mark.parametrize("T,shared_f,dtype", [(768, 320, "f32"), (800, 1088, "bf16")])
def test_shared_expert_on_tiles(fake, T, shared_f, dtype):
    """Chunks that end inside the last one (800 positions in chunks of 64), and
    a W2 reduction in two parts (1088 columns)."""
    L = Layer(_spec(f=64, d=256, k=2, T=T, shared_f=shared_f, x_dtype=dtype)).pack()
    ops = _gemms(fake, L.spec, kind="forward", shared_f=shared_f)
    assert sum(stream != fake_hip.STREAM and "tile_gemm" in op for op, stream in ops) == 2
    L.route()
    got = L.forward()
    _check(L, got)
    assert np.array_equal(L.forward(), got)
