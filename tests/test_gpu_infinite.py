"""An infinite value is an event like any other: it reaches the outputs whose window holds it, and no other one.  Kernels that
pad a window with zero weights must not pad it with values that can be infinite."""
import numpy as np
import pytest

import oracle
from workloads import conv, round_to_bf16
from helpers import gpu_run, rel_err, TOL

pytestmark = pytest.mark.gpu


def one_layer(prec, H, W, c_in, c_out, streams, seg):
    rng = np.random.default_rng(c_in * 1000 + W)
    rnd = round_to_bf16 if prec == "bf16" else (lambda a: a.astype(np.float32))
    w = rng.normal(0, 0.2, size=(c_out, c_in, 3, 3))
    w = rnd(np.where(w < 0, w - 0.01, w + 0.01).astype(np.float32))          # (no weight is zero)
    x = rnd(rng.random((streams, H, W, c_in), dtype=np.float32))
    x[rng.random(x.shape) < 0.3] = 0
    return dict(name="one", precision=prec, in_h=H, in_w=W, in_c=c_in, layers=[conv(c_in, c_out, 3, 3, p_h=1, p_w=1, act="none")],
                weights=[w], biases=[None], x=x, seg_rows=seg, streams=streams)


def places(wl):
    """Per stream: row, column and channel of its infinite value; the columns where tiles meet come first."""
    rng = np.random.default_rng(3)
    W, C = wl["in_w"], wl["in_c"]
    xs = [x for x in (0, W - 1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65) if x < W]
    for b in range(wl["streams"]):
        yield int(rng.integers(wl["in_h"])), xs[b % len(xs)] if b < 2 * len(xs) else int(rng.integers(W)), int(C - 1 - b % min(C, 8))


def check(wl, out):
    at = list(places(wl))
    for b in range(wl["streams"]):
        y, x, c = at[b]
        finite = wl["x"][b].copy()
        finite[y, x, c] = 0
        want = oracle.dense(wl["layers"], finite, wl["weights"], wl["biases"])
        reached = np.zeros(want.shape, bool)
        for ky in range(3):
            for kx in range(3):
                o, p = y + 1 - ky, x + 1 - kx
                if 0 <= o < wl["in_h"] and 0 <= p < wl["in_w"]:
                    want[o, p] = np.copysign(np.inf, wl["weights"][0][:, c, ky, kx])
                    reached[o, p] = True
        assert np.array_equal(out[b][reached].astype(np.float64), want[reached]), f"stream {b}: infinite at {at[b]}"
        assert np.isfinite(out[b][~reached]).all(), f"stream {b}: infinite at {at[b]}"
        assert rel_err(out[b][~reached], want[~reached]) <= TOL["f32"], f"stream {b}"


@pytest.mark.parametrize("prec,c_in,c_out,W,streams,seg", [
    ("f32", 1, 16, 35, 24, 1), ("f32", 3, 32, 50, 24, 1), ("f32", 4, 32, 66, 24, 2), ("f32", 8, 32, 50, 24, 1),
    ("f32", 12, 64, 33, 24, 3), ("f32", 20, 16, 70, 24, 1), ("f32", 16, 32, 35, 24, 1), ("f32", 100, 16, 40, 24, 2),
    ("bf16", 2, 16, 35, 24, 1), ("bf16", 3, 64, 66, 64, 8), ("bf16", 8, 32, 50, 24, 1), ("bf16", 16, 64, 66, 64, 8),
    ("bf16", 24, 64, 70, 64, 8), ("bf16", 40, 32, 130, 64, 8), ("bf16", 16, 16, 20, 24, 1), ("bf16", 32, 64, 66, 64, 8)])
def test_only_windows_that_hold_it_are_reached(prec, c_in, c_out, W, streams, seg):
    wl = one_layer(prec, 8, W, c_in, c_out, streams, seg)
    for b, (y, x, c) in enumerate(places(wl)):
        wl["x"][b, y, x, c] = np.inf
    out, st, net = gpu_run(wl, return_streams=True)
    assert st.layer_kernels() == ["conv3x3_mfma"]
    st.close(); net.destroy()
    check(wl, out)


@pytest.mark.parametrize("c_in,c_out,W,seg", [(1, 16, 35, 1), (2, 32, 50, 2), (3, 32, 66, 1), (4, 48, 33, 3), (8, 32, 50, 1), (12, 64, 34, 4), (20, 16, 70, 2), (16, 32, 35, 1)])
def test_only_windows_that_hold_it_are_reached_in_eager_emission(c_in, c_out, W, seg):
    import torch
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    wl = one_layer("f32", 8, W, c_in, c_out, 24, seg)
    for b, (y, x, c) in enumerate(places(wl)):
        wl["x"][b, y, x, c] = np.inf
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, wl["streams"], max_seg_rows=seg)
    st.enable_eager()
    x = input_tensor(wl)
    st.profile_begin()
    for r in range(0, 8, seg):
        st.push_segment(x[:, r:r + seg].contiguous())
    prof = st.profile_end()
    out = st.read_announced(1, (8, W, c_out))
    torch.cuda.synchronize()
    assert [(p["name"], p["launches"]) for p in prof] == [("eager@0", -(-8 // seg))]      # a launch per push
    check(wl, out.cpu().numpy())
    st.close(); net.destroy()
