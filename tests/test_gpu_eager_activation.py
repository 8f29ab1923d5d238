"""Activations of the one-launch eager pass: layers without one announce what their sums are, NaN and infinities included, rectified
layers announce zero for NaN; through several layers a net without activations announces the conventional network's values."""
import numpy as np
import pytest

import oracle
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


def announced(wl, seg, levels):
    """The announced values of `levels` after the last row, pushed seg rows at a time; one launch per push."""
    import torch
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, wl["streams"], max_seg_rows=seg)
    st.enable_eager()
    x = input_tensor(wl)
    st.profile_begin()
    for r in range(0, wl["in_h"], seg):
        st.push_segment(x[:, r:r + seg].contiguous())
    assert [(p["name"], p["launches"]) for p in st.profile_end()] == [("eager@0", -(-wl["in_h"] // seg))]
    shapes = oracle.layer_shapes(wl["layers"], wl["in_h"], wl["in_w"])
    out = {lv: st.read_announced(lv, shapes[lv - 1]) for lv in levels}
    torch.cuda.synchronize()
    st.close(); net.destroy()
    return {lv: v.cpu().numpy() for lv, v in out.items()}


@pytest.mark.parametrize("act", ["none", "relu"])
@pytest.mark.parametrize("c_in,c_out,pool,seg", [(3, 16, False, 1), (16, 32, False, 2), (32, 64, True, 1), (32, 64, True, 3)])
def test_sums_that_are_not_finite(act, c_in, c_out, pool, seg):
    rng = np.random.default_rng(c_in + seg)
    x = rng.normal(size=(2, 6, 20, c_in)).astype(np.float32)
    x[0, 2, 3, 1], x[0, 3, 12, 0], x[1, 4, 6, 2] = np.nan, np.inf, -np.inf
    w = rng.normal(0, 0.2, size=(c_out, c_in, 3, 3)).astype(np.float32)
    layers = [conv(c_in, c_out, 3, 3, p_h=1, p_w=1, act=act)] + ([maxpool(c_out)] if pool else [])
    wl = dict(name="nan", precision="f32", in_h=6, in_w=20, in_c=c_in, layers=layers, weights=[w] + [None] * pool, biases=[None] * len(layers),
              x=x, seg_rows=seg, streams=2)
    got = announced(wl, seg, [len(layers)])[len(layers)]
    xp = np.pad(x.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0)))
    with np.errstate(invalid="ignore"):
        c = sum(np.einsum("byxc,oc->byxo", xp[:, ky:ky + 6, kx:kx + 20], w[:, :, ky, kx].astype(np.float64)) for ky in range(3) for kx in range(3))
    want = c if act == "none" else np.where(c > 0, c, 0.0)            # (NaN > 0 is false)
    if pool:
        # a NaN may win or lose against its neighbours in a window: windows without one are compared
        win = want.reshape(2, 3, 2, 10, 2, c_out)
        known = ~np.isnan(win).any(axis=(2, 4))
        want = np.where(known, np.nan_to_num(win, nan=-1.0, posinf=np.inf, neginf=-np.inf).max(axis=(2, 4)), 0.0)
        got = np.where(known, got, 0.0)
    assert np.isnan(c).any() and np.isinf(c).any()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    ok = np.isfinite(want)
    assert np.array_equal(np.sign(got[~ok & ~np.isnan(want)]), np.sign(want[~ok & ~np.isnan(want)]))
    assert np.max(np.abs(got[ok] - want[ok])) <= 1e-4 * np.max(np.abs(want[ok]))


@pytest.mark.parametrize("prec", ["f32", "i8"])
@pytest.mark.parametrize("seg", [1, 2])
def test_layers_without_activation(prec, seg):
    """float32: every layer, below a pool too; int8 (which clamps what it passes on): the last one, whose values are of both signs."""
    rng = np.random.default_rng(seg)
    h, w, streams, chans = 12, 19, 2, (3, 16, 32, 16)
    inner = dict(act="none") if prec == "f32" else dict(act="relu_shr_clamp", shr=5, clamp_hi=15)
    layers = [conv(chans[i], chans[i + 1], 3, 3, p_h=1, p_w=1, **(inner if i < 2 else dict(act="none"))) for i in range(3)]
    layers.insert(1, maxpool(16))
    if prec == "i8":
        ws = [None if L["kind"] != "conv" else rng.integers(-8, 8, size=(L["c_out"], L["c_in"], 3, 3)).astype(np.int8) for L in layers]
        x = rng.integers(-9, 16, size=(streams, h, w, 3)).astype(np.int8)
    else:
        ws = [None if L["kind"] != "conv" else rng.normal(0, (1 / (9 * L["c_in"])) ** 0.5, size=(L["c_out"], L["c_in"], 3, 3)).astype(np.float32) for L in layers]
        x = rng.normal(size=(streams, h, w, 3)).astype(np.float32)
    wl = dict(name="none", precision=prec, in_h=h, in_w=w, in_c=3, layers=layers, weights=ws, biases=[None] * 4, x=x, seg_rows=seg, streams=streams)
    got = announced(wl, seg, [4])[4]
    for b in range(streams):
        want = oracle.dense(layers, x[b], ws, [None] * 4, integer=prec == "i8")
        assert (want < 0).any() and (want > 0).any()
        if prec == "i8":
            assert np.array_equal(got[b].astype(np.int64), want)
        else:                                     # 32-bit sums of at most 288 products against 64-bit ones, through three layers
            assert np.max(np.abs(got[b] - want)) <= 1e-5 * np.max(np.abs(want))
