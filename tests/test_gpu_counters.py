"""Counters of events and multiply-adds where the waves of a workgroup add up before one of them adds for all (a step of five
workgroups per stream and more, few streams) and where each adds by itself: widths and channels that leave waves of a workgroup without
work, pools, narrow and wide tiles.  Whole numbers: exact."""
import numpy as np
import pytest

from helpers import check_stream, gpu_run, oracle_stream
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels", [16, 48, 128])
@pytest.mark.parametrize("W", [4, 17, 62, 130])
@pytest.mark.parametrize("streams,seg", [(1, 1), (23, 1), (23, 8), (24, 1)])
def test_counters_by_workgroup_and_by_wave(channels, W, streams, seg):
    check_int8(channels, W, streams, seg)


@pytest.mark.parametrize("channels,W,streams,seg", [
    (16, 256, 1, 1), (16, 257, 1, 1), (16, 257, 3, 8),             # four and five workgroups per row, the last with a wave of four
    (32, 129, 1, 2), (48, 65, 23, 1), (48, 65, 24, 1),             # the most streams that add by workgroup, and one more
    (80, 33, 2, 1), (160, 17, 2, 1),                               # groups of channels, the last with two waves of four
    (80, 97, 21, 8), (80, 97, 22, 8),                              # wide tiles: the most streams that add by workgroup, and one more
])
def test_counters_on_both_sides_of_the_choice(channels, W, streams, seg):
    check_int8(channels, W, streams, seg)


def check_int8(channels, W, streams, seg):
    rng = np.random.default_rng(channels + W)
    q = dict(act="relu_shr_clamp", shr=4, clamp_hi=15)
    c = (16, channels, channels, 16)
    x = rng.integers(1, 16, size=(streams, 8, W, c[0])).astype(np.int8)            # every value an event: the largest counts
    x[:, :, W // 2:] *= rng.random((streams, 8, W - W // 2, c[0])) < 0.3
    layers = [conv(c[0], c[1], 3, 3, p_h=1, p_w=1, **q), maxpool(c[1]), conv(c[1], c[2], 3, 3, p_h=1, p_w=1, **q), conv(c[2], c[3], 3, 3, p_h=1, p_w=1, act="relu")]
    w = [rng.integers(-6, 9, size=(L["c_out"], L["c_in"], 3, 3)).astype(np.int8) if L["kind"] == "conv" else None for L in layers]
    wl = dict(name="counters", precision="i8", in_h=8, in_w=W, in_c=c[0], layers=layers, weights=w, biases=[None] * 4, x=x, seg_rows=1, streams=streams)
    out, st, net = gpu_run(wl, seg_rows=seg, return_streams=True)
    assert st.layer_kernels()[0] == "conv3x3_mfma"
    for b in sorted({0, streams - 1}):
        e_out, e_st = oracle_stream(wl, b)
        g = st.get_stats(b)
        assert np.array_equal(out[b], e_out)
        assert g["events_in"].tolist() == e_st["events_in"].tolist()
        assert g["macs"].tolist() == e_st["macs"].tolist()
    st.close(); net.destroy()


@pytest.mark.parametrize("prec,c_in,channels,W,streams,seg", [
    ("f32", 16, 16, 256, 1, 1), ("f32", 16, 16, 257, 1, 1), ("f32", 8, 16, 257, 3, 8),       # four and five workgroups per row, the last with a wave of four
    ("f32", 16, 32, 128, 1, 1), ("f32", 16, 32, 129, 1, 2), ("bf16", 32, 32, 129, 1, 1),     # two waves side by side along the channels
    ("f32", 16, 48, 64, 1, 1), ("f32", 8, 48, 65, 39, 1), ("f32", 16, 48, 65, 40, 1),        # four; the most streams that add by workgroup, and one more
    ("bf16", 32, 64, 65, 39, 2), ("bf16", 32, 64, 65, 40, 2), ("bf16", 16, 16, 257, 3, 8),
    ("f32", 16, 80, 33, 2, 1), ("f32", 16, 160, 17, 2, 1),                                   # groups of channels, the last with two waves of four
    ("bf16", 32, 96, 97, 21, 8), ("bf16", 32, 96, 97, 22, 8), ("bf16", 16, 80, 97, 21, 8),   # wide tiles: likewise
])
def test_counters_of_float_nets(prec, c_in, channels, W, streams, seg):
    """Values and weights of -1, 0 and 1: up to the last layer every sum is a whole number that 32 bits hold (9 * 160 * 9 * 32 at most),
    and the first layer's are at most 288, so that no event is lost or made by rounding."""
    rng = np.random.default_rng(channels + W)
    c = (c_in, channels, channels, 16)
    x = rng.integers(0, 2, size=(streams, 8, W, c_in)).astype(np.float32)
    x[:, :, W // 2:] *= rng.random((streams, 8, W - W // 2, 1)) < 0.5
    layers = [conv(c[0], c[1], 3, 3, p_h=1, p_w=1), maxpool(c[1]), conv(c[1], c[2], 3, 3, p_h=1, p_w=1), conv(c[2], c[3], 3, 3, p_h=1, p_w=1)]
    w = [rng.integers(-1, 2, size=(L["c_out"], L["c_in"], 3, 3)).astype(np.float32) if L["kind"] == "conv" else None for L in layers]
    wl = dict(name="counters", precision=prec, in_h=8, in_w=W, in_c=c_in, layers=layers, weights=w, biases=[None] * 4, x=x, seg_rows=1, streams=streams)
    out, st, net = gpu_run(wl, seg_rows=seg, return_streams=True)
    assert st.layer_kernels()[0] == "conv3x3_mfma"
    for b in sorted({0, streams - 1}):
        check_stream(wl, out[b], b)
        _, e_st = oracle_stream(wl, b, emit_round="bf16" if prec == "bf16" else None)
        g = st.get_stats(b)
        assert g["events_in"].tolist() == e_st["events_in"].tolist()
        assert g["macs"].tolist() == e_st["macs"].tolist()
    st.close(); net.destroy()
