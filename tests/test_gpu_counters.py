"""Counters of events and multiply-adds where the waves of a workgroup add up before one of them adds for all (fewer than 24 streams)
and where each adds by itself: widths and channels that leave waves of a workgroup without work, pools, narrow and wide tiles.
Whole numbers: exact."""
import numpy as np
import pytest

from helpers import gpu_run, oracle_stream
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels", [16, 48, 128])
@pytest.mark.parametrize("W", [4, 17, 62, 130])
@pytest.mark.parametrize("streams,seg", [(1, 1), (23, 1), (23, 8), (24, 1)])
def test_counters_by_workgroup_and_by_wave(channels, W, streams, seg):
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
