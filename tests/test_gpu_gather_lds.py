"""1-D layers whose windows go through LDS, which they do in launches of many tiles: one, two and four streams per tile, a stream that
fills no tile, windows over the ring's end and the signal's ends, strides, channels of one K-step and several to a row; bit for bit what
a launch of few streams gives, and the oracle's values.  (That these launches go that way, and those of few streams do not, is checked
without a GPU: test_host_schedule.)"""
import numpy as np
import pytest

from helpers import check_stream, gpu_run
from workloads import conv

pytestmark = pytest.mark.gpu


CASES = [
    ((1, 32, 32, 64, 64, 64, 64), 9, (1, 2, 1, 2, 1, 1), 0, 16, 61),       # four streams per tile behind the second stride, two before
    ((1, 64, 64, 64), 9, (1, 1, 1), 4, 16, 45),                            # one stream per tile; rows outside the signal
    ((1, 64, 64, 48), 9, (1, 1, 2), 0, 5, 130),                            # two, five of eight positions; channels that fill no tile
    ((1, 16, 32, 16), 9, (1, 1, 1), 0, 13, 200),                           # one K-step to a row
    ((4, 64, 64), 5, (2, 2), 2, 16, 150),                                  # windows of every second row, over the signal's ends
]


@pytest.mark.parametrize("chans,k,strides,pad,seg,streams", CASES)
def test_windows_through_lds(chans, k, strides, pad, seg, streams):
    rng = np.random.default_rng(streams)
    n, h = len(strides), 150
    layers = [conv(chans[i], chans[i + 1], k, 1, s=strides[i], p_h=pad) for i in range(n)]
    ws = [rng.normal(0, (2 / (k * chans[i])) ** 0.5, size=(chans[i + 1], chans[i], k, 1)).astype(np.float32) for i in range(n)]
    x = rng.normal(size=(streams, h, 1, chans[0])).astype(np.float32)
    x[:, 40:75] = 0
    wl = dict(name="lds", precision="f32", in_h=h, in_w=1, in_c=chans[0], layers=layers, weights=ws, biases=[None] * n, x=x, seg_rows=seg, streams=streams)
    out = gpu_run(wl, seg_rows=seg)
    for b in (0, 1, streams - 1):
        check_stream(wl, out[b], b)
    few = gpu_run({**wl, "x": x[:3], "streams": 3}, seg_rows=seg)
    assert np.array_equal(few, out[:3])
