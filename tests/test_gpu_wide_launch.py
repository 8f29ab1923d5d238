"""Steps of the 3x3 matrix-core kernel take wide tiles where the launch's steps together are many, though each alone is not: layers on
both sides of that line, of the least step that does and of layers that cannot, against the oracle and, bit for bit, against the same
streams in a small launch."""
import numpy as np
import pytest

from helpers import check_stream, gpu_run
from workloads import conv, round_to_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,channels,W,streams", [
    ("bf16", (8, 64, 64, 96), 62, 52),               # four rows at once: 416, 416 and 624 waves, 1,456 together
    ("bf16", (8, 64, 32, 64, 64, 64), 100, 24),      # 192 in the second layer, the least that goes along, 384 in the others
    ("bf16", (8, 64, 32, 64, 64, 64), 100, 23),      # 184
    ("bf16", (8, 16, 64, 64), 70, 59),               # the first layer has one tile of channels: never wide
    ("i8", (16, 64, 64, 64), 62, 60)])
def test_wide_by_launch(prec, channels, W, streams):
    rng = np.random.default_rng(W)
    H, n = 12, len(channels) - 1
    layers, weights = [], []
    for i in range(n):
        act = dict(act="relu") if prec == "bf16" or i == n - 1 else dict(act="relu_shr_clamp", shr=6, clamp_hi=15)
        layers.append(conv(channels[i], channels[i + 1], 3, 3, p_h=1, p_w=1, **act))
        shape = (channels[i + 1], channels[i], 3, 3)
        weights.append(rng.integers(-8, 8, size=shape).astype(np.int8) if prec == "i8"
                       else round_to_bf16(rng.normal(0, np.sqrt(2.0 / (9 * channels[i])), size=shape).astype(np.float32)))
    shape = (streams, H, W, channels[0])
    x = rng.integers(0, 16, size=shape).astype(np.int8) if prec == "i8" else round_to_bf16(rng.random(shape, dtype=np.float32))
    x[1, :, W // 2:] = 0
    wl = dict(name="wide", precision=prec, in_h=H, in_w=W, in_c=channels[0], layers=layers, weights=weights, biases=[None] * n, x=x,
              seg_rows=4, streams=streams)
    out = gpu_run(wl, seg_rows=4)
    for b in (0, 1, streams - 1):
        check_stream(wl, out[b], b)
    few = {**wl, "x": x[:3], "streams": 3}
    assert np.array_equal(gpu_run(few, seg_rows=4), out[:3])
