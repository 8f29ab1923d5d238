"""One 3x3 layer on the matrix cores at the ends of what its contraction distinguishes: numbers of K-steps around whole rounds of
three, stretches with events in every K-step, in some and in none, widths around the edges of tiles and of the blocks that rows are
brought in by, narrow and wide tiles."""
import numpy as np
import pytest

from helpers import check_stream, gpu_run
from workloads import conv, round_to_bf16

pytestmark = pytest.mark.gpu


def layer(prec, c_in, c_out, H, W, streams, seed):
    rng = np.random.default_rng(seed)
    if prec == "i8":
        x = rng.integers(1, 16, size=(streams, H, W, c_in)).astype(np.int8)
        w = rng.integers(-8, 8, size=(c_out, c_in, 3, 3)).astype(np.int8)
    else:
        x = rng.random((streams, H, W, c_in), dtype=np.float32) + 0.1
        w = rng.normal(0, np.sqrt(2.0 / (9 * c_in)), size=(c_out, c_in, 3, 3)).astype(np.float32)
    x[1 % streams, :, :, c_in // 2:] = 0                       # the second half of the channels without events
    x[1 % streams, : H // 2, W // 2:] = 0
    x[2 % streams, 1:] = 0                                     # events in the first row only: those of row 3 have none
    x[2 % streams, 0, :, 1:] = 0
    if prec == "bf16":
        x, w = round_to_bf16(x), round_to_bf16(w)
    return dict(name="ksteps", precision=prec, in_h=H, in_w=W, in_c=c_in, layers=[conv(c_in, c_out, 3, 3, p_h=1, p_w=1)], weights=[w],
                biases=[None], x=x, seg_rows=1, streams=streams)


@pytest.mark.parametrize("prec,c_in,c_out,W", [
    ("i8", 16, 16, 64), ("i8", 32, 32, 33), ("i8", 48, 16, 65), ("i8", 64, 64, 15), ("i8", 80, 32, 31), ("i8", 128, 48, 17),
    ("f32", 8, 32, 31), ("f32", 16, 16, 63), ("f32", 32, 32, 33), ("f32", 48, 64, 16),
    ("bf16", 24, 16, 64), ("bf16", 32, 64, 17), ("bf16", 64, 64, 2), ("bf16", 96, 32, 47), ("bf16", 160, 32, 32), ("bf16", 256, 64, 18)])
@pytest.mark.parametrize("seg", [1, 2, 5])
def test_every_number_of_ksteps(prec, c_in, c_out, W, seg):
    wl = layer(prec, c_in, c_out, 7, W, 3, seed=c_in * 100 + W)
    out, st, net = gpu_run(wl, seg_rows=seg, return_streams=True)
    assert st.layer_kernels() == ["conv3x3_mfma"]
    st.close(); net.destroy()
    for b in range(3):
        check_stream(wl, out[b], b)


@pytest.mark.parametrize("prec,c_in,c_out,W,streams", [("bf16", 64, 64, 65, 50), ("bf16", 128, 64, 31, 100), ("bf16", 256, 32, 33, 100),
                                                       ("bf16", 24, 64, 64, 50), ("i8", 64, 64, 56, 50), ("i8", 16, 32, 130, 50)])
def test_wide_tiles(prec, c_in, c_out, W, streams):
    """50 streams and more, eight rows at once: enough for tiles of 32 positions x 32 channels."""
    wl = layer(prec, c_in, c_out, 8, W, streams, seed=W)
    out = gpu_run(wl, seg_rows=8)
    for b in (0, 1, 2, streams - 1):
        check_stream(wl, out[b], b)
    # (the others hold what streams of a net of their own would: the same bits for the same rows)
    few = {**wl, "x": wl["x"][3:6], "streams": 3}
    assert np.array_equal(gpu_run(few, seg_rows=1), out[3:6])
