"""The gathering kernel where a launch has so many tiles that they go two by two: against the oracle, and bit for bit against the single
tiles that the same streams go through when they are few.  Channels and positions that leave half a tile over, windows of one cell,
over the ends of a signal and past the end of a ring, streams without events."""
import numpy as np
import pytest

import workloads as wl_mod
from helpers import TOL, rel_err
from test_gpu_gather import _image, _signal
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


def _run(wl, streams, seg, batch=1):
    import torch
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, len(streams), max_seg_rows=seg)
    assert set(st.layer_kernels()) <= {"cascade1d", "conv_gather"}
    if batch > 1:
        st.set_push_batching(batch)
    x = input_tensor(wl)[streams].contiguous()
    keep = []
    for r in range(0, wl["in_h"], seg):
        keep.append(x[:, r:r + seg].contiguous())
        st.push_segment(keep[-1])
    out, _, cnt = st.read_outputs(int(st.sizes.out_h))
    torch.cuda.synchronize()
    assert (cnt == st.sizes.out_h).all()
    o, stats = out.cpu().numpy(), [st.get_stats(i) for i in (0, len(streams) - 1)]
    st.close(); net.destroy()
    return o, stats


def _compare(wl, n, seg, batch=1, emulate=None):
    import oracle
    o, stats = _run(wl, list(range(n)), seg, batch)
    few, few_stats = _run(wl, [0, 1, n - 1], seg)                # single tiles
    assert np.array_equal(o[[0, 1, n - 1]], few)
    for a, b in zip(stats, few_stats):
        assert np.array_equal(a["events_in"], b["events_in"]) and np.array_equal(a["macs"], b["macs"])
    for i, b in enumerate((0, 1, n - 1)):
        want = oracle.dense(wl["layers"], wl["x"][b], wl["weights"], wl["biases"], integer=wl["precision"] == "i8", emit_round=emulate)
        if wl["precision"] == "i8":
            assert np.array_equal(few[i].astype(np.int64), want)
        else:
            assert rel_err(few[i], want) <= TOL["f32" if wl["precision"] == "f32" else "bf16_emul"]


@pytest.mark.parametrize("n,length,seg,chans,kernels,strides,pads", [
    (61, 300, 16, (1, 40, 33, 64), (9, 7, 5), (1, 1, 2), (0, 3, 2)),
    (70, 270, 15, (5, 64, 17), (2, 9), (1, 1), (1, 8)),
    (100, 260, 16, (3, 48, 20, 33), (1, 4, 9), (1, 2, 1), (0, 1, 4)),
])
def test_signals_two_by_two(n, length, seg, chans, kernels, strides, pads):
    wl = _signal(n, length, chans, kernels, strides, pads, seed=n)
    wl["x"][n - 1, length // 2:] = 0
    _compare(wl, n, seg, batch=16)


@pytest.mark.parametrize("prec", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("n,h,w,c0,layers", [
    (70, 20, 37, 2, [conv(2, 40, 3, 1, p_h=1), conv(40, 33, 2, 3, s=2, p_w=2), conv(33, 48, 3, 3)]),
    (64, 32, 45, 3, [conv(3, 20, 5, 5, s=2, p_h=2, p_w=2), conv(20, 65, 1, 1), maxpool(65), conv(65, 18, 3, 2, p_h=2, p_w=1)]),
])
def test_images_two_by_two(prec, n, h, w, c0, layers):
    layers, weights, biases, x = _image(prec, n, h, w, c0, layers, seed=w)
    x[1, :, w // 3:] = 0
    wl = wl_mod._finish("gather2d", prec, h, w, c0, layers, weights, biases, x, 1)
    _compare(wl, n, 16, emulate="bf16" if prec == "bf16" else None)


def test_large_windows_two_by_two():
    """float32, 1,550 cells."""
    layers, weights, biases, x = _image("f32", 40, 16, 31, 248, [conv(248, 33, 5, 5, p_h=2, p_w=2)], seed=1)
    _compare(wl_mod._finish("gather2d", "f32", 16, 31, 248, layers, weights, biases, x, 1), 40, 8)
