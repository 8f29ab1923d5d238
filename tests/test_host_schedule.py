"""The schedule of pushes, launch by launch, on a stand-in for the HIP runtime (no GPU): which rows every launch of the 3x3
kernel reads and writes, what is refused, and what a failed launch leaves behind."""
import numpy as np
import pytest

import host_runtime


@pytest.fixture(scope="session")
def runtime(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("runtime"))


def chain(prec, h, w, channels, pools=()):
    """A net of 3x3 layers, with a 2x2 pool behind the layers in `pools`."""
    import paper_1804_10727_amd as idf
    from workloads import conv, maxpool
    layers, weights = [], []
    for i, (a, b) in enumerate(zip(channels, channels[1:])):
        kw = dict(act="relu_shr_clamp", shr=4, clamp_hi=15) if prec == "i8" and i + 2 < len(channels) else {}
        layers.append(conv(a, b, 3, 3, p_h=1, p_w=1, **kw))
        weights.append(np.ones((b, a, 3, 3), {"f32": np.float32, "bf16": np.uint16, "i8": np.int8}[prec]))
        if i in pools:
            layers.append(maxpool(b))
            weights.append(None)
    return idf.Net(prec, h, w, channels[0], layers, weights)


# ---- the event path next to layers large enough for wide tiles -------------------------------------------------
def event_path(rt, streams, seg):
    net = chain("i8", 16, 112, [1, 16, 32, 32])
    st = host_runtime.Streams(net, streams, seg)
    rt.host_begin()
    st.check(st.L.idf_set_event_path(st.h, 4))
    for _ in range(2):
        for _ in range(16 // seg):
            st.push(seg)
        assert (st.read(16) == 16).all()
    assert rt.host_error() == b"", rt.host_error()
    st.close()


@pytest.mark.parametrize("streams,seg", [(192, 1), (256, 2), (64, 8), (1, 16)])
def test_event_path_next_to_wide_layers(runtime, streams, seg):
    host_runtime.run(runtime, "test_host_schedule", "event_path", streams, seg)
