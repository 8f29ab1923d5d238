"""Eager emission of a whole net in one launch: every level's announced values after every push against
the conventional network on the input seen so far, at the edges of the kernel's tiles (16 positions, pairs
of 16 channels), with pools at even and odd rows, few and many input channels, one to four rows per push,
streams pushed alone; and the sizes at which the layer-by-layer kernels take over."""
import numpy as np
import pytest

import oracle
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "i8"])
@pytest.mark.parametrize("w,h,c0,chans,seg,streams", [
    (16, 8, 1, (16, 16, 16), 1, 1),
    (33, 11, 3, (16, 48, 32), 1, 3),
    (2, 6, 16, (32, 16, 16), 2, 2),
    (70, 13, 4, (48, 64, 80), 3, 2),
    (31, 20, 2, (32, 32, 16), 4, 2),
    (18, 24, 3, (16, 32, 16), 9, 2),          # bands of more rows than one launch holds
])
def test_levels_after_every_push(prec, w, h, c0, chans, seg, streams):
    import torch
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    rng = np.random.default_rng(w * 100 + h)
    q = dict(act="relu_shr_clamp", shr=5, clamp_hi=15) if prec == "i8" else {}
    layers = [conv(c0, chans[0], 3, 3, p_h=1, p_w=1, **q), maxpool(chans[0]), conv(chans[0], chans[1], 3, 3, p_h=1, p_w=1, **q),
              conv(chans[1], chans[2], 3, 3, p_h=1, p_w=1, **({"act": "relu"} if prec == "i8" else {}))]
    if prec == "i8":
        ws = [None if L["kind"] != "conv" else rng.integers(-8, 8, size=(L["c_out"], L["c_in"], 3, 3)).astype(np.int8) for L in layers]
        x = rng.integers(-9, 16, size=(streams, h, w, c0)).astype(np.int8)
    else:
        ws = [None if L["kind"] != "conv" else rng.normal(0, (2 / (9 * L["c_in"])) ** 0.5, size=(L["c_out"], L["c_in"], 3, 3)).astype(np.float32) for L in layers]
        x = rng.normal(size=(streams, h, w, c0)).astype(np.float32)
    x[rng.random((streams, h, w)) < 0.3] = 0
    wl = dict(name="pass", precision=prec, in_h=h, in_w=w, in_c=c0, layers=layers, weights=ws, biases=[None] * 4, x=x, seg_rows=seg, streams=streams)
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, streams, max_seg_rows=seg)
    st.enable_eager()
    xd = input_tensor(wl)
    shp = [(h, w, c0)] + list(oracle.layer_shapes(layers, h, w))
    for sample in range(2):
        for r in range(0, h, seg):
            if r // seg % 2:                                      # every stream on its own, then all together
                for b in range(streams):
                    st.push_segment(xd[b:b + 1, r:r + seg].contiguous(), stream_ids=np.array([b], np.int32))
            else:
                st.push_segment(xd[:, r:r + seg].contiguous())
            xp = x.copy()
            xp[:, r + seg:] = 0
            for lv in range(5):
                got, first, cnt = st.read_announced_rows(lv, shp[lv][1:], shp[lv][0])
                got = got.cpu().numpy()
                for b in range(streams):
                    want = xp[b] if lv == 0 else oracle.dense(layers[:lv], xp[b], ws[:lv], [None] * lv, integer=prec == "i8")
                    lo, n = int(first[b]), int(cnt[b])
                    assert n >= 1
                    if prec == "i8":
                        assert np.array_equal(got[b, :n].astype(np.int64), want[lo:lo + n]), (r, lv, b)
                    else:
                        assert np.max(np.abs(got[b, :n] - want[lo:lo + n])) <= 1e-5 * max(1e-30, np.max(np.abs(want))), (r, lv, b)
        if sample == 0:
            ev = [st.get_stats(b)["events_in"] for b in range(streams)]
            assert all(int(e[0]) == np.count_nonzero(x[b]) and (e[1:] > 0).all() for b, e in enumerate(ev))
    st.close(); net.destroy()
