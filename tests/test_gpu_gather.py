"""The matrix-core kernel that gathers its windows: shapes at the edges of its tiles -- channel counts that fill
no cell or tile, kernels from one tap to nine, strides, padding, streams that share a tile and streams that do not,
more rows than a tile -- against the oracle, pushed together, in parts, and several pushes per launch."""
import numpy as np
import pytest

import workloads as wl_mod
from helpers import TOL, oracle_dense, rel_err
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


def _signal(streams, length, chans, kernels, strides, pads, seed):
    rng = np.random.default_rng(seed)
    x = rng.normal(size=(streams, length, 1, chans[0])).astype(np.float32)
    x[rng.random((streams, length)) < 0.4] = 0.0
    layers = [conv(chans[i], chans[i + 1], kernels[i], 1, s=strides[i], p_h=pads[i]) for i in range(len(kernels))]
    weights = wl_mod._normal_weights(rng, layers, 2.0)
    biases = [None if i % 2 else rng.normal(0.0, 0.1, size=L["c_out"]).astype(np.float32) for i, L in enumerate(layers)]
    return wl_mod._finish("gather", "f32", length, 1, chans[0], layers, weights, biases, x, 1)


@pytest.mark.parametrize("streams,length,seg,chans,kernels,strides,pads", [
    (1, 40, 1, (1, 3, 16), (3, 1), (1, 1), (0, 0)),
    (17, 61, 1, (2, 17, 64), (9, 2), (1, 2), (0, 0)),          # one row per push: sixteen streams to a tile, and one over
    (33, 100, 5, (5, 64, 33, 7), (4, 9, 3), (2, 1, 1), (1, 4, 1)),
    (3, 200, 16, (64, 64, 64), (9, 9), (1, 2), (8, 0)),
    (40, 130, 16, (1, 20, 12, 40), (9, 7, 5), (1, 2, 2), (0, 3, 2)),
])
@pytest.mark.parametrize("batch", [1, 16])
def test_signals_at_the_edges_of_the_tiles(streams, length, seg, chans, kernels, strides, pads, batch):
    import torch
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    wl = _signal(streams, length, chans, kernels, strides, pads, seed=streams)
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, streams, max_seg_rows=seg)
    assert set(st.layer_kernels()) == {"cascade1d"}
    st.set_push_batching(batch)
    x = input_tensor(wl)
    keep, half = [], (streams + 1) // 2
    for i, r in enumerate(range(0, length, seg)):
        rows = x[:, r:r + seg].contiguous()
        if i % 7 == 3 and streams > 1:                            # the streams in two parts, out of step in between
            parts = [np.arange(half, streams, dtype=np.int32), np.arange(half, dtype=np.int32)]
        else:
            parts = [None]
        for ids in parts:
            keep.append(rows if ids is None else rows[torch.from_numpy(ids.astype(np.int64)).to(rows.device)].contiguous())
            st.push_segment(keep[-1], stream_ids=ids)
    out, _, cnt = st.read_outputs(int(st.sizes.out_h))
    o = out.cpu().numpy()
    for b in range(streams):
        want = oracle_dense(wl, b)
        assert cnt[b] == want.shape[0]
        assert rel_err(o[b, :cnt[b]], want) <= TOL["f32"], b
    ev = st.get_stats(streams - 1)["events_in"]
    assert ev[0] == np.count_nonzero(wl["x"][streams - 1]) and (ev[1:] > 0).all()
    st.close(); net.destroy()


def _image(prec, streams, h, w, c0, layers, seed):
    rng = np.random.default_rng(seed)
    convs = [L["kind"] == "conv" for L in layers]
    if prec == "i8":
        q = dict(act="relu_shr_clamp", shr=4, clamp_hi=15)
        layers = [dict(L, **(q if i + 1 < len(layers) else dict(act="relu"))) if c else L for i, (L, c) in enumerate(zip(layers, convs))]
        weights = [rng.integers(-8, 8, size=(L["c_out"], L["c_in"], L["k_h"], L["k_w"])).astype(np.int8) if c else None for L, c in zip(layers, convs)]
        biases = [rng.integers(-20, 40, size=L["c_out"]).astype(np.int32) if c and i % 2 else None for i, (L, c) in enumerate(zip(layers, convs))]
        x = rng.integers(-9, 16, size=(streams, h, w, c0)).astype(np.int8)
    else:
        weights = wl_mod._normal_weights(rng, layers, 2.0)
        biases = [rng.normal(0.0, 0.1, size=L["c_out"]).astype(np.float32) if c and i % 2 else None for i, (L, c) in enumerate(zip(layers, convs))]
        x = rng.random((streams, h, w, c0)).astype(np.float32)
        if prec == "bf16":
            x, weights = wl_mod.round_to_bf16(x), [None if v is None else wl_mod.round_to_bf16(v) for v in weights]
    x[rng.random((streams, h, w)) < 0.4] = 0
    return layers, weights, biases, x


# (input rows, columns, channels, layers): kernels of one tap to five, strides 1, 2 and 4, padding, pools of even and odd
# maps, channels that fill no cell or tile, maps of fewer positions than a tile and of more
_NETS = [
    (31, 45, 3, [conv(3, 20, 5, 5, s=2, p_h=2, p_w=2), conv(20, 16, 3, 3, p_h=1, p_w=1), maxpool(16), conv(16, 33, 3, 3, s=2, p_h=1, p_w=1),
                 conv(33, 40, 1, 1), conv(40, 7, 3, 3)]),
    (23, 17, 1, [conv(1, 5, 4, 3, s=4, p_h=3, p_w=1), conv(5, 64, 1, 2), conv(64, 9, 2, 1, p_h=1)]),
    (26, 6, 17, [conv(17, 3, 3, 5, p_h=2, p_w=4), maxpool(3), maxpool(3), conv(3, 48, 2, 2)]),
    (9, 70, 40, [conv(40, 65, 2, 3, s=1, p_w=2), conv(65, 18, 3, 1, s=2)]),
]


@pytest.mark.parametrize("net_i", range(len(_NETS)))
@pytest.mark.parametrize("prec", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("streams,seg", [(1, 1), (5, 3), (18, 1)])
def test_images_through_layers_of_several_kinds(prec, net_i, streams, seg):
    """Two samples: streams in step, in two parts, rows in pixel segments, a stream that moves to another slot half way;
    outputs and counters against the oracle."""
    import torch
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    import oracle
    h, w, c0, layers = _NETS[net_i]
    layers, weights, biases, x = _image(prec, streams, h, w, c0, layers, seed=net_i * 10 + streams)
    wl = wl_mod._finish("gather2d", prec, h, w, c0, layers, weights, biases, x, 1)
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, streams, max_seg_rows=seg)
    assert set(st.layer_kernels()) == {"conv_gather"}
    xd, half = input_tensor(wl), (streams + 1) // 2
    emulate = "bf16" if prec == "bf16" else None
    for sample in range(2):
        for i, r in enumerate(range(0, h, seg)):
            rows = xd[:, r:r + seg].contiguous()
            if seg == 1 and i % 5 == 2 and w > 4:
                for a, b in ((0, 1), (1, w - 2), (w - 2, w)):
                    st.push_pixels(xd[:, r, a:b].contiguous(), a)
            elif i % 5 == 3 and streams > 1:
                for ids in (np.arange(half, streams, dtype=np.int32), np.arange(half, dtype=np.int32)):
                    st.push_segment(rows[torch.from_numpy(ids.astype(np.int64)).to(rows.device)].contiguous(), stream_ids=ids)
            else:
                st.push_segment(rows)
        if sample == 0:
            ev = [st.get_stats(b) for b in range(streams)]
        out, _, cnt = st.read_outputs(int(st.sizes.out_h))
        o = out.cpu().numpy()
        assert (cnt == st.sizes.out_h).all()
        for b in range(streams):
            want = oracle.dense(layers, wl["x"][b], wl["weights"], wl["biases"], integer=prec == "i8", emit_round=emulate)
            if prec == "i8":
                assert np.array_equal(o[b].astype(np.int64), want), b
            else:
                assert rel_err(o[b], want) <= TOL["f32" if prec == "f32" else "bf16_emul"], b
    for b in range(streams):
        _, e = oracle.stream_run(layers, wl["x"][b], wl["weights"], wl["biases"], seg_rows=1, integer=prec == "i8", emit_round=emulate)
        if prec == "bf16":                                       # (a value that rounds to zero on one side only: a handful at most)
            assert np.allclose(ev[b]["events_in"].astype(float), e["events_in"], rtol=2e-3, atol=2), b
        else:
            assert ev[b]["events_in"].tolist() == e["events_in"].tolist() and ev[b]["macs"].tolist() == e["macs"].tolist(), b
    st.close(); net.destroy()


@pytest.mark.parametrize("prec", ["f32", "i8"])
def test_a_stream_of_several_kinds_of_layers_resumes_in_another_slot(prec):
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    h, w, c0, layers = _NETS[0]
    layers, weights, biases, x = _image(prec, 2, h, w, c0, layers, seed=3)
    wl = wl_mod._finish("gather2d", prec, h, w, c0, layers, weights, biases, x, 1)
    net = idf.net_from_workload(wl)
    for cut in (1, 14, 22):
        st = idf.Streams(net, 2, max_seg_rows=1)
        xd, a, b = input_tensor(wl), np.array([0], np.int32), np.array([1], np.int32)
        for r in range(cut):
            st.push_segment(xd[:1, r:r + 1].contiguous(), stream_ids=a)
        top, _, n0 = st.read_outputs(int(st.sizes.out_h), stream_ids=a)
        buf, pos = st.snapshot(0)
        st.restore(1, buf, pos)
        for r in range(cut, h):
            st.push_segment(xd[:1, r:r + 1].contiguous(), stream_ids=b)
        rest, _, n1 = st.read_outputs(int(st.sizes.out_h), stream_ids=b)
        got = np.concatenate([top.cpu().numpy()[0, :n0[0]], rest.cpu().numpy()[0, :n1[0]]])
        want = oracle_dense(wl, 0)
        assert got.shape == want.shape and rel_err(got, want) <= (0 if prec == "i8" else TOL["f32"])
        st.close()
    net.destroy()


def test_a_static_workspace_too_small_for_the_rings_still_holds_the_streams():
    """A net of several kinds of layers whose rings do not fit the library's own workspace goes layer by layer in it."""
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    h, w, c0, layers = _NETS[3]
    streams = 300                                                # 60 MiB with rings, 25 without
    layers, weights, biases, x = _image("f32", 2, h, w, c0, layers, seed=8)
    wl = wl_mod._finish("gather2d", "f32", h, w, c0, layers, weights, biases, np.repeat(x, streams // 2, axis=0), 1)
    net = idf.net_from_workload(wl)
    outs = []
    for static in (True, False):
        st = idf.Streams(net, streams, max_seg_rows=1, static_workspace=static)
        assert (set(st.layer_kernels()) == {"conv_gather"}) == (not static)
        xd = input_tensor(wl)
        for r in range(h):
            st.push_segment(xd[:, r:r + 1].contiguous())
        outs.append(st.read_outputs(int(st.sizes.out_h))[0].cpu().numpy())
        st.close()
    net.destroy()
    for o in outs:
        for b in (0, streams - 1):
            assert rel_err(o[b], oracle_dense(wl, b)) <= TOL["f32"]


@pytest.mark.parametrize("streams,seg,h,w,c0,layers", [
    (3, 2, 12, 11, 192, [conv(192, 20, 7, 7, p_h=3, p_w=3), conv(20, 5, 1, 1)]),
    (2, 1, 11, 3, 248, [conv(248, 17, 9, 2, p_h=1, p_w=1), conv(17, 16, 2, 2)]),       # a window of 1,116 cells
    (17, 3, 26, 2, 250, [conv(250, 5, 23, 1, p_h=2)]),
    (2, 4, 34, 33, 201, [conv(201, 16, 32, 32, p_h=1)]),
    (2, 1, 60, 1, 250, [conv(250, 7, 22, 1, p_h=2)]),                                  # one position per row
])
def test_large_windows(streams, seg, h, w, c0, layers):
    """float32: 200 input channels and more, windows of a thousand cells and more."""
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    import oracle
    layers, weights, biases, x = _image("f32", streams, h, w, c0, layers, seed=c0)
    x[0, :, w // 2:] = 0
    wl = wl_mod._finish("gather2d", "f32", h, w, c0, layers, weights, biases, x, 1)
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, streams, max_seg_rows=seg)
    assert set(st.layer_kernels()) == {"conv_gather"}
    xd = input_tensor(wl)
    for r in range(0, h, seg):
        st.push_segment(xd[:, r:r + seg].contiguous())
    ev = [st.get_stats(b) for b in range(streams)]
    o = st.read_outputs(int(st.sizes.out_h))[0].cpu().numpy()
    for b in range(streams):
        assert rel_err(o[b], oracle.dense(layers, wl["x"][b], wl["weights"], wl["biases"])) <= TOL["f32"], b
        _, e = oracle.stream_run(layers, wl["x"][b], wl["weights"], wl["biases"], seg_rows=1)
        assert ev[b]["events_in"].tolist() == e["events_in"].tolist() and ev[b]["macs"].tolist() == e["macs"].tolist(), b
    st.close(); net.destroy()
