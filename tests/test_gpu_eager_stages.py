"""Eager emission in stages: pushes that follow one another without a read go through the net side by side, each a stage behind the
next.  The announced values and the counted events have to be those of the layers one after the other (IDF_NO_ROW_STAGES), and those
of the conventional network on the rows pushed so far: reads after some pushes and after every one, stages of one and of several
layers (and workgroups of eight waves, from 129 streams on), rows that no deeper layer sees any more, streams pushed apart, a reset on the way,
pushes recorded into a graph."""
import numpy as np
import pytest

import oracle
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


def workload(prec, h, w, streams, n_conv, seed):
    rng = np.random.default_rng(seed)
    chans = (2, 16, 32, 16, 48, 16, 16, 32, 16, 16)[:n_conv + 1]
    inner = dict(act="relu_shr_clamp", shr=5, clamp_hi=15) if prec == "i8" else {}
    layers, ws = [], []
    for i in range(n_conv):
        layers.append(conv(chans[i], chans[i + 1], 3, 3, p_h=1, p_w=1, **(inner if i + 1 < n_conv else dict(act="relu"))))
        shape = (chans[i + 1], chans[i], 3, 3)
        ws.append(rng.integers(-8, 8, size=shape).astype(np.int8) if prec == "i8" else
                  rng.normal(0, (2 / (9 * chans[i])) ** 0.5, size=shape).astype(np.float32))
        if i in (0, 3) and i + 1 < n_conv:
            layers.append(maxpool(chans[i + 1]))
            ws.append(None)
    x = rng.integers(-9, 16, size=(streams, h, w, 2)).astype(np.int8) if prec == "i8" else rng.normal(size=(streams, h, w, 2)).astype(np.float32)
    x[rng.random((streams, h, w)) < 0.4] = 0
    return dict(name="stages", precision=prec, in_h=h, in_w=w, in_c=2, layers=layers, weights=ws, biases=[None] * len(ws), x=x, seg_rows=1, streams=streams)


def open_eager(wl, seg):
    import paper_1804_10727_amd as idf
    from paper_1804_10727_amd.binding import input_tensor
    net = idf.net_from_workload(wl)
    st = idf.Streams(net, wl["streams"], max_seg_rows=seg)
    st.enable_eager()
    return net, st, input_tensor(wl), (len(wl["layers"]), list(oracle.layer_shapes(wl["layers"], wl["in_h"], wl["in_w"]))[-1])


def check(wl, got, rows, streams):
    xp = wl["x"].copy()
    xp[:, rows:] = 0
    for b in streams:
        want = oracle.dense(wl["layers"], xp[b], wl["weights"], wl["biases"], integer=wl["precision"] == "i8")
        if wl["precision"] == "i8":
            assert np.array_equal(got[b].astype(np.int64), want), (rows, b)
        else:       # float32 sums of up to 432 products, seven layers deep
            assert np.max(np.abs(got[b] - want)) <= 1e-5 * max(1e-30, np.max(np.abs(want))), (rows, b)


@pytest.mark.parametrize("prec,h,w,streams,n_conv,seg", [
    ("f32", 21, 18, 2, 4, 1), ("i8", 22, 33, 3, 9, 1), ("f32", 17, 16, 5, 7, 3), ("i8", 23, 21, 65, 4, 2), ("f32", 13, 17, 130, 3, 1),
    ("i8", 12, 16, 256, 5, 2), ("i8", 9, 2, 1, 2, 1), ("f32", 4, 20, 4, 3, 1),
])
def test_against_layers_one_after_the_other(prec, h, w, streams, n_conv, seg, monkeypatch):
    wl = workload(prec, h, w, streams, n_conv, h * w + streams)
    some = sorted({0, streams // 2, streams - 1})
    pauses = [3, 4, 5, 9, 10]                  # pushes after which results are asked for, in a row and further apart
    results = []
    for plain in (False, True):
        if plain:
            monkeypatch.setenv("IDF_NO_ROW_STAGES", "1")
        net, st, x, out = open_eager(wl, seg)
        seen = []
        for sample in range(2):
            for i, r in enumerate(range(0, h, seg)):
                st.push_segment(x[:, r:r + seg].contiguous())
                if (i + sample) in pauses:
                    got = st.read_announced(*out).cpu().numpy()
                    check(wl, got, r + seg, some)
                    seen.append(got)
        seen.append(st.read_announced(*out).cpu().numpy())
        check(wl, seen[-1], h, some)
        results.append((seen, [st.get_stats(b)["events_in"].tolist() for b in some]))
        st.close(); net.destroy()
    assert results[0][1] == results[1][1]
    for a, b in zip(results[0][0], results[1][0]):
        assert np.array_equal(a, b)                # the same sums in the same order


@pytest.mark.parametrize("prec,h,w,streams,n_conv,seg", [("i8", 26, 16, 256, 5, 1), ("f32", 23, 17, 130, 4, 1), ("f32", 17, 20, 201, 4, 1), ("i8", 25, 33, 140, 7, 2)])
def test_two_workgroups_to_a_compute_unit(prec, h, w, streams, n_conv, seg, monkeypatch):
    """Samples long enough for the stages to pay there, read once on the way and at the end."""
    wl = workload(prec, h, w, streams, n_conv, h * w + streams)
    some = sorted({0, streams // 2, streams - 1})
    results = []
    for plain in (False, True):
        if plain:
            monkeypatch.setenv("IDF_NO_ROW_STAGES", "1")
        net, st, x, out = open_eager(wl, seg)
        seen = []
        for sample in range(3):
            for r in range(0, h, seg):
                st.push_segment(x[:, r:r + seg].contiguous())
                if sample == 2 and r // seg == 6:
                    seen.append(st.read_announced(*out).cpu().numpy())
                    check(wl, seen[-1], r + seg, some)
            seen.append(st.read_announced(*out).cpu().numpy())
            check(wl, seen[-1], h, some)
        results.append((seen, [st.get_stats(b)["events_in"].tolist() for b in some]))
        st.close(); net.destroy()
    assert results[0][1] == results[1][1]
    for a, b in zip(results[0][0], results[1][0]):
        assert np.array_equal(a, b)


def test_streams_apart_reset_and_inner_levels():
    wl = workload("f32", 19, 18, 3, 4, 7)
    net, st, x, out = open_eager(wl, 1)
    for r in range(5):
        st.push_segment(x[:, r:r + 1].contiguous())
    for b in (1, 0, 2):                            # one row each, out of order, with four pushes on their way
        st.push_segment(x[b:b + 1, 5:6].contiguous(), stream_ids=np.array([b], np.int32))
    for r in range(6, 8):
        st.push_segment(x[:, r:r + 1].contiguous())
    shapes = list(oracle.layer_shapes(wl["layers"], wl["in_h"], wl["in_w"]))
    xp = wl["x"].copy()
    xp[:, 8:] = 0
    for lv in (2, 3, out[0]):
        got, first, cnt = st.read_announced_rows(lv, shapes[lv - 1][1:], shapes[lv - 1][0])
        got = got.cpu().numpy()
        for b in range(3):
            want = oracle.dense(wl["layers"][:lv], xp[b], wl["weights"][:lv], [None] * lv)[int(first[b]):int(first[b] + cnt[b])]
            assert cnt[b] > 0 and np.max(np.abs(got[b, :int(cnt[b])] - want)) <= 1e-5 * max(1e-30, np.max(np.abs(want))), (lv, b)
    for r in range(8, 11):
        st.push_segment(x[:, r:r + 1].contiguous())
    st.reset()                                     # with pushes on their way: they are gone, and their events with them
    assert not any(st.get_stats(b)["events_in"].any() for b in range(3))
    for r in range(19):
        st.push_segment(x[:, r:r + 1].contiguous())
    check(wl, st.read_announced(*out).cpu().numpy(), 19, range(3))
    assert int(st.get_stats(1)["events_in"][0]) == np.count_nonzero(wl["x"][1])
    st.close(); net.destroy()


def test_recorded_pushes():
    """A whole sample recorded without its read: every replay leaves the output complete."""
    import torch
    import paper_1804_10727_amd as idf
    wl = workload("i8", 14, 18, 2, 4, 11)
    net = idf.net_from_workload(wl)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = idf.Streams(net, 2, stream=stream)
        st.enable_eager()
        x = torch.from_numpy(wl["x"]).cuda()
        rows = [x[:, r:r + 1].contiguous() for r in range(14)]
        for row in rows:
            st.push_segment(row)
    stream.synchronize()
    out = (len(wl["layers"]), list(oracle.layer_shapes(wl["layers"], 14, 18))[-1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for row in rows:
            st.push_segment(row)
    for k in range(3):
        wl["x"] = np.roll(wl["x"], 3, axis=2)
        for r in range(14):
            rows[r].copy_(torch.from_numpy(np.ascontiguousarray(wl["x"][:, r:r + 1])))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            got = st.read_announced(*out)
        stream.synchronize()
        check(wl, got.cpu().numpy(), 14, range(2))
    st.close(); net.destroy()
