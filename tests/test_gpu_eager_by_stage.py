"""Eager emission of float32 nets too large for one workgroup per stream: pushes in stages, and, read push by push, pushed apart or
recorded into a graph, a stage after the other, against the conventional network on the rows pushed so far and against the layers one
after the other, whose counters must be the same."""
import numpy as np
import pytest

import oracle
from test_gpu_eager_stages import check, open_eager
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


def workload(h, w, streams, seed):
    rng = np.random.default_rng(seed)
    chans = (3, 32, 32, 64, 48)
    layers, ws = [], []
    for i in range(4):
        layers.append(conv(chans[i], chans[i + 1], 3, 3, p_h=1, p_w=1))
        ws.append(rng.normal(0, (2 / (9 * chans[i])) ** 0.5, size=(chans[i + 1], chans[i], 3, 3)).astype(np.float32))
        if i == 1:
            layers.append(maxpool(32))
            ws.append(None)
    x = rng.normal(size=(streams, h, w, 3)).astype(np.float32)
    x[rng.random((streams, h, w)) < 0.5] = 0
    return dict(name="by_stage", precision="f32", in_h=h, in_w=w, in_c=3, layers=layers, weights=ws, biases=[None] * 5, x=x, seg_rows=1, streams=streams)


@pytest.mark.parametrize("h,w,streams,seg,reads", [(14, 97, 3, 2, ()), (14, 97, 3, 2, tuple(range(7))), (13, 64, 60, 3, (1, 2)), (11, 128, 1, 3, (0, 1, 3))])
def test_reads_in_between(h, w, streams, seg, reads, monkeypatch):
    wl = workload(h, w, streams, h + w)
    some = sorted({0, streams // 2, streams - 1})
    stats = []
    for plain in (False, True):
        if plain:
            monkeypatch.setenv("IDF_NO_ROW_STAGES", "1")
        net, st, x, out = open_eager(wl, seg)
        for sample in range(2):
            for i, r in enumerate(range(0, h, seg)):
                st.push_segment(x[:, r:r + seg].contiguous())
                if i in reads:
                    check(wl, st.read_announced(*out).cpu().numpy(), min(r + seg, h), some)
            check(wl, st.read_announced(*out).cpu().numpy(), h, some)
        # (events of the first layer are those of the input; sums in another order may be zero here and not there)
        stats.append([int(st.get_stats(b)["events_in"][0]) for b in some])
        st.close(); net.destroy()
    assert stats[0] == stats[1] == [2 * np.count_nonzero(wl["x"][b]) for b in some]


@pytest.mark.parametrize("h,w,streams,seg,reads", [(14, 97, 3, 2, ()), (14, 97, 3, 2, tuple(range(7))), (13, 64, 60, 3, (1, 2)), (11, 128, 1, 3, (0, 1, 3))])
def test_counters_of_every_layer(h, w, streams, seg, reads, monkeypatch):
    """Whole numbers with few weights per channel: every sum is exact (eight taps per channel, below 8^4), whatever its order, and so is
    which differences are zero."""
    wl = workload(h, w, streams, h + w)
    rng = np.random.default_rng(h)
    for i, L in enumerate(wl["layers"]):
        if L["kind"] != "conv":
            continue
        k = np.zeros((L["c_out"], 9 * L["c_in"]), np.float32)
        for o in range(L["c_out"]):
            k[o, rng.choice(9 * L["c_in"], 8, replace=False)] = rng.choice([-1, 1], 8)
        wl["weights"][i] = k.reshape(L["c_out"], L["c_in"], 3, 3)
    wl["x"] = (rng.random(wl["x"].shape) < 0.5).astype(np.float32)
    results = []
    for plain in (False, True):
        if plain:
            monkeypatch.setenv("IDF_NO_ROW_STAGES", "1")
        net, st, x, out = open_eager(wl, seg)
        for i, r in enumerate(range(0, h, seg)):
            st.push_segment(x[:, r:r + seg].contiguous())
            if i in reads:
                st.read_announced(*out)
        results.append((st.read_announced(*out).cpu().numpy(), [st.get_stats(b)["events_in"].tolist() for b in range(streams)]))
        st.close(); net.destroy()
    assert all(min(e) > 0 for e in results[0][1]) and results[0][1] == results[1][1]
    assert np.array_equal(results[0][0], results[1][0])


def test_streams_apart():
    wl = workload(12, 100, 4, 5)
    net, st, x, out = open_eager(wl, 2)
    order = [0, 1, 1, 3, 2, 0, 2, 1, 3, 0, 3, 2]
    at = [0] * 4
    for r in range(0, 4, 2):
        st.push_segment(x[:, r:r + 2].contiguous())
    at = [4] * 4
    for b in order:
        st.push_segment(x[b:b + 1, at[b]:at[b] + 2].contiguous(), stream_ids=[b])
        at[b] += 2
    st.push_segment(x[:, 10:12].contiguous())
    check(wl, st.read_announced(*out).cpu().numpy(), 12, range(4))
    st.close(); net.destroy()


def test_recorded():
    import torch
    import paper_1804_10727_amd as idf
    wl = workload(8, 128, 2, 9)
    net = idf.net_from_workload(wl)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = idf.Streams(net, 2, max_seg_rows=2, stream=stream)
        st.enable_eager()
        x = torch.from_numpy(wl["x"]).cuda()
        rows = [x[:, r:r + 2].contiguous() for r in range(0, 8, 2)]
        for row in rows:
            st.push_segment(row)
    stream.synchronize()
    out = (len(wl["layers"]), list(oracle.layer_shapes(wl["layers"], 8, 128))[-1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for row in rows:
            st.push_segment(row)
    for k in range(3):
        wl["x"] = np.roll(wl["x"], 5, axis=2)
        for i, r in enumerate(range(0, 8, 2)):
            rows[i].copy_(torch.from_numpy(np.ascontiguousarray(wl["x"][:, r:r + 2])))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            got = st.read_announced(*out)
        stream.synchronize()
        check(wl, got.cpu().numpy(), 8, range(2))
    st.close(); net.destroy()
