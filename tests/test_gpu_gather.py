"""The matrix-core kernel that gathers its windows: shapes at the edges of its tiles -- channel counts that fill
no cell or tile, kernels from one tap to nine, strides, padding, streams that share a tile and streams that do not,
more rows than a tile -- against the oracle, pushed together, in parts, and several pushes per launch."""
import numpy as np
import pytest

import workloads as wl_mod
from helpers import TOL, oracle_dense, rel_err
from workloads import conv

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
