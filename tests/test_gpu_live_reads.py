"""1-D signals: a push goes through all layers at once where every push so far has been read by itself, and side by side with the ones
before it else.  Whatever the order of pushes and reads, outputs, their places and the counters are those of one read at the end."""
import numpy as np
import pytest

from workloads import conv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("streams,seg,bounded", [(1, 1, False), (1, 16, False), (3, 5, True), (40, 16, False), (70, 7, True)])
def test_reads_between_pushes(streams, seg, bounded):
    import torch
    import paper_1804_10727_amd as idf
    rng = np.random.default_rng(streams + seg)
    chans, strides = (1, 32, 32, 64, 64), (1, 2, 1, 2)
    layers = [conv(chans[i], chans[i + 1], 9, 1, s=strides[i]) for i in range(4)]
    ws = [rng.normal(0, (2 / (9 * chans[i])) ** 0.5, size=(chans[i + 1], chans[i], 9, 1)).astype(np.float32) for i in range(4)]
    n = 40 * seg
    x = rng.normal(size=(streams, n, 1, 1)).astype(np.float32)
    x[:, n // 3:n // 2] = 0
    x = torch.from_numpy(x).cuda()
    # after which pushes outputs are read: after each, after each again, after several, after each
    patterns = [[], list(range(40)), [0, 1, 2, 5, 6, 7, 11, 20, 21, 22, 23, 30, 39]]
    results = []
    for reads in patterns:
        net = idf.Net("f32", n if bounded else 0, 1, 1, layers, ws)
        st = idf.Streams(net, streams, max_seg_rows=seg, out_cap_rows=0 if bounded else n)
        outs = [[] for _ in range(streams)]
        for i in range(40):
            st.push_segment(x[:, i * seg:(i + 1) * seg].contiguous())
            if i in reads or i == 39:
                out, first, cnt = st.read_outputs(n)
                assert all(int(first[b]) == sum(len(o) for o in outs[b]) for b in range(streams))
                for b in range(streams):
                    outs[b].append(out[b, :int(cnt[b])].cpu().numpy())
        results.append(([np.concatenate(o) for o in outs], [(st.get_stats(b)["events_in"].tolist(), st.get_stats(b)["macs"].tolist()) for b in range(streams)]))
        st.close(); net.destroy()
    for outs, stats in results[1:]:
        assert stats == results[0][1]
        assert all(len(a) > 0 or n < 60 for a in outs) and all(np.array_equal(a, b) for a, b in zip(outs, results[0][0]))
