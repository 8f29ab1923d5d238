"""Eager emission in stages of one layer that several workgroups share: tiles that divide among them and that do not, more tiles than
waves, layers with fewer tiles than workgroups, pools, odd widths and channels that fill no pair of tiles, against the layers one after
the other in one workgroup, bit for bit, and the conventional network."""
import numpy as np
import pytest

from test_gpu_eager_stages import check, open_eager, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,h,w,streams,n_conv,seg", [
    ("i8", 18, 112, 1, 8, 1),          # eight workgroups of four waves to a stage
    ("i8", 14, 65, 16, 8, 2),          # all eight, on half as many units
    ("i8", 11, 33, 31, 8, 1),          # four, a remainder of streams
    ("f32", 16, 130, 2, 4, 3),         # tiles in several rounds
    ("f32", 15, 31, 63, 4, 1),         # four
    ("f32", 9, 17, 85, 3, 2),          # four, three layers
    ("f32", 8, 16, 128, 2, 1),         # four, two layers
    ("i8", 7, 2, 3, 1, 1),             # one layer, one tile: no stages
])
def test_against_one_workgroup(prec, h, w, streams, n_conv, seg, monkeypatch):
    wl = workload(prec, h, w, streams, n_conv, h * w + streams)
    some = sorted({0, streams // 2, streams - 1})
    results = []
    for plain in (False, True):
        if plain:
            monkeypatch.setenv("IDF_NO_ROW_STAGES", "1")
        net, st, x, out = open_eager(wl, seg)
        seen = []
        for r in range(0, h, seg):
            st.push_segment(x[:, r:r + seg].contiguous())
            if r // seg in (4, 5):
                seen.append(st.read_announced(*out).cpu().numpy())
                check(wl, seen[-1], r + seg, some)
        seen.append(st.read_announced(*out).cpu().numpy())
        check(wl, seen[-1], h, some)
        results.append((seen, [st.get_stats(b)["events_in"].tolist() for b in some]))
        st.close(); net.destroy()
    assert results[0][1] == results[1][1]
    for a, b in zip(results[0][0], results[1][0]):
        assert np.array_equal(a, b)
