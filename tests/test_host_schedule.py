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


# ---- a launch that cannot be enqueued ---------------------------------------------------------------------------
def failed_launch(rt, net_args, streams, seg, fail_at, apart):
    """Every push is tried with a failing launch; what it says it has taken in is not pushed again."""
    import ctypes as C
    from paper_1804_10727_amd import IdfError
    h = net_args[1]
    net = chain(*net_args)
    st = host_runtime.Streams(net, streams, seg)

    def rows(i):
        r = C.c_int64()
        st.check(st.L.idf_rows_pushed(st.h, i, C.byref(r)))
        return r.value
    rt.host_begin()
    for ids in [[i] for i in range(streams)] if apart else [None]:
        of, r, failures = (ids or [0])[0], 0, 0
        while True:
            rt.host_fail_in(fail_at)
            before = r
            try:
                st.push(min(seg, h - r), ids)
            except IdfError as e:
                assert e.code == -4
                failures += 1
            rt.host_fail_in(-1)
            r = rows(of)
            if r == before:                            # nothing went in: at least the next push has to go well
                st.push(1, ids)
                r = rows(of)
            if r == 0:                                 # the sample is complete
                break
        assert failures > 0
    assert (st.read(h) == int(net.query_sizes(1, seg).out_h)).all()
    assert rt.host_error() == b"", rt.host_error()
    st.close()


@pytest.mark.parametrize("fail_at", [0, 1, 2])
@pytest.mark.parametrize("apart", [False, True])
def test_rows_go_in_once_when_a_launch_fails(runtime, fail_at, apart):
    host_runtime.run(runtime, "test_host_schedule", "failed_launch", ("f32", 64, 20, [3, 32, 32, 64, 64], (1,)), 3, 40, fail_at, apart)


# ---- pushes of more rows than a launch has tiles for ---------------------------------------------------------------
def mixed(prec, h, w, channels, pools=(), last_1x1=True):
    """The same with a 1x1 layer behind, or in front: the layers go one after the other."""
    import paper_1804_10727_amd as idf
    from workloads import conv, maxpool
    dt = {"f32": np.float32, "bf16": np.uint16}[prec]
    layers, weights = [], []
    for i, (a, b) in enumerate(zip(channels, channels[1:])):
        k = 1 if i == (len(channels) - 2 if last_1x1 else 0) else 3
        layers.append(conv(a, b, k, k, p_h=k // 2, p_w=k // 2))
        weights.append(np.ones((b, a, k, k), dt))
        if i in pools:
            layers.append(maxpool(b))
            weights.append(None)
    return idf.Net(prec, h, w, channels[0], layers, weights)


def long_push(rt, kind, net_args, seg):
    net = (chain if kind == "chain" else mixed)(*net_args)
    h = net_args[1]
    st = host_runtime.Streams(net, 1, seg)
    rt.host_begin()
    for _ in range(2):
        for r in range(0, h, seg):
            st.push(min(seg, h - r))
        st.read(h)
    assert rt.host_error() == b"", rt.host_error()
    st.close()


@pytest.mark.parametrize("kind,net_args,seg", [
    ("mixed", ("f32", 1080, 3840, [3, 64, 64, 16]), 1080),
    ("mixed", ("f32", 1080, 3840, [3, 64, 64, 16], (0,)), 1080),
    ("mixed", ("f32", 1081, 3840, [3, 64, 64, 16], (1,)), 700),
    ("mixed", ("f32", 512, 1920, [3, 256, 256, 16]), 512),
    ("mixed", ("f32", 70001, 40, [3, 16, 16]), 70001),                # (more rows taken than a launch has tiles)
    ("mixed", ("bf16", 1080, 3840, [8, 64, 128, 16], (), False), 1080),
    ("chain", ("f32", 64, 60000, [3, 256, 256], (0,)), 64),
    ("mixed", ("bf16", 1200, 7680, [256, 256, 256, 16]), 1200),       # (streams 2^31 elements apart, in the rings and in the buffer)
])
def test_long_pushes_are_several_launches(runtime, kind, net_args, seg):
    host_runtime.run(runtime, "test_host_schedule", "long_push", kind, net_args, seg)


# ---- workspaces that do not hold the fastest layout ----------------------------------------------------------------
def small_workspace(rt, kind, net_args, streams, seg):
    """From the workspace of idf_query_sizes down to the smallest that is accepted: every row still goes where it should."""
    import random
    from paper_1804_10727_amd import IdfError
    h, w = net_args[1], net_args[2]
    net = (chain if kind == "chain" else mixed)(*net_args)
    size = net.query_sizes(streams, seg).workspace_bytes
    opened = 0
    while True:
        try:
            st = host_runtime.Streams(net, streams, seg, workspace_bytes=size)
        except IdfError as e:
            assert e.code == -1
            break
        opened += 1
        for way in ("together", "apart", "pixels"):
            rng = random.Random(way)
            rt.host_begin()
            st.check(st.L.idf_reset_streams(st.h, None, streams))
            rows = [0] * streams                       # of two samples, one after the other
            while min(rows) < 2 * h:
                ids = list(range(streams)) if way == "together" else [rng.choice([i for i in range(streams) if rows[i] < 2 * h])]
                n = min(rng.randint(1, seg), h - rows[ids[0]] % h)
                if way == "pixels" and n == 1:
                    cut = rng.randint(1, w - 1)
                    st.push_pixels(0, cut, ids)
                    st.push_pixels(cut, w - cut, ids)
                else:
                    st.push(n, ids)
                for i in ids:
                    rows[i] += n
                if rng.random() < 0.1:
                    st.stats(0)
                if rows[ids[0]] % h == 0 or rng.random() < 0.1:
                    st.read(h)
            assert rt.host_error() == b"", (way, size, opened, rt.host_error())
        st.close()
        size -= max(256, size // 20)
    assert opened >= 2
    net.destroy()


@pytest.mark.parametrize("kind,net_args,streams,seg", [
    ("chain", ("f32", 32, 32, [3, 32, 32, 64, 64], (1,)), 3, 8),
    ("chain", ("f32", 31, 32, [3, 32, 32, 64, 64], (1,)), 2, 16),
    ("chain", ("bf16", 45, 33, [3, 64, 64, 128, 128, 64], (0, 2)), 2, 16),
    ("chain", ("bf16", 38, 40, [64, 16, 64, 16], ()), 2, 1),
    ("chain", ("i8", 50, 48, [1, 16, 16, 32, 32, 64, 64, 64, 64], (1, 3, 5)), 2, 20),
    ("chain", ("f32", 43, 20, [3, 16, 16], (0, 1)), 2, 5),
    ("mixed", ("f32", 33, 32, [3, 32, 64, 16], (0,)), 2, 8),
    ("mixed", ("bf16", 34, 32, [8, 64, 32, 64], (1,), False), 2, 16),
])
def test_small_workspaces_hold_the_same_schedule(runtime, kind, net_args, streams, seg):
    host_runtime.run(runtime, "test_host_schedule", "small_workspace", kind, net_args, streams, seg)


def capacity(rt):
    """Streams of a net whose layers keep rows of c and the rows of one push (four bytes and an event each) within the library's
    own workspace: as many of them open as did when that was what layers kept."""
    for net_args, seg, streams in [(("f32", 32, 32, [3, 32, 32, 64, 64], (1,)), 8, 160), (("f32", 32, 32, [3, 32, 32, 64, 64], (1,)), 16, 132),
                                   (("f32", 48, 47, [3, 32, 32, 64, 64], (1,)), 8, 95), (("f32", 48, 47, [3, 32, 32, 64, 64], (1,)), 16, 80),
                                   (("bf16", 112, 112, [3, 64, 64, 128, 128, 256, 256, 256], (1, 3)), 16, 12),
                                   (("f32", 64, 64, [64, 16], ()), 1, 121)]:
        net = chain(*net_args)
        st = host_runtime.Streams(net, streams, seg, static=True)
        st.close()
        net.destroy()


def test_as_many_streams_as_before_open_in_the_static_workspace(runtime):
    host_runtime.run(runtime, "test_host_schedule", "capacity")


# ---- held-back pushes ------------------------------------------------------------------------------------------------
def batching(rt, when):
    from workloads import make
    import paper_1804_10727_amd as idf
    net = idf.net_from_workload(make(2, streams=4, length=1600))
    st = host_runtime.Streams(net, 4, 16)
    for _ in range(when):
        st.push(16)
    st.check(st.L.idf_set_push_batching(st.h, 16))
    rt.host_begin()
    for _ in range(32):
        st.push(16)
    assert rt.host_launches(b"k_conv_gather") == 2, rt.host_launches(b"k_conv_gather")
    st.close()


@pytest.mark.parametrize("when", [0, 1, 20])
def test_pushes_are_held_back_from_whenever_it_is_asked_for(runtime, when):
    host_runtime.run(runtime, "test_host_schedule", "batching", when)


# ---- which kernels serve a net -----------------------------------------------------------------------------------------
def finite_weights(rt):
    """A net of several kinds of layers goes through the gathering kernel, which multiplies zeros, if all its weights are finite."""
    import paper_1804_10727_amd as idf
    from workloads import conv
    layers = [conv(3, 32, 5, 5, p_h=2, p_w=2), conv(32, 33, 3, 3, p_h=1, p_w=1)]
    for prec, bad in (("f32", [np.inf, -np.inf, np.nan]), ("bf16", [0x7F80, 0xFF80, 0x7FC1, 0xFF81])):
        dt = np.float32 if prec == "f32" else np.uint16
        largest = np.finfo(np.float32).max if prec == "f32" else 0x7F7F
        for value, at in [(largest, 0)] + [(v, i) for v in bad for i in (0, 1, 9503)]:
            w = [np.full((L["c_out"], L["c_in"], L["k_h"], L["k_w"]), 1, dt) for L in layers]
            w[1].reshape(-1)[at] = value
            net = idf.Net(prec, 32, 32, 3, layers, w)
            st = host_runtime.Streams(net, 2)
            assert st.L.idf_layer_kernel(st.h, 1) == (b"conv_gather" if value == largest else b"conv_generic"), (prec, value, at)
            st.close()
            net.destroy()


def test_infinite_weights_stay_off_the_gathering_kernel(runtime):
    host_runtime.run(runtime, "test_host_schedule", "finite_weights")


def depth_first(rt):
    """IDF_CASCADE_STAGES=1 counts when streams are opened: theirs are launches of all layers, one after the other."""
    import os
    from workloads import make
    import paper_1804_10727_amd as idf
    net = idf.net_from_workload(make(2, streams=4, length=1600))
    for strict in (True, False):
        os.environ["IDF_CASCADE_STAGES"] = "1" if strict else "2"
        st = host_runtime.Streams(net, 4, 16)
        os.environ["IDF_CASCADE_STAGES"] = "2" if strict else "1"
        rt.host_begin()
        for _ in range(10):
            st.push(16)
        assert (rt.host_launches(b"k_conv_gather_chain"), rt.host_launches(b"k_conv_gather_rows")) == ((10, 0) if strict else (0, 10))
        st.close()


def test_streams_keep_the_mode_they_were_opened_in(runtime):
    host_runtime.run(runtime, "test_host_schedule", "depth_first")


# ---- dynamic LDS beyond 64 KB ------------------------------------------------------------------------------------------
def large_lds(rt, kind, precs, kernels):
    """One process launches the variants of a kernel one after the other: each has asked for its LDS itself."""
    import ctypes as C
    rt.host_begin()
    for prec in precs:
        if kind == "eager":
            cases = [(64, 2, w, [16, 64, 64]) for w in (62, 130, 200)]
        else:                                      # (whole K-steps and not; of few streams and of many; narrow tiles and wide ones)
            c = {"f32": 132, "bf16": 248, "i8": 512}[prec]
            cases = [(streams, seg, 400, channels) for channels in ([c, 16, 16], [256, 64, 64]) for streams in (2, 64) for seg in (1, 8)]
        for streams, seg, w, channels in cases:
            net = chain(prec, 16, w, channels)
            st = host_runtime.Streams(net, streams, seg)
            if kind == "eager":
                nb = C.c_size_t()
                st.check(st.L.idf_query_eager_bytes(net._h, streams, seg, C.byref(nb)))
                st.check(st.L.idf_enable_eager(st.h, C.c_void_p(1 << 42), nb))
            for r in range(0, 16, seg):
                st.push(min(seg, 16 - r))
            st.close()
            net.destroy()
    assert rt.host_error() == b"", rt.host_error()
    assert rt.host_large_kernels() >= kernels, rt.host_large_kernels()


@pytest.mark.parametrize("kind,precs,kernels", [("rows", ("f32",), 2), ("rows", ("bf16",), 3), ("rows", ("i8",), 2), ("eager", ("f32", "i8"), 2)])
def test_every_kernel_asks_for_its_lds(runtime, kind, precs, kernels):
    host_runtime.run(runtime, "test_host_schedule", "large_lds", kind, precs, kernels)


# ---- tiles of the gathering kernel ----------------------------------------------------------------------------------------
def wide_tiles(rt, channels, streams, wide, strides=()):
    """Held-back pushes of 256 rows in all: single tiles or two by two."""
    import paper_1804_10727_amd as idf
    from workloads import conv
    layers = [conv(a, b, 9, 1, s=2 if i in strides else 1) for i, (a, b) in enumerate(zip(channels, channels[1:]))]
    net = idf.Net("f32", 4096, 1, 1, layers, [np.ones((L["c_out"], L["c_in"], 9, 1), np.float32) for L in layers])
    st = host_runtime.Streams(net, streams, 16)
    st.check(st.L.idf_set_push_batching(st.h, 16))
    rt.host_begin()
    for _ in range(256):
        st.push(16)
    assert rt.host_launches(b"k_conv_gather_rows") == 16
    assert (rt.host_launches(b"k_conv_gather_rowsINS0_9TraitsF32ELi9ELb0ELb1EE") > 0) == wide
    st.close()


@pytest.mark.parametrize("channels,streams,wide", [
    ((1, 8, 8, 8), 64, False), ((1, 16, 16, 16, 16), 64, False),                       # 3,072 and 4,096 tiles, none that could go two by two
    ((1, 16, 16, 16, 16, 32), 15, False), ((1, 16, 16, 16, 16, 32), 16, True),         # 96 tiles per stream, 32 of them could
    ((1, 16, 16, 16, 16, 16, 16, 32), 11, False), ((1, 16, 16, 16, 16, 16, 16, 32), 12, True),     # 128 and 32
    ((1, 32, 64, 64), 9, False), ((1, 32, 64, 64), 10, True),                          # 160, all
])
def test_tiles_go_two_by_two_where_many_can(runtime, channels, streams, wide):
    host_runtime.run(runtime, "test_host_schedule", "wide_tiles", channels, streams, wide)


@pytest.mark.parametrize("channels,strides,wide", [
    ((1, 16, 16, 16, 16, 32, 16), (4,), True),                  # 16 of 88 tiles per stream
    ((1, 16, 16, 16, 16, 16, 16, 32), (5, 6), True),            # 8 of 96
    ((1, 16, 16, 16, 16, 16, 16, 32), (4, 5, 6), False),        # 4 of 80
])
def test_tiles_stay_single_where_few_can_go_two_by_two(runtime, channels, strides, wide):
    host_runtime.run(runtime, "test_host_schedule", "wide_tiles", channels, 64, wide, strides)


# ---- windows of many cells ----------------------------------------------------------------------------------------------
def large_windows(rt):
    """The gathering kernel counts a window's cells in 32 bits; only where a row is one position it divides by a multiplication of 16."""
    import paper_1804_10727_amd as idf
    from workloads import conv
    for w, c_in, k_h, k_w, kernel in [(32, 192, 7, 7, b"conv_gather"), (32, 248, 9, 2, b"conv_gather"), (32, 256, 32, 32, b"conv_gather"), (32, 201, 32, 31, b"conv_gather"),
                                      (32, 257, 7, 7, b"conv_generic"), (33, 16, 33, 1, b"conv_generic"),
                                      (2, 248, 18, 1, b"conv_gather"), (1, 248, 17, 1, b"conv_gather"), (1, 248, 18, 1, b"conv_generic")]:
        net = idf.Net("f32", 40, w, c_in, [conv(c_in, 16, k_h, k_w)], [np.ones((16, c_in, k_h, k_w), np.float32)])
        st = host_runtime.Streams(net, 1)
        assert st.L.idf_layer_kernel(st.h, 0) == kernel, (w, c_in, k_h, k_w)
        st.close()
        net.destroy()


def test_which_windows_the_gathering_kernel_takes(runtime):
    host_runtime.run(runtime, "test_host_schedule", "large_windows")


def test_division_of_a_window_into_rows_is_exact():
    """ceil(2^32 / n) for windows of up to 32 x 32 positions of 64 cells, and the cells that the last K-step reads too far."""
    q = np.arange(32 * 2048 + 4, dtype=np.uint64)
    for n in sorted({k_w * cells for k_w in range(1, 33) for cells in range(1, 65)} - {1}):
        few = q[:32 * n + 4]
        assert np.array_equal(few * np.uint64(-(-2**32 // n)) >> np.uint64(32), few // np.uint64(n)), n


# ---- eager emission in stages -----------------------------------------------------------------------------------------------
def enable_eager(st, net, streams, seg):
    import ctypes as C
    nb = C.c_size_t()
    st.check(st.L.idf_query_eager_bytes(net._h, streams, seg, C.byref(nb)))
    st.check(st.L.idf_enable_eager(st.h, C.c_void_p(1 << 42), nb))


def eager_reads(rt, prec, h, w, channels, pools, streams, seg, every, staged):
    """Reads after every so many pushes, or at the end of the sample (0): a launch per push, or more where the pushes go in stages."""
    import ctypes as C
    net = chain(prec, h, w, channels, pools)
    n_layers = len(channels) - 1 + len(pools)
    st = host_runtime.Streams(net, streams, seg)
    enable_eager(st, net, streams, seg)
    pushes = -(-h // seg)
    for sample in range(4):                        # (the first reads are what later pushes go by)
        rt.host_begin()
        for i in range(pushes):
            st.push(min(seg, h - i * seg))
            if (every and (i + 1) % every == 0) or i + 1 == pushes:
                st.check(st.L.idf_read_announced(st.h, n_layers, None, streams, C.c_void_p(1 << 51)))
    assert (rt.host_launches(b"k_eager_pass") > pushes) == staged, (rt.host_launches(b"k_eager_pass"), pushes)
    assert rt.host_error() == b"", rt.host_error()
    st.close()
    net.destroy()


EVENTS, EVENTS_POOLS = [1, 16, 16, 32, 32, 64, 64, 64, 64], (1, 3, 5)
SMALL = [3, 32, 32, 64, 64]


@pytest.mark.parametrize("prec,h,w,channels,pools,streams,seg,every,staged", [
    ("i8", 60, 60, EVENTS, EVENTS_POOLS, 16, 1, 1, False), ("i8", 60, 60, EVENTS, EVENTS_POOLS, 16, 1, 2, False),
    ("i8", 60, 60, EVENTS, EVENTS_POOLS, 16, 1, 3, True), ("i8", 60, 60, EVENTS, EVENTS_POOLS, 16, 1, 0, True),
    ("i8", 112, 112, EVENTS, EVENTS_POOLS, 8, 1, 2, True),                       # stages of many multiply-adds
    ("f32", 32, 32, SMALL, (1,), 64, 1, 1, False), ("f32", 32, 32, SMALL, (1,), 64, 1, 2, True),
    ("f32", 30, 20, [3, 16, 16], (), 4, 1, 3, False), ("f32", 30, 20, [3, 16, 16], (), 4, 1, 5, True),
    ("f32", 32, 32, SMALL, (1,), 256, 1, 4, False), ("f32", 32, 32, SMALL, (1,), 256, 1, 8, True),          # two workgroups to a compute unit
    ("f32", 15, 32, SMALL, (1,), 256, 3, 0, False), ("f32", 18, 32, SMALL, (1,), 256, 3, 0, True),          # samples of five and of six pushes
    ("f32", 24, 40, SMALL, (1,), 140, 2, 6, False), ("f32", 24, 40, SMALL, (1,), 140, 2, 0, True),
    ("f32", 48, 24, [3, 16, 16, 64, 64], (), 140, 1, 0, False),                  # one stage would have most of the work
    ("i8", 48, 24, [1, 16, 32, 32], (), 200, 1, 0, True),                        # little work anywhere
    ("i8", 26, 16, [2, 16, 32, 16, 48, 16], (0, 3), 256, 1, 0, True), ("f32", 23, 17, [2, 16, 32, 16, 48], (0,), 130, 1, 0, True),
    ("f32", 17, 20, [2, 16, 32, 16, 48], (0,), 201, 1, 0, True), ("i8", 25, 33, [2, 16, 32, 16, 48, 16, 16, 32], (0, 3), 140, 2, 0, True),
])
def test_pushes_go_in_stages_where_the_reads_leave_enough_of_them(runtime, prec, h, w, channels, pools, streams, seg, every, staged):
    host_runtime.run(runtime, "test_host_schedule", "eager_reads", prec, h, w, channels, pools, streams, seg, every, staged)


def eager_history(rt):
    """What was read push by push before is in stages again after a row of pushes, and at once after two; counters and pushes of some
    streams count as reads do."""
    import ctypes as C
    net = chain("i8", 112, 30, EVENTS, EVENTS_POOLS)
    st = host_runtime.Streams(net, 3)
    enable_eager(st, net, 3, 1)

    def read():
        st.check(st.L.idf_read_announced(st.h, len(EVENTS) + 2, None, 3, C.c_void_p(1 << 51)))

    def launches(n, after):                        # of n pushes and whatever comes after them
        rt.host_begin()
        for _ in range(n):
            st.push(1)
        after()
        return rt.host_launches(b"k_eager_pass")
    assert launches(1, read) == 8 and launches(1, read) == launches(1, read) == 1
    assert launches(20, read) == 6 + 14 + 7        # six by themselves, the others in stages
    assert launches(20, read) == 1 + 5 + 14 + 7    # (one of the last two reads came after a single push)
    assert launches(20, read) == 20 + 7
    for _ in range(2):
        launches(1, lambda: st.stats(0))
    assert launches(1, lambda: st.stats(0)) == 1
    st.check(st.L.idf_reset_streams(st.h, None, 3))
    for _ in range(2):
        launches(6, read)
    for _ in range(2):                             # pushes of some streams and of all in turn
        launches(1, lambda: [st.push(1, [i]) for i in range(3)])
    assert launches(1, lambda: [st.push(1, [i]) for i in range(3)]) == 1 + 3
    st.close()
    net.destroy()


def test_what_pushes_in_stages_go_by(runtime):
    host_runtime.run(runtime, "test_host_schedule", "eager_history")


def eager_lds(rt, prec, h, w, channels, pools, streams, seg):
    """The largest LDS of a launch: stages of one layer that several workgroups share, and the whole net in one workgroup."""
    import os
    lds = []
    for plain in (False, True):
        if plain:
            os.environ["IDF_NO_ROW_STAGES"] = "1"
        net = chain(prec, h, w, channels, pools)
        st = host_runtime.Streams(net, streams, seg)
        enable_eager(st, net, streams, seg)
        rt.host_begin()
        for r in range(0, h, seg):
            st.push(min(seg, h - r))
        assert rt.host_error() == b"", rt.host_error()
        assert rt.host_launches(b"k_eager_pass") > 0
        lds.append(rt.host_max_lds())
        st.close()
        net.destroy()
    assert lds[0] <= 0.8 * lds[1], lds                 # a band, and not the band in front and the one behind


@pytest.mark.parametrize("prec,h,w,channels,pools,streams,seg", [("i8", 40, 112, EVENTS, EVENTS_POOLS, 8, 1), ("f32", 20, 60, SMALL, (1,), 64, 1)])
def test_a_shared_stage_asks_for_its_band_only(runtime, prec, h, w, channels, pools, streams, seg):
    host_runtime.run(runtime, "test_host_schedule", "eager_lds", prec, h, w, channels, pools, streams, seg)


# ---- windows by way of LDS --------------------------------------------------------------------------------------------------
def staged_windows(rt, chans, k, strides, pad, seg, streams):
    import paper_1804_10727_amd as idf
    from workloads import conv
    h, n = 150, len(strides)
    layers = [conv(chans[i], chans[i + 1], k, 1, s=strides[i], p_h=pad) for i in range(n)]
    net = idf.Net("f32", h, 1, chans[0], layers, [np.ones((L["c_out"], L["c_in"], k, 1), np.float32) for L in layers])
    for b in (streams, 3):
        st = host_runtime.Streams(net, b, seg)
        rt.host_begin()
        for r in range(0, h, seg):
            st.push(min(seg, h - r))
        assert (rt.host_launches(b"k_conv_gather_rows_staged") >= 3) == (b == streams), (b, rt.host_launches(b"k_conv_gather_rows_staged"))
        st.close()
    net.destroy()


def test_windows_go_through_lds_where_tiles_are_many(runtime):
    from test_gpu_gather_lds import CASES
    for case in CASES:
        host_runtime.run(runtime, "test_host_schedule", "staged_windows", *case)


# ---- eager emission recorded into a graph -----------------------------------------------------------------------------------
def eager_recorded(rt):
    """What is on its way goes into every graph once, by launches that look whether it is still to be done, and through once more, by the
    same kind, with the next call that is not recorded.  Pushes go through all layers at once from then on."""
    import ctypes as C
    net = chain("i8", 112, 30, EVENTS, EVENTS_POOLS)
    st = host_runtime.Streams(net, 3)
    enable_eager(st, net, 3, 1)

    def read():
        st.check(st.L.idf_read_announced(st.h, len(EVENTS) + 2, None, 3, C.c_void_p(1 << 51)))

    def launches(*calls):
        rt.host_begin()
        for f in calls:
            f()
        return rt.host_launches(b"k_eager_passINS0_8TraitsI8ELi4ELb1ELb1ELb1EE"), rt.host_launches(b"k_eager_pass"), rt.host_launches(b"k_fill")

    def push():
        st.push(1)
    assert launches(*[push] * 10)[:2] == (0, 10)
    for graph in (7, 8):
        rt.host_record(graph)
        assert launches(push, push, read, push) == (7, 7 + 3, 1)
    rt.host_record(0)
    assert launches(read) == (7, 7, 1)
    assert launches(read) == (0, 0, 0)
    assert launches(*[push] * 20, read) == (0, 20, 0)
    st.close()
    net.destroy()


def test_recorded_calls_bring_through_what_is_on_its_way(runtime):
    host_runtime.run(runtime, "test_host_schedule", "eager_recorded")
