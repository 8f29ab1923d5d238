"""Eager emission and graphs: calls recorded in the middle of a sample, with pushes on their way through the stages and without, replayed
more than once, before and after further pushes.  Every read shows the conventional network on the rows pushed by then."""
import numpy as np
import pytest

import oracle
from test_gpu_eager_by_stage import workload as wide_workload
from test_gpu_eager_stages import check, workload

pytestmark = pytest.mark.gpu


class Session:
    def __init__(self, wl, seg=1):
        import torch
        import paper_1804_10727_amd as idf
        self.wl, self.seg, self.at, self.torch = wl, seg, 0, torch
        self.net = idf.net_from_workload(wl)
        self.stream = torch.cuda.Stream()
        n = len(wl["layers"])
        self.shape = list(oracle.layer_shapes(wl["layers"], wl["in_h"], wl["in_w"]))[-1]
        self.level = n
        x = torch.from_numpy(wl["x"]).cuda()
        self.rows = [x[:, r:r + seg].contiguous() for r in range(0, wl["in_h"], seg)]
        torch.cuda.synchronize()
        with torch.cuda.stream(self.stream):
            self.st = idf.Streams(self.net, wl["streams"], max_seg_rows=seg, stream=self.stream)
            self.st.enable_eager()
        self.stream.synchronize()

    def push(self, n=1):
        with self.torch.cuda.stream(self.stream):
            for _ in range(n):
                self.st.push_segment(self.rows[self.at])
                self.at += 1

    def record(self, calls):
        graph = self.torch.cuda.CUDAGraph()
        with self.torch.cuda.graph(graph, stream=self.stream):
            out = calls()
        return graph, out

    def read(self):
        return self.st.read_announced(self.level, self.shape)

    def replay(self, graph):
        with self.torch.cuda.stream(self.stream):
            graph.replay()
        self.stream.synchronize()

    def shows(self, out, rows=None):
        self.stream.synchronize()
        check(self.wl, out.cpu().numpy(), min(self.wl["in_h"], (self.at if rows is None else rows) * self.seg), range(self.wl["streams"]))

    def now(self):
        with self.torch.cuda.stream(self.stream):
            out = self.read()
        self.shows(out)

    def close(self):
        events = [int(self.st.get_stats(b)["events_in"][0]) for b in range(self.wl["streams"])]
        assert events == [np.count_nonzero(self.wl["x"][b, :self.at * self.seg]) for b in range(self.wl["streams"])]
        self.st.close(); self.net.destroy()


NETS = [("i8", 1), ("f32", 1), ("wide", 2), ("half", 1)]          # ("half": two stages of half as many waves)


def session(kind, seg):
    if kind == "wide":
        return Session(wide_workload(30, 97, 3, 3), seg)
    return Session(workload("f32" if kind == "half" else kind, 18, 21, 130 if kind == "half" else 3, 3 if kind == "half" else 6, 5), seg)


@pytest.mark.parametrize("kind,seg", NETS)
def test_a_read_recorded_with_pushes_on_their_way(kind, seg):
    for first in ("replay", "push", "read"):       # what comes next
        s = session(kind, seg)
        s.push(5)
        graph, out = s.record(s.read)
        if first == "push":
            s.push()
        if first == "read":
            s.now()
        for _ in range(3):
            s.replay(graph)
            s.shows(out)
        for _ in range(4):
            s.push()
            s.replay(graph)
            s.shows(out)
        s.push(len(s.rows) - s.at)
        s.replay(graph)
        s.shows(out)
        s.now()
        s.close()


@pytest.mark.parametrize("kind,seg", NETS)
def test_a_read_recorded_before_any_push(kind, seg):
    s = session(kind, seg)
    graph, out = s.record(s.read)
    while s.at < len(s.rows):
        s.push()
        s.replay(graph)
        s.shows(out)
    s.now()
    s.close()


@pytest.mark.parametrize("kind,seg", NETS)
def test_pushes_recorded_behind_pushes_on_their_way(kind, seg):
    s = session(kind, seg)
    s.push(4)

    def calls():
        s.push(3)
        return s.read()
    graph, out = s.record(calls)
    s.replay(graph)
    s.shows(out)
    s.push(2)
    s.now()
    s.push(len(s.rows) - s.at)
    s.now()
    s.close()


def test_two_graphs_recorded_with_the_same_pushes_on_their_way():
    s = session("i8", 1)
    s.push(6)
    a, read_first = s.record(s.read)
    b, read_second = s.record(s.read)
    for graph, out in ((b, read_second), (a, read_first), (b, read_second)):
        s.replay(graph)
        s.shows(out)
    s.push(3)
    s.replay(a)
    s.shows(read_first)
    s.close()
