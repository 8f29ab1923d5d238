"""Pushes go into the library by csrc/push.cpp: what it hands over is what the conversion by ctypes hands over, for every form of the
arguments; what it does not take goes that way, and raises what it raised."""
import ctypes as C
import os

import numpy as np
import pytest
import torch

import paper_1804_10727_amd as idf
from paper_1804_10727_amd import binding

_FN = C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_int)


class Recorder:
    """Stands in for the library: takes down the call."""

    def __init__(self, monkeypatch):
        binding.load_push()
        from paper_1804_10727_amd import _push as native
        self.calls = []

        def seen(streams, ids, n_ids, rows, n_rows):
            got = None if not ids else list((C.c_int32 * n_ids).from_address(ids))
            self.calls.append((streams, got, n_ids, rows, n_rows))
            return 0
        self.fn, self.native = _FN(seen), native
        self.real = C.cast(binding._LIB.idf_push_segment, C.c_void_p).value
        native.bind(C.cast(self.fn, C.c_void_p).value)

        class Lib:
            @staticmethod
            def idf_push_segment(h, ids, n_ids, rows, n_rows):
                return self.fn(h, None if ids is None else C.cast(C.c_char_p(ids), C.c_void_p), n_ids, rows, n_rows)
        self.lib = Lib

    def close(self):
        self.native.bind(self.real)


@pytest.fixture
def recorder(monkeypatch):
    r = Recorder(monkeypatch)
    yield r
    r.close()


def _streams():
    binding.load_push()
    s = object.__new__(idf.Streams)
    s._h, s._address = C.c_void_p(4096), 4096
    return s


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.int8])
@pytest.mark.parametrize("ids", [None, [2], [3, 0, 1], (1,), np.array([5, 4], dtype=np.int32), np.array([5, 4], dtype=np.int64),
                                 np.arange(10, dtype=np.int32)[::3], np.arange(100, dtype=np.int32), np.zeros(0, dtype=np.int32),
                                 np.array([7], dtype=np.uint32), torch.tensor([1, 2], dtype=torch.int32)],
                         ids=["none", "list1", "list3", "tuple", "int32", "int64", "strided", "many", "empty", "uint32", "tensor"])
@pytest.mark.parametrize("n_rows", [None, 1, np.int64(2), 2 ** 31])
def test_hands_over_what_the_conversion_does(recorder, monkeypatch, dtype, ids, n_rows):
    n = 4 if ids is None else len(ids)
    rows = torch.zeros((n, 3, 5, 2), dtype=dtype, device="cuda:0")
    s = _streams()

    def outcome(f):
        recorder.calls.clear()
        try:
            f()
        except Exception as e:
            return type(e)
        return list(recorder.calls)
    monkeypatch.setattr(binding, "_LIB", recorder.lib)
    want = outcome(lambda: s._push_converted(rows, ids, n_rows))
    assert outcome(lambda: s.push_segment(rows, ids, n_rows)) == want
    assert outcome(lambda: s.push_segment(rows=rows, stream_ids=ids, n_rows=n_rows)) == want


@pytest.mark.gpu
def test_tensors_without_contiguous_memory_are_refused():
    s = _streams()
    rows = torch.zeros((4, 3, 5, 2), device="cuda:0")
    for bad in (rows[:, ::2], rows.transpose(0, 1), rows.cpu()):
        with pytest.raises(AssertionError):
            s.push_segment(bad)
    with pytest.raises(IndexError):
        s.push_segment(rows[0, 0, 0].contiguous())
    with pytest.raises(idf.IdfError):
        s._h, s._address = None, 0
        s.push_segment(rows)


def test_what_is_no_plain_tensor_goes_the_long_way():
    binding.load_push()
    s = _streams()
    with pytest.raises(AssertionError):
        s.push_segment(torch.zeros((1, 1, 1, 1)))
    with pytest.raises(AttributeError):
        s.push_segment(np.zeros((1, 1, 1, 1), dtype=np.float32))
    assert binding._push(0, None, None, None) is None
    with pytest.raises(TypeError):
        binding._push(0, None)


def test_the_module_is_of_this_interpreter_and_torch(monkeypatch):
    """Another torch's or interpreter's module has another name; where this one's is absent it is built, and nothing else."""
    import shutil
    import sys
    import sysconfig
    from paper_1804_10727_amd import build
    binding.load_push()
    from paper_1804_10727_amd import _push as native
    monkeypatch.setitem(sys.modules, native.__name__, native)          # (both are as they were behind this test)
    monkeypatch.setattr(idf, "_push", native)
    path = build.push_path()
    assert path.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and torch.__version__ in path
    monkeypatch.setattr(torch, "__version__", "0.0.0+another")
    other = build.push_path()
    assert other != path and not build.up_to_date()
    built = []

    def build_push():
        built.append(build.push_path())
        shutil.copy(path, other)                   # (this torch's, in place of one that cannot be built here)
    monkeypatch.setattr(build, "build_push", build_push)
    for name in ("build", "build_library"):
        monkeypatch.setattr(build, name, lambda *a, **k: pytest.fail("the library is there"))
    monkeypatch.setattr(binding, "_push", None)
    try:
        monkeypatch.setattr(binding, "_LIB", None)
        binding.load_library()                     # the library alone asks for no module
        assert not built
        binding.load_push()
        assert built == [other]
    finally:
        if os.path.exists(other):
            os.remove(other)
