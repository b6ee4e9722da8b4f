"""The two ways into the entry points that are called once per step -- the extension module and ctypes -- take the same
arguments and return the same codes (host-only trees: every call is refused before it reaches a device)."""
import numpy as np
import pytest

import paper_2508_07014_amd as pb
from paper_2508_07014_amd import binding as B

TREE = dict(tokens=np.array([1, 2, 3], np.int32), offs=np.array([0, 3], np.int64))


class Buffer:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


def _forms():
    lib = pb.load()
    forms = [B._CtypesCalls(lib)]
    try:
        from paper_2508_07014_amd import _pbcall
        forms.append(_pbcall)
    except ImportError:
        pass
    return forms


def test_codes_of_refused_calls():
    tree = pb.pb_build(TREE["tokens"], TREE["offs"], 16, 0, device=-1)
    some = np.zeros(64, np.float32)
    p = Buffer(some.ctypes.data)
    for f in _forms():
        for handle in (tree.handle, None, 0):
            for buf in (p, p.address, np.int64(p.address), None):
                for n in (1, np.int32(1), -1):
                    assert f.pb_score(handle, buf, n, buf, buf, 0) == pb.PB_EINVAL
                    assert f.pb_fuse_step(handle, buf, 16, buf, 0.5, n, buf, buf, buf, 0) == pb.PB_EINVAL
                    assert f.pb_fuse_step_select(handle, buf, 16, buf, None, 1, n, 1, buf, buf, buf, None) == pb.PB_EINVAL
                    assert f.pb_fuse_frames_ws(handle, buf, 16, 16, buf, None, 0.5, n, n, 2, buf, buf, buf, buf, 8, 0) == pb.PB_EINVAL
                    assert f.pb_fuse_step_beam(handle, buf, 16, buf, buf, 0.5, n, 4, buf, buf, buf, buf, 0) == pb.PB_EINVAL
    with pytest.raises(pb.PbError) as e:
        pb.pb_fuse_step(tree, p, 16, p, 0.5, 1, p, p, p)
    assert e.value.code == pb.PB_EINVAL


def test_arguments_of_the_wrong_kind():
    tree = pb.pb_build(TREE["tokens"], TREE["offs"], 16, 0, device=-1)
    for f in _forms():
        with pytest.raises(TypeError):
            f.pb_score(tree.handle, 0, 1)
        with pytest.raises((TypeError, ValueError)):
            f.pb_score(tree.handle, "text", 1, 0, 0, 0)
        with pytest.raises(Exception):
            f.pb_score(tree.handle, 0, 1.5, 0, 0, 0)
        with pytest.raises(Exception):
            f.pb_fuse_step(tree.handle, 0, 16, 0, "half", 1, 0, 0, 0, 0)


class Recorder:
    """Stands in for the library: every entry point records the arguments it is called with."""

    def __init__(self):
        import ctypes as C
        self.calls, self.keep = [], []
        lib = pb.load()
        for name in B.HOT:
            types = getattr(lib, name).argtypes
            fn = C.CFUNCTYPE(C.c_int, *types)(lambda *a, name=name: self.calls.append((name,) + a) or 7)
            fn.argtypes, fn.restype = types, C.c_int
            self.keep.append(fn)
            setattr(self, name, fn)


@pytest.fixture(params=["extension", "ctypes"])
def recorded(request):
    import ctypes as C
    lib = Recorder()
    if request.param == "ctypes":
        yield lib, B._CtypesCalls(lib)
        return
    from paper_2508_07014_amd import _pbcall  # (built with the library, see build.py)
    assert B._hot is None or B._hot is _pbcall
    yield lib, B._bind_hot(lib)
    B._bind_hot(pb.load())


# p: pointer, l: 64-bit, i: 32-bit, f: float -- the C declarations, written out a second time
SIGNATURES = dict(pb_score="ppippp", pb_fuse_step="pplpfipppp", pb_fuse_frames="ppllpfiipppp", pb_fuse_step_select="pplppfiipppp",
                  pb_fuse_frames_select="ppllppfiiipppp", pb_fuse_frames_ws="ppllppfiiippppl" + "p",
                  pb_fuse_frames_static="ppllppfiiipppp", pb_fuse_step_beam="pplppfiippppp", pb_score_forest="pppippp",
                  pb_fuse_step_forest="pplpppfiipppp", pb_fuse_frames_forest="ppllpppfiiipppp",
                  pb_fuse_step_beam_forest="pplpppfiippppp")


def _arguments(sig, forms, none=False):
    """(arguments, what the library must see), every one another value."""
    given, seen = [], []
    for k, t in enumerate(sig):
        edge = k in (0, len(sig) - 1)  # the handle and the stream are not device buffers
        if t == "p":
            v = 0x7f0000001000 + 0x10000 * k
            given.append(None if none else v if edge and forms != "ctypes" else forms_of(forms, "p", v, edge))
            seen.append(None if none else v)
        elif t == "l":
            v = (1 << 33) + 7 * k
            given.append(forms_of(forms, "l", v, edge))
            seen.append(v)
        elif t == "i":
            v = -(3 + k)
            given.append(forms_of(forms, "i", v, edge))
            seen.append(v)
        else:
            given.append(forms_of(forms, "f", 0.375 + k, edge))
            seen.append(0.375 + k)
    return given, tuple(seen)


def forms_of(forms, t, v, edge):
    import ctypes as C
    if forms == "plain" or (t != "p" and forms == "buffers"):
        return v
    if forms == "buffers":
        return Buffer(v)
    if forms == "numpy":  # (device buffers and numbers as numpy scalars)
        return {"p": np.uint64, "l": np.int64, "i": np.int32, "f": np.float32}[t](v)
    if t == "p" and not edge:
        return v  # (a ctypes pointer was never a device buffer)
    return {"p": C.c_void_p, "l": C.c_int64, "i": C.c_int32, "f": C.c_float}[t](v)


@pytest.mark.parametrize("forms", ["plain", "buffers", "numpy", "ctypes"])
def test_every_argument_arrives_as_it_is(recorded, forms):
    lib, calls = recorded
    assert sorted(SIGNATURES) == sorted(B.HOT)
    for name, sig in SIGNATURES.items():
        for none in (False, True):
            given, seen = _arguments(sig, forms, none)
            lib.calls.clear()
            assert getattr(calls, name)(*given) == 7
            assert lib.calls == [(name,) + seen], name


def test_integers_wrap_and_buffers_fail_as_ctypes_has_it(recorded):
    import ctypes as C
    lib, calls = recorded
    calls.pb_score(1 << 64 | 5, 3, (1 << 32) + 9, True, 2, 0)
    assert lib.calls == [("pb_score", 5, 3, 9, 1, 2, None)]
    for bad in ((0, 1, 1.5, 0, 0, 0), (0, 1, 1, 0, 0, 1.5), (0, 1, "1", 0, 0, 0)):
        with pytest.raises(C.ArgumentError):
            calls.pb_score(*bad)
    with pytest.raises((TypeError, ValueError)):   # device buffers: int() is asked
        calls.pb_score(0, C.c_void_p(5), 1, 0, 0, 0)
    with pytest.raises(ValueError):
        calls.pb_score(0, "text", 1, 0, 0, 0)

    class Broken:
        def data_ptr(self):
            raise RuntimeError("no storage")
    with pytest.raises(RuntimeError, match="no storage"):
        calls.pb_score(0, Broken(), 1, 0, 0, 0)


def test_stream_and_numbers_as_ctypes_objects():
    """What a program with its own ctypes bindings of the runtime holds: a stream handle as c_void_p, sizes as c_int32."""
    import ctypes as C
    tree = pb.pb_build(TREE["tokens"], TREE["offs"], 16, 0, device=-1)
    p = Buffer(np.zeros(64, np.float32).ctypes.data)
    for stream in (C.c_void_p(64), C.c_void_p(), None, 0):
        with pytest.raises(pb.PbError) as e:
            pb.pb_fuse_step(tree, p, C.c_int64(16), p, C.c_float(0.5), C.c_int32(1), p, p, p, stream)
        assert e.value.code == pb.PB_EINVAL
