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
