"""GPU parity of the wave kernels on rows of any length and alignment: vocabularies that are no multiple of 4, rows
that start 4, 8 or 12 bytes off a 16-byte boundary, the edges of the row shapes (a wave's 1024 and 1280 positions, whole
and partial chunks), blank and EOS in the last tokens (behind the last whole group), exact ties and rows of -inf.  Every
output against the CPU oracle: ids bit-exact, scores within 1e-5.  (From 257 tokens on, under the CTC rule from 128, the
multi-frame calls here are short enough for the two-pass decoder; test_gpu_segments has the longer ones.)"""
import numpy as np
import pytest

import pb_workloads as W
from oracle import OracleTree

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, TOL, dev  # noqa: E402


def _tree(rng, V, blank, eos, wmode, unk):
    n, hi = int(rng.integers(1, 400)), int(rng.integers(2, 8))
    ids = np.array([v for v in range(V) if v not in (blank, eos)], dtype=np.int32)
    lens = rng.integers(1, hi + 1, n)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    # Zipf from both ends of the vocabulary: the last tokens (a group that straddles the end) are common ones
    at = np.minimum(rng.zipf(1.3, int(offs[-1])) - 1, len(ids) - 1)
    at = np.where(rng.random(len(at)) < 0.5, at, len(ids) - 1 - at)
    toks = ids[at]
    ot = OracleTree(toks, offs, V, blank, weight_mode=wmode, unk_score=unk, eos_id=eos, final_eos_score=0.75)
    tr = pb.pb_build(toks, offs, V, blank, device=0, weight_mode=wmode, unk_score=unk, eos_id=eos, final_eos_score=0.75)
    return toks, offs, ot, tr


def _rows(rng, T, B, V, blank, toks, offs):
    kind = int(rng.integers(0, 4))
    if kind == 0:
        x = W.sticky_logp(int(rng.integers(1 << 30)), T, B, V, blank, grid=None, bump=float(rng.choice([3.0, 8.0])))
    elif kind == 1:
        shape = W.Config(9, "ragged", V, blank, 1, 1, 8, "uniform", 1.1, B, 1, T, 2.0)
        x = W.make_logp(shape, seed=int(rng.integers(1 << 30)), planting=W.Planting(toks, offs, cover=0.5, bump=10.0))
    else:
        x = np.round(rng.standard_normal((T, B, V)) * 2).astype(np.float32)   # many exact ties
        x[..., -3:] += (rng.random((T, B, min(V, 3))) < 0.3) * 8.0            # winners in the last tokens
        x[rng.random((T, B)) < 0.1] = -np.inf                                 # whole rows of -inf
    return x.astype(np.float32)


def _on_device(x, stride, shift):
    """Rows of x [T, B, V] on the device with a row stride and `shift` floats in front; NaN everywhere else."""
    T, B, V = x.shape
    buf = torch.full((T * B * stride + shift,), float("nan"), dtype=torch.float32, device=DEV)
    rows = buf[shift:].view(T, B, stride)
    rows[:, :, :V] = dev(x)
    return buf, rows


def _check(got, want, ok, where):
    tk, st, sc = (g.cpu().numpy() for g in got)
    assert np.array_equal(tk[..., ok], want[0]) and np.array_equal(st[..., ok], want[1]), where
    a, b = sc[..., ok], want[2]
    assert np.array_equal(a[~np.isfinite(b)], b[~np.isfinite(b)]) and np.allclose(a[np.isfinite(b)], b[np.isfinite(b)], atol=TOL, rtol=0), where


@pytest.mark.parametrize("V", [4, 5, 7, 255, 258, 1021, 1023, 1024, 1025, 1026, 1028, 1277, 1280, 1281, 2046, 2049,
                               3071, 3075, 4095, 4097, 5125, 9217, 16381, 16384])
def test_ragged_rows(V):
    rng = np.random.default_rng(31000 + V)
    for case in range(3):
        blank = int(rng.choice([0, -1, V - 1, V // 2]))
        eos = int(rng.choice([-1, -1, V - 2 if blank != V - 2 else V - 3, 1 if blank != 1 else 2]))
        wmode, unk = int(rng.integers(0, 3)), float(rng.choice([0.0, 0.5, -0.25]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos, wmode, unk)
        B = int(rng.choice([1, 3, 6]))
        T = int(rng.choice([9, 33, 70])) if V <= 2100 else int(rng.choice([9, 20]))
        x = _rows(rng, T, B, V, blank, toks, offs)
        stride, shift = V + int(rng.choice([0, 1, 2, 4, 7])), int(rng.integers(0, 4))
        buf, rows = _on_device(x, stride, shift)
        ptr = buf.data_ptr() + 4 * shift
        alpha = float(rng.choice([0.0, 0.5, 1.0, -0.5]))
        s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
        last0 = rng.integers(-1, V, B).astype(np.int32)
        if B > 1 and rng.random() < 0.3:
            s0[1] = -1
        ok = [b for b in range(B) if s0[b] >= 0]
        for mode in (0, 1, 2):
            where = dict(V=V, case=case, blank=blank, eos=eos, mode=mode, stride=stride, shift=shift, T=T, B=B, alpha=alpha)
            want = ot.fuse_step_select(np.ascontiguousarray(x[0, ok]), s0[ok], last0[ok], alpha, mode)
            o = [torch.full((B,), -7, dtype=torch.int32, device=DEV), torch.full((B,), -7, dtype=torch.int32, device=DEV),
                 torch.zeros(B, device=DEV)]
            print("step", where, flush=True)
            pb.pb_fuse_step_select(tr, ptr, stride, dev(s0), dev(last0), alpha, B, mode, o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            _check(o, want, ok, where)
            want = ot.fuse_frames_select(np.ascontiguousarray(x[:, ok]), s0[ok], last0[ok], alpha, mode)
            need = pb.pb_fuse_frames_workspace_bytes(tr, T, B)
            ws = torch.full((max(need, 8) // 4,), 0x7f7f7f7f, dtype=torch.int32, device=DEV)
            for with_ws in (False, True):
                o = [torch.full((T, B), -7, dtype=torch.int32, device=DEV), torch.full((T, B), -7, dtype=torch.int32, device=DEV),
                     torch.zeros((T, B), device=DEV)]
                print("frames", with_ws, where, flush=True)
                if with_ws:
                    pb.pb_fuse_frames_ws(tr, ptr, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode, o[0], o[1],
                                         o[2], ws, need, 0)
                else:
                    pb.pb_fuse_frames_select(tr, ptr, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode, o[0],
                                             o[1], o[2], 0)
                torch.cuda.synchronize()
                _check(o, want, ok, where)
        pb.pb_free(tr)


@pytest.mark.parametrize("V", [257, 1025, 2047, 4097])
def test_ragged_rows_with_a_table_of_trees(V):
    rng = np.random.default_rng(32000 + V)
    blank, T, B = V - 1, 25, 7
    pairs = [_tree(rng, V, blank, -1, i % 3, 0.0) for i in range(3)]
    forest = pb.pb_forest_build([p[3] for p in pairs])
    ids = rng.integers(0, 3, B).astype(np.int32)
    x = _rows(rng, T, B, V, blank, pairs[0][0], pairs[0][1])
    s0 = np.array([rng.integers(0, pairs[i][2].num_states) for i in ids], dtype=np.int32)
    d_x, d_ids, d_s0 = dev(x), dev(ids), dev(s0)
    for mode in (0, 1, 2):
        o = [torch.full((T, B), -7, dtype=torch.int32, device=DEV), torch.full((T, B), -7, dtype=torch.int32, device=DEV),
             torch.zeros((T, B), device=DEV)]
        pb.pb_fuse_frames_forest(forest, d_x, B * V, V, d_ids, d_s0, None, 0.5, T, B, mode, o[0], o[1], o[2], 0)
        p = [torch.full((B,), -7, dtype=torch.int32, device=DEV), torch.full((B,), -7, dtype=torch.int32, device=DEV),
             torch.zeros(B, device=DEV)]
        pb.pb_fuse_step_forest(forest, d_x, V, d_ids, d_s0, None, 0.5, B, mode, p[0], p[1], p[2], 0)
        torch.cuda.synchronize()
        for b in range(B):
            want = pairs[ids[b]][2].fuse_frames_select(np.ascontiguousarray(x[:, b:b + 1]), s0[b:b + 1], None, 0.5, mode)
            _check([g[:, b:b + 1] for g in o], want, [0], (V, mode, b))
            _check([g[b:b + 1] for g in p], [w[0] for w in want], [0], (V, mode, b, "step"))
    pb.pb_forest_free(forest)


@pytest.mark.parametrize("V", [16385, 32768, 32771, 49152, 49153, 65533, 65536, 65537])
def test_step_on_very_wide_rows(V):
    """The single step with two, three and four chunks per wave, and the first width past them."""
    rng = np.random.default_rng(33000 + V)
    for case in range(2):
        blank, eos = int(rng.choice([0, -1, V - 1])), int(rng.choice([-1, V - 2]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos, case, float(rng.choice([0.0, -0.25])))
        B, stride, shift = 5, V + int(rng.choice([0, 3])), int(rng.integers(0, 4))
        x = _rows(rng, 1, B, V, blank, toks, offs)
        buf, _ = _on_device(x, stride, shift)
        s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
        s0[2] = ot.num_states
        last = rng.integers(-1, V, B).astype(np.int32)
        ok = [b for b in range(B) if b != 2]
        forest = pb.pb_forest_build([tr]) if eos < 0 else None
        for mode in (0, 1, 2):
            want = ot.fuse_step_select(np.ascontiguousarray(x[0, ok]), s0[ok], last[ok], 0.5, mode)
            for table in ([False, True] if forest else [False]):
                o = [torch.full((B,), -7, dtype=torch.int32, device=DEV), torch.full((B,), -7, dtype=torch.int32, device=DEV),
                     torch.zeros(B, device=DEV)]
                where = dict(V=V, case=case, blank=blank, eos=eos, mode=mode, stride=stride, shift=shift, table=table)
                print("step", where, flush=True)
                ptr = buf.data_ptr() + 4 * shift
                if table:
                    pb.pb_fuse_step_forest(forest, ptr, stride, dev(np.zeros(B, np.int32)), dev(s0), dev(last), 0.5, B, mode,
                                           o[0], o[1], o[2], 0)
                else:
                    pb.pb_fuse_step_select(tr, ptr, stride, dev(s0), dev(last), 0.5, B, mode, o[0], o[1], o[2], 0)
                torch.cuda.synchronize()
                _check(o, want, ok, where)
                assert int(o[0][2]) == -1 and int(o[1][2]) == -1 and torch.isnan(o[2][2]), where
        if forest:
            pb.pb_forest_free(forest)
        pb.pb_free(tr)


@pytest.mark.parametrize("V", [516, 640, 768, 1000, 1020, 1284, 5000, 10000, 16380])
def test_aligned_rows_that_end_inside_a_chunk(V):
    """Whole 16-byte groups, the last chunk part empty: the form without copies (all rules, a table of trees among them)."""
    rng = np.random.default_rng(34000 + V)
    for case in range(4):
        blank = int(rng.choice([0, -1, V - 1, V // 2]))
        eos = -1 if case == 3 else int(rng.choice([-1, V - 2 if blank != V - 2 else V - 3, V - 1 if blank != V - 1 else 1]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos, case % 3, float(rng.choice([0.0, 0.5, -0.25])))
        B = int(rng.choice([1, 3, 6]))
        T = int(rng.choice([9, 33, 70])) if V <= 1100 else 9
        x = _rows(rng, T, B, V, blank, toks, offs)
        stride = V + int(rng.choice([0, 4, 8]))
        buf, _ = _on_device(x, stride, 0)
        alpha = float(rng.choice([0.0, 0.5, 1.0, -0.5]))
        s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
        last0 = rng.integers(-1, V, B).astype(np.int32)
        if B > 1:
            s0[1] = ot.num_states
        ok = [b for b in range(B) if s0[b] < ot.num_states]
        forest = pb.pb_forest_build([tr]) if case == 3 else None
        ids = dev(np.zeros(B, np.int32))
        for mode in (0, 1, 2):
            where = dict(V=V, case=case, blank=blank, eos=eos, mode=mode, stride=stride, T=T, B=B, alpha=alpha)
            print("groups", where, flush=True)
            o = [torch.full((B,), -7, dtype=torch.int32, device=DEV), torch.full((B,), -7, dtype=torch.int32, device=DEV),
                 torch.zeros(B, device=DEV)]
            if forest:
                pb.pb_fuse_step_forest(forest, buf, stride, ids, dev(s0), dev(last0), alpha, B, mode, o[0], o[1], o[2], 0)
            else:
                pb.pb_fuse_step_select(tr, buf, stride, dev(s0), dev(last0), alpha, B, mode, o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            _check(o, ot.fuse_step_select(np.ascontiguousarray(x[0, ok]), s0[ok], last0[ok], alpha, mode), ok, where)
            want = ot.fuse_frames_select(np.ascontiguousarray(x[:, ok]), s0[ok], last0[ok], alpha, mode)
            need = pb.pb_fuse_frames_workspace_bytes(tr, T, B)
            ws = torch.full((max(need, 8) // 4,), 0x7f7f7f7f, dtype=torch.int32, device=DEV)
            for with_ws in (False, True):
                o = [torch.full((T, B), -7, dtype=torch.int32, device=DEV), torch.full((T, B), -7, dtype=torch.int32, device=DEV),
                     torch.zeros((T, B), device=DEV)]
                if forest and not with_ws:
                    pb.pb_fuse_frames_forest(forest, buf, B * stride, stride, ids, dev(s0), dev(last0), alpha, T, B, mode,
                                             o[0], o[1], o[2], 0)
                else:
                    pb.pb_fuse_frames_ws(tr, buf, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode, o[0], o[1],
                                         o[2], ws, need, 0)
                torch.cuda.synchronize()
                _check(o, want, ok, where)
        if forest:
            pb.pb_forest_free(forest)
        pb.pb_free(tr)
