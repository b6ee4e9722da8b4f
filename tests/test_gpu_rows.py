"""GPU parity of the multi-frame decoder in two passes (all rows first, then the automaton on their winners), against
the CPU oracle: ids bit-exact, scores within 1e-5.  Rows where the winner under root boosts need not be the winner in
another state (exact ties, ties up to rounding, rows of -inf), more frames than one block of the second pass holds,
segments that start from wrong guesses, invalid states and trees, and outputs that overlap the start states."""
import numpy as np
import pytest

import pb_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, dev  # noqa: E402
from sizes import LINES  # noqa: E402
from test_gpu_ragged import _check, _on_device, _rows, _tree  # noqa: E402


def _outputs(T, B):
    return [torch.full((T, B), -7, dtype=torch.int32, device=DEV), torch.full((T, B), -7, dtype=torch.int32, device=DEV),
            torch.zeros((T, B), device=DEV)]


def _near_ties(rng, tr, T, B, V, alpha):
    """Rows in which every token's fused value in the root is the same up to a few units in the last place."""
    root = pb.pb_host_arrays(tr)["root_score"].astype(np.float64)
    x = -6.0 - alpha * root[None, None] + rng.integers(-3, 4, (T, B, V)) * 2.0 ** -22
    return x.astype(np.float32)


@pytest.mark.parametrize("V", [16385, 16388, 20001, 40960, 65539])
def test_rows_then_automaton(V):
    rng = np.random.default_rng(41000 + V)
    for case in range(4):
        blank = int(rng.choice([0, -1, V - 1, V // 2]))
        eos = int(rng.choice([-1, -1, V - 2]))
        wmode, unk = int(rng.integers(0, 3)), float(rng.choice([0.0, 0.5, -0.25]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos, wmode, unk)
        B, T = int(rng.choice([1, 3])), int(rng.choice([1, 2, 9, 40]))
        alpha = float(rng.choice([0.0, 0.5, 1.0, -0.5])) if case else 0.3
        x = _near_ties(rng, tr, T, B, V, alpha) if case == 0 else _rows(rng, T, B, V, blank, toks, offs)
        stride, shift = V + int(rng.choice([0, 1, 2, 4, 7])), int(rng.integers(0, 4))
        buf, _ = _on_device(x, stride, shift)
        s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
        last0 = rng.integers(-1, V, B).astype(np.int32)
        if B > 1 and rng.random() < 0.5:
            s0[1] = -1
        ok = [b for b in range(B) if s0[b] >= 0]
        for mode in (0, 1, 2):
            where = dict(V=V, case=case, blank=blank, eos=eos, mode=mode, stride=stride, shift=shift, T=T, B=B, alpha=alpha)
            print("rows", where, flush=True)
            want = ot.fuse_frames_select(np.ascontiguousarray(x[:, ok]), s0[ok], last0[ok], alpha, mode)
            o = _outputs(T, B)
            pb.pb_fuse_frames_select(tr, buf.data_ptr() + 4 * shift, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode,
                                     o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            _check(o, want, ok, where)
            for b in set(range(B)) - set(ok):
                assert bool((o[0][:, b] == -1).all()) and bool((o[1][:, b] == -1).all()) and bool(torch.isnan(o[2][:, b]).all()), where
        pb.pb_free(tr)


@pytest.mark.parametrize("T,planted", [(1024, 0.9), (1025, 0.5), (1100, 0.9)])
def test_more_frames_than_a_block(T, planted):
    rng = np.random.default_rng(42000 + T)
    V = 16390
    toks, offs, ot, tr = _tree(rng, V, V - 1, -1, 1, 0.0)
    shape = W.Config(9, "rows", V, V - 1, 1, 1, 8, "uniform", 1.1, 1, 1, T, 2.0)
    x = W.make_logp(shape, seed=T, planting=W.Planting(toks, offs, cover=planted, bump=10.0)).astype(np.float32)
    s0 = np.array([int(rng.integers(0, ot.num_states))], dtype=np.int32)
    for mode in (0, 1, 2):
        want = ot.fuse_frames_select(x, s0, None, 0.5, mode)
        o = _outputs(T, 1)
        print("block", T, mode, flush=True)
        pb.pb_fuse_frames_select(tr, dev(x), V, V, dev(s0), None, 0.5, T, 1, mode, o[0], o[1], o[2], 0)
        torch.cuda.synchronize()
        _check(o, want, [0], (T, mode))
    pb.pb_free(tr)


def test_a_table_of_trees_and_overlapping_outputs():
    rng = np.random.default_rng(43000)
    V, T, B = 16386, 21, 5
    blank = 0
    pairs = [_tree(rng, V, blank, -1, i % 3, 0.0) for i in range(3)]
    forest = pb.pb_forest_build([p[3] for p in pairs])
    ids = np.array([0, 1, 2, 7, 1], dtype=np.int32)            # (7: no such tree)
    x = _rows(rng, T, B, V, blank, pairs[0][0], pairs[0][1])
    s0 = np.array([rng.integers(0, pairs[i % 3][2].num_states) for i in ids], dtype=np.int32)
    for mode in (0, 1, 2):
        want = [pairs[ids[b]][2].fuse_frames_select(np.ascontiguousarray(x[:, b:b + 1]), s0[b:b + 1], None, 0.5, mode)
                if ids[b] < 3 else None for b in range(B)]
        for inside in (False, True):                            # the start states are the last row of the states output
            o = _outputs(T, B)
            d_s0 = dev(s0)
            if inside:
                o[1][T - 1] = d_s0
                d_s0 = o[1][T - 1]
            print("forest", mode, inside, flush=True)
            pb.pb_fuse_frames_forest(forest, dev(x), B * V, V, dev(ids), d_s0, None, 0.5, T, B, mode, o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            for b in range(B):
                if want[b] is None:
                    assert bool((o[0][:, b] == -1).all()) and bool((o[1][:, b] == -1).all())
                else:
                    _check([g[:, b:b + 1] for g in o], want[b], [0], (mode, inside, b))
    pb.pb_forest_free(forest)


# (the smaller ones of the list, which the CPU oracle decodes whole)
@pytest.mark.parametrize("V,T,B", [c[:3] for c in LINES if c[0] * c[1] * c[2] <= 1 << 23] + [(1025, 255, 2), (1280, 60, 5), (2500, 156, 2), (1100, 33, 500)])
def test_both_sides_of_the_dispatch(V, T, B):
    """Sizes on either side of the lines between the two passes and the segment decoders, with a workspace and without,
    phrases spoken, every rule, every hypothesis."""
    rng = np.random.default_rng(44000 + V + T)
    blank = V - 1
    toks, offs, ot, tr = _tree(rng, V, blank, -1, T % 3, 0.0)
    shape = W.Config(9, "rows", V, blank, 1, 1, 8, "uniform", 1.1, B, 1, T, 2.0)
    x = W.make_logp(shape, seed=V + T, planting=W.Planting(toks, offs, cover=0.5, bump=10.0), blank_bias=6.0, blank_frac=0.3)
    x = x.astype(np.float32)
    s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
    last0 = rng.integers(-1, V, B).astype(np.int32)
    d_x = dev(x)
    for mode in (0, 1, 2):
        want = ot.fuse_frames_select(x, s0, last0, 0.5, mode)
        need = pb.pb_fuse_frames_workspace_bytes(tr, T, B)
        ws = torch.full((max(need, 8) // 4,), 0x7f7f7f7f, dtype=torch.int32, device=DEV)
        for with_ws in (False, True):
            o = _outputs(T, B)
            print("dispatch", V, T, B, mode, with_ws, flush=True)
            if with_ws:
                pb.pb_fuse_frames_ws(tr, d_x, B * V, V, dev(s0), dev(last0), 0.5, T, B, mode, o[0], o[1], o[2], ws, need, 0)
            else:
                pb.pb_fuse_frames_select(tr, d_x, B * V, V, dev(s0), dev(last0), 0.5, T, B, mode, o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            _check(o, want, list(range(B)), (V, T, B, mode, with_ws))
    pb.pb_free(tr)
