"""GPU parity of the segment decoders on calls past the lines to the two-pass decoder (sizes.SEGMENTS, which test_dispatch.py
holds the dispatch to): every row shape of the narrow ones and every ring of the wide one, whole and ragged rows, with a
workspace and without, a tree with EOS and a table of trees (one id unknown), padded and shifted rows, exact ties, rows of
-inf, phrases spoken, negative alpha, an invalid start state, every selection rule; and calls on either side of every line.
Some hypotheses of each call against the CPU oracle: ids bit-exact, scores within 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, dev  # noqa: E402
from test_gpu_ragged import _check, _on_device, _tree  # noqa: E402
from sizes import LINES, SEGMENTS  # noqa: E402
from test_gpu_rows import _near_ties, _outputs  # noqa: E402


def _spoken(rng, T, B, V, lists):
    """Rows on the device: rounded normal values (exact ties), phrases spoken on some frames, whole rows of -inf."""
    x = torch.round(torch.randn((T, B, V), device=DEV) * 4) / 2
    t, b, v = [], [], []
    for h in range(B):
        toks, offs = lists[h % len(lists)]
        f = int(rng.integers(0, 12))
        while f < T:
            i = int(rng.integers(0, len(offs) - 1))
            for tok in toks[offs[i]:offs[i + 1]]:
                for _ in range(int(rng.integers(1, 3))):
                    if f < T:
                        t.append(f), b.append(h), v.append(int(tok))
                        f += 1
            f += int(rng.integers(0, 25))
    x[torch.tensor(t, device=DEV), torch.tensor(b, device=DEV), torch.tensor(v, device=DEV)] += 12.0
    x[torch.rand((T, B), device=DEV) < 0.03] = -float("inf")
    return x


# (a row of whole vectors also at a stride and an address that are none: another shape up to 1024 tokens)
@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("V,whole", [(V, V % 4 == 0) for V in sorted(SEGMENTS)] + [(512, False), (1024, False), (2048, False)])
def test_segment_decoders_past_the_dispatch_line(V, whole, table):
    rng = np.random.default_rng(81000 + 2 * V + table)
    torch.manual_seed(V)
    T, B = SEGMENTS[V]
    blank = int(rng.choice([0, -1, V - 1]))
    eos = -1 if table else V - 2
    trees = [_tree(rng, V, blank, eos, i, 0.25 if i == 1 else 0.0) for i in range(3 if table else 1)]
    x = _spoken(rng, T, B, V, [(p[0], p[1]) for p in trees])
    stride, shift = (V + (4 if V % 1024 else 0), 0) if whole else (V + 3, 1)
    buf = torch.full((T * B * stride + shift,), float("nan"), dtype=torch.float32, device=DEV)
    buf[shift:].view(T, B, stride)[:, :, :V] = x
    ptr = buf.data_ptr() + 4 * shift
    ids = np.arange(B, dtype=np.int32) % len(trees)
    s0 = np.array([rng.integers(0, trees[i][2].num_states) for i in ids], dtype=np.int32)
    s0[:2] = 0
    ids[B - 1] = 5                                  # (no such tree)
    if not table:
        s0[B - 1] = trees[0][2].num_states          # (no such state)
    last0 = rng.integers(-1, V, B).astype(np.int32)
    alpha = -0.5 if V in (1027, 2049, 9217) else 0.5
    look = sorted({0, 1, B - 2, *rng.integers(0, B - 1, 3).tolist()})
    xs = x[:, torch.tensor(look, device=DEV)].cpu().numpy()
    del x
    forest = pb.pb_forest_build([p[3] for p in trees]) if table else None
    for mode in (0, 1, 2):
        o = _outputs(T, B)
        print("segments", V, T, B, whole, table, mode, flush=True)
        if table:
            pb.pb_fuse_frames_forest(forest, ptr, B * stride, stride, dev(ids), dev(s0), dev(last0), alpha, T, B, mode, o[0],
                                     o[1], o[2], 0)
        else:
            pb.pb_fuse_frames_select(trees[0][3], ptr, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode, o[0], o[1],
                                     o[2], 0)
        torch.cuda.synchronize()
        need = 0 if table else pb.pb_fuse_frames_workspace_bytes(trees[0][3], T, B)
        if need > 0:  # (wrong guesses repaired by patches instead of in the second pass: the same bits)
            ws, p = torch.full((need // 4,), 0x7f7f7f7f, dtype=torch.int32, device=DEV), _outputs(T, B)
            pb.pb_fuse_frames_ws(trees[0][3], ptr, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode, p[0], p[1], p[2], ws,
                                 need, 0)
            torch.cuda.synchronize()
            assert all(torch.equal(g.view(torch.int32), q.view(torch.int32)) for g, q in zip(o, p)), (V, whole, mode)
        for q, h in enumerate(look):
            want = trees[ids[h]][2].fuse_frames_select(np.ascontiguousarray(xs[:, q:q + 1]), s0[h:h + 1], last0[h:h + 1], alpha, mode)
            _check([g[:, h:h + 1] for g in o], want, [0], (V, whole, table, mode, h, blank, alpha))
        assert bool((o[0][:, B - 1] == -1).all()) and bool((o[1][:, B - 1] == -1).all()) and bool(torch.isnan(o[2][:, B - 1]).all())
    if forest:
        pb.pb_forest_free(forest)
    for p in trees:
        pb.pb_free(p[3])


@pytest.mark.parametrize("V", [1025, 1027, 1152, 1280])
def test_near_ties_in_the_narrow_two_pass_decoder(V):
    """Values a few units in the last place apart: the winner under root boosts need not win in another state."""
    rng = np.random.default_rng(82000 + V)
    for case in range(3):
        blank, eos = int(rng.choice([0, -1, V - 1])), int(rng.choice([-1, V - 2]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos, case, float(rng.choice([0.0, 0.5])))
        T, B, alpha = 40, 3, float(rng.choice([0.3, 1.0, -0.5]))
        x = _near_ties(rng, tr, T, B, V, alpha)
        stride, shift = V + int(rng.choice([0, 3])), int(rng.integers(0, 4))
        buf, _ = _on_device(x, stride, shift)
        s0, last0 = rng.integers(0, ot.num_states, B).astype(np.int32), rng.integers(-1, V, B).astype(np.int32)
        for mode in (0, 1, 2):
            o = _outputs(T, B)
            print("near", V, case, mode, flush=True)
            pb.pb_fuse_frames_select(tr, buf.data_ptr() + 4 * shift, B * stride, stride, dev(s0), dev(last0), alpha, T, B, mode,
                                     o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            _check(o, ot.fuse_frames_select(x, s0, last0, alpha, mode), list(range(B)), (V, case, mode, blank, eos, alpha))
        pb.pb_free(tr)


@pytest.mark.parametrize("V,T,B", [c[:3] for c in LINES if c[0] * c[1] * c[2] <= 1 << 28])
def test_both_sides_of_the_lines(V, T, B):
    """Sizes on either side of the lines between the two passes and the segment decoders, phrases spoken, every rule."""
    rng = np.random.default_rng(83000 + V + T)
    torch.manual_seed(T)
    toks, offs, ot, tr = _tree(rng, V, V - 1, -1, T % 3, 0.0)
    x = _spoken(rng, T, B, V, [(toks, offs)])
    s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
    last0 = rng.integers(-1, V, B).astype(np.int32)
    look = sorted({0, B - 1, *rng.integers(0, B, 3).tolist()})
    xs = x[:, torch.tensor(look, device=DEV)].cpu().numpy()
    for mode in (0, 1, 2):
        o = _outputs(T, B)
        print("lines", V, T, B, mode, flush=True)
        pb.pb_fuse_frames_select(tr, x, B * V, V, dev(s0), dev(last0), 0.5, T, B, mode, o[0], o[1], o[2], 0)
        torch.cuda.synchronize()
        _check([g[:, look] for g in o], ot.fuse_frames_select(xs, s0[look], last0[look], 0.5, mode), list(range(len(look))), (V, T, B, mode))
    pb.pb_free(tr)
