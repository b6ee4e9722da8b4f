"""Multi-frame calls whose start states, previous labels or tree ids are a row of the outputs (a decoding loop that goes on
from its last states in place), on the widths of every multi-frame kernel, against the CPU oracle.  Such a call must
read every start before anything of the hypothesis is written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, dev  # noqa: E402
from test_gpu_ragged import _check, _on_device, _rows, _tree  # noqa: E402


def _outputs(T, B):
    return [torch.full((T, B), -7, dtype=torch.int32, device=DEV), torch.full((T, B), -7, dtype=torch.int32, device=DEV),
            torch.zeros((T, B), device=DEV)]


@pytest.mark.parametrize("V,T,B", [(300, 65, 4), (1000, 30, 9), (1024, 200, 3), (1025, 40, 5), (1027, 520, 2), (2500, 160, 3),
                                   (4096, 40, 3), (16383, 20, 2), (16386, 21, 3)])
def test_start_states_and_labels_inside_the_outputs(V, T, B):
    rng = np.random.default_rng(61000 + V)
    blank = V - 1
    toks, offs, ot, tr = _tree(rng, V, blank, -1, 1, 0.0)
    x = _rows(rng, T, B, V, blank, toks, offs)
    s0, last0 = rng.integers(0, ot.num_states, B).astype(np.int32), rng.integers(-1, V, B).astype(np.int32)
    s0[0] = 0
    buf, _ = _on_device(x, V, 0)
    for mode in (0, 1, 2):
        want = ot.fuse_frames_select(x, s0, last0, 0.5, mode)
        need = pb.pb_fuse_frames_workspace_bytes(tr, T, B)
        ws = torch.full((max(need, 8) // 4,), 0x7f7f7f7f, dtype=torch.int32, device=DEV)
        for row in (0, T // 2, T - 1):
            for with_ws in (False, True):
                o = _outputs(T, B)
                o[1][row], o[0][row] = dev(s0), dev(last0)
                print("overlap", V, T, B, mode, row, with_ws, flush=True)
                if with_ws:
                    pb.pb_fuse_frames_ws(tr, buf, B * V, V, o[1][row], o[0][row], 0.5, T, B, mode, o[0], o[1], o[2], ws, need, 0)
                else:
                    pb.pb_fuse_frames_select(tr, buf, B * V, V, o[1][row], o[0][row], 0.5, T, B, mode, o[0], o[1], o[2], 0)
                torch.cuda.synchronize()
                _check(o, want, list(range(B)), (V, mode, row, with_ws))
    pb.pb_free(tr)


@pytest.mark.parametrize("V,T", [(300, 33), (1025, 40), (2500, 200), (16386, 12)])
def test_tree_ids_inside_the_outputs(V, T):
    rng = np.random.default_rng(62000 + V)
    blank = 0
    pairs = [_tree(rng, V, blank, -1, i % 3, 0.0) for i in range(3)]
    forest = pb.pb_forest_build([p[3] for p in pairs])
    ids = np.array([0, 2, 7, 1], dtype=np.int32)               # (7: no such tree)
    B = len(ids)
    x = _rows(rng, T, B, V, blank, pairs[0][0], pairs[0][1])
    s0 = np.array([rng.integers(0, pairs[i % 3][2].num_states) for i in ids], dtype=np.int32)
    for mode in (0, 2):
        for out, row in ((0, 0), (0, T - 1), (1, T // 2)):      # a row of the tokens, of the states
            o = _outputs(T, B)
            o[out][row] = dev(ids)
            print("ids", V, T, mode, out, row, flush=True)
            pb.pb_fuse_frames_forest(forest, dev(x), B * V, V, o[out][row], dev(s0), None, 0.5, T, B, mode, o[0], o[1], o[2], 0)
            torch.cuda.synchronize()
            for b in range(B):
                if ids[b] > 2:
                    assert bool((o[0][:, b] == -1).all()) and bool((o[1][:, b] == -1).all())
                    continue
                want = pairs[ids[b]][2].fuse_frames_select(np.ascontiguousarray(x[:, b:b + 1]), s0[b:b + 1], None, 0.5, mode)
                _check([g[:, b:b + 1] for g in o], want, [0], (V, mode, out, row, b))
    pb.pb_forest_free(forest)
