"""GPU parity of the dense rows at any length and alignment of the outputs, against the CPU oracle, scores within 1e-5: rows
that are no multiple of four, the ends of a tile, outputs that start off a 16-byte boundary, without next states, with
invalid states; nothing outside the rows is written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, TOL, dev  # noqa: E402
from test_gpu_ragged import _tree  # noqa: E402


@pytest.mark.parametrize("V", [4, 5, 6, 7, 255, 257, 1024, 1025, 2047, 2048, 2049, 2051, 4096, 4099, 8193])
def test_rows_at_any_alignment(V):
    rng = np.random.default_rng(61000 + V)
    for case in range(3):
        blank, eos = int(rng.choice([0, -1, V - 1])), int(rng.choice([-1, V - 2 if V > 4 else -1]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos if eos != blank else -1, case, float(rng.choice([0.0, -0.25])))
        B, shift = int(rng.choice([1, 3, 17])), case
        states = rng.integers(0, ot.num_states, B).astype(np.int32)
        states[0] = 0
        if B > 3:
            states[2] = ot.num_states
        ok = states < ot.num_states
        want = ot.score(states[ok])
        for with_next in (True, False):
            sc = torch.full((B * V + 8,), 5.0, device=DEV)
            nx = torch.full((B * V + 8,), -9, dtype=torch.int32, device=DEV)
            print("score", V, case, B, shift, with_next, flush=True)
            pb.pb_score(tr, dev(states), B, sc.data_ptr() + 4 * shift, nx.data_ptr() + 4 * shift if with_next else None, 0)
            torch.cuda.synchronize()
            s, n = sc.cpu().numpy(), nx.cpu().numpy()
            rows, nrows = s[shift:shift + B * V].reshape(B, V), n[shift:shift + B * V].reshape(B, V)
            assert np.allclose(rows[ok], want[0], atol=TOL, rtol=0) and np.isnan(rows[~ok]).all(), (V, case)
            assert (s[:shift] == 5.0).all() and (s[shift + B * V:] == 5.0).all(), (V, case)
            if with_next:
                assert np.array_equal(nrows[ok], want[1]) and (nrows[~ok] == -1).all(), (V, case)
                assert (n[:shift] == -9).all() and (n[shift + B * V:] == -9).all(), (V, case)
            else:
                assert (n == -9).all(), (V, case)
        pb.pb_free(tr)


def test_rows_past_the_caches():
    """Outputs of more than 192 MiB (written past the caches): every row equals the same state's row of a small call."""
    rng = np.random.default_rng(62000)
    V, B = 4096, 6200
    toks, offs, ot, tr = _tree(rng, V, 0, -1, 0, 0.0)
    states = rng.integers(0, min(ot.num_states, 50), B).astype(np.int32)
    few = np.arange(min(ot.num_states, 50), dtype=np.int32)
    want = [torch.from_numpy(np.ascontiguousarray(w)).to(DEV) for w in ot.score(few)]
    sc = torch.full((B, V), 5.0, device=DEV)
    nx = torch.full((B, V), -9, dtype=torch.int32, device=DEV)
    pb.pb_score(tr, dev(states), B, sc, nx, 0)
    torch.cuda.synchronize()
    pick = dev(states).long()
    assert bool(((sc - want[0][pick]).abs() <= TOL).all()) and bool((nx == want[1][pick]).all())
    pb.pb_free(tr)
