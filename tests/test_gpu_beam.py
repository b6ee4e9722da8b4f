"""GPU parity of the beam step on rows of every kernel shape (positions per lane, waves per beam, streamed rows), against
the CPU oracle: ids bit-exact, scores within 1e-5.  Exact ties across beams, more ties than the list of survivors holds,
dead beams, the first step of a search (one live beam), states with several hundred arcs (several survivors in one lane),
log-probs at any alignment, invalid utterances and a table of trees."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, TOL, dev  # noqa: E402
from test_gpu_ragged import _on_device, _rows, _tree  # noqa: E402


def _hyp(rng, U, K):
    h = np.round(-5 * rng.random((U, K)) * 4).astype(np.float32) / 4
    kind = int(rng.integers(0, 4))
    if kind == 0:
        h[:, 1:] = -np.inf                      # the first step of a search
    elif kind == 1:
        h[rng.random((U, K)) < 0.4] = -np.inf   # some dead beams, whole utterances among them
        h[0] = -np.inf
    elif kind == 2:
        h[:] = 0.0
    return h.reshape(-1)


def _outputs(n):
    return [torch.full((n,), -7, dtype=torch.int32, device=DEV) for _ in range(3)] + [torch.zeros(n, device=DEV)]


def _compare(o, want, rows, where):
    tok, par, st, sc = (x.cpu().numpy()[rows] for x in o)
    wt, wp, ws, wc = (np.asarray(w).reshape(-1) for w in want)
    assert np.array_equal(tok, wt) and np.array_equal(par, wp) and np.array_equal(st, ws), where
    fin = np.isfinite(wc)
    assert np.array_equal(sc[~fin], wc[~fin]) and np.allclose(sc[fin], wc[fin], atol=TOL, rtol=0), where


@pytest.mark.parametrize("V,K", [(4, 3), (5, 8), (7, 32), (256, 16), (257, 1), (512, 8), (1023, 4), (1024, 4), (1024, 8), (1025, 8),
                                 (1025, 32), (2047, 16), (2048, 8), (4096, 16), (4097, 4), (5000, 16), (8192, 8), (8193, 8),
                                 (9217, 32), (16385, 4), (20001, 3), (40000, 2), (33000, 32), (65540, 1)])
def test_beam_shapes(V, K):
    rng = np.random.default_rng(51000 + 40 * V + K)
    for case in range(4):
        blank = int(rng.choice([0, -1, V - 1]))
        eos = int(rng.choice([-1, V - 2 if blank != V - 2 else V - 3]))
        toks, offs, ot, tr = _tree(rng, V, blank, eos, int(rng.integers(0, 3)), float(rng.choice([0.0, 0.5, -0.25])))
        U = int(rng.choice([1, 3]))
        x = _rows(rng, 1, U * K, V, blank, toks, offs)[0]
        if case == 1:
            x[:] = np.round(x / 8) * 8          # so many exact ties that the list overflows
        stride, shift = V + int(rng.choice([0, 0, 4, 3])), int(rng.choice([0, 0, 1, 3]))
        buf, _ = _on_device(x[None], stride, shift)
        states = rng.integers(0, ot.num_states, U * K).astype(np.int32)
        if case == 2:                           # depth-1 states, the ones with the most arcs among them
            deg = pb.pb_host_arrays(tr)["arc_count"]
            states[:] = np.argsort(-deg)[rng.integers(0, min(4, len(deg)), U * K)]
        hyp, alpha = _hyp(rng, U, K), float(rng.choice([0.0, 0.5, 1.0, -0.5]))
        bad = U == 3 and case == 3
        if bad:
            states[K] = ot.num_states
        good = [i for i in range(U * K) if not (bad and K <= i < 2 * K)]
        where = dict(V=V, K=K, case=case, blank=blank, eos=eos, stride=stride, shift=shift, U=U, alpha=alpha)
        print("beam", where, flush=True)
        o = _outputs(U * K)
        pb.pb_fuse_step_beam(tr, buf.data_ptr() + 4 * shift, stride, dev(hyp), dev(states), alpha, U, K, o[0], o[1], o[2], o[3], 0)
        torch.cuda.synchronize()
        want = ot.fuse_step_beam(np.ascontiguousarray(x[good]), hyp[good], states[good], alpha, len(good) // K, K)
        _compare(o, want, good, where)
        if bad:
            assert all(bool((g[K:2 * K] == -1).all()) for g in o[:3]) and bool(torch.isnan(o[3][K:2 * K]).all()), where
        pb.pb_free(tr)


@pytest.mark.parametrize("V,K", [(1025, 8), (1024, 4), (6000, 12)])
def test_beams_with_a_table_of_trees(V, K):
    rng = np.random.default_rng(52000 + V)
    pairs = [_tree(rng, V, V - 1, -1, i % 3, 0.0) for i in range(3)]
    forest = pb.pb_forest_build([p[3] for p in pairs])
    ids = np.array([2, 0, 5, 1], dtype=np.int32)   # (5: no such tree)
    U = len(ids)
    x = _rows(rng, 1, U * K, V, V - 1, pairs[0][0], pairs[0][1])[0]
    states = np.concatenate([rng.integers(0, pairs[i % 3][2].num_states, K) for i in ids]).astype(np.int32)
    hyp = _hyp(rng, U, K)
    o = _outputs(U * K)
    print("forest", V, K, flush=True)
    pb.pb_fuse_step_beam_forest(forest, dev(x), V, dev(ids), dev(hyp), dev(states), 0.5, U, K, o[0], o[1], o[2], o[3], 0)
    torch.cuda.synchronize()
    for u in range(U):
        rows = list(range(u * K, u * K + K))
        if ids[u] > 2:
            assert all(bool((g[rows] == -1).all()) for g in o[:3])
            continue
        want = pairs[ids[u]][2].fuse_step_beam(np.ascontiguousarray(x[rows]), hyp[rows], states[rows], 0.5, 1, K)
        _compare(o, want, rows, (V, K, u))
    pb.pb_forest_free(forest)


@pytest.mark.parametrize("V,K", [(300, 4), (1024, 16), (9000, 8), (20000, 16)])
def test_scores_written_over_the_hypothesis_scores(V, K):
    """A decoding loop may keep one buffer for the hypothesis scores; dead utterances take the selection by rounds."""
    rng = np.random.default_rng(53000 + V)
    toks, offs, ot, tr = _tree(rng, V, 0, -1, 0, 0.0)
    U = 3
    x = _rows(rng, 1, U * K, V, 0, toks, offs)[0]
    x[K:2 * K] = -3.0                             # one utterance of nothing but ties
    states = rng.integers(0, ot.num_states, U * K).astype(np.int32)
    hyp = np.where(np.arange(U * K) < K, -np.inf, -rng.random(U * K)).astype(np.float32)   # one of dead beams
    want = ot.fuse_step_beam(x, hyp, states, 0.5, U, K)
    o, d_hyp = _outputs(U * K), dev(hyp)
    print("in place", V, K, flush=True)
    pb.pb_fuse_step_beam(tr, dev(x), V, d_hyp, dev(states), 0.5, U, K, o[0], o[1], o[2], d_hyp, 0)
    torch.cuda.synchronize()
    _compare(o[:3] + [d_hyp], want, list(range(U * K)), (V, K))
    pb.pb_free(tr)


@pytest.mark.parametrize("kind", ["dead", "const", "flat", "few finite", "steps"])
@pytest.mark.parametrize("V,K", [(4, 32), (5, 3), (40, 16), (256, 1), (300, 8), (1024, 4), (1025, 16), (1030, 1), (2050, 2), (4100, 8),
                                 (9000, 8), (16390, 16), (33000, 16), (70000, 2)])
def test_totals_that_do_not_fit_the_list(V, K, kind):
    """Dead utterances and rows that are flat or tie: far more totals reach any bound than the list of survivors holds."""
    rng = np.random.default_rng(54000 + 40 * V + K)
    blank, eos = (0, V - 2) if V > 8 else (V - 1, -1)
    toks, offs, ot, tr = _tree(rng, V, blank, eos, 0, 0.0)
    U = 3
    x = (rng.standard_normal((U * K, V)) * 2 - 8).astype(np.float32)
    hyp = (-3 * rng.random(U * K)).astype(np.float32)
    u = slice(K, 2 * K)                        # the utterance in the middle
    if kind == "dead":
        hyp[u] = -np.inf
    elif kind == "const":
        x[u], hyp[u] = -3.0, -1.0
    elif kind == "flat":                       # all within 0.01: below the finest distance the first bound looks at
        x[u] = (-7 + 0.01 * rng.random((K, V))).astype(np.float32)
        hyp[u] = -2.0
    elif kind == "few finite":
        keep = x[u].reshape(-1)[:max(1, K - 1)].copy()
        x[u] = -np.inf
        x[u].reshape(-1)[np.arange(len(keep)) * (K * V // len(keep))] = keep
    else:                                      # eight values in all
        x[u], hyp[u] = -rng.integers(1, 9, (K, V)).astype(np.float32), 0.0
    states = rng.integers(0, ot.num_states, U * K).astype(np.int32)
    deg = pb.pb_host_arrays(tr)["arc_count"]
    states[K:K + max(1, K // 2)] = np.argsort(-deg)[:max(1, K // 2)] % ot.num_states if len(deg) > K else 0
    d_x, d_st = dev(x), dev(states)
    for alpha in (0.5, 0.0):
        want = ot.fuse_step_beam(x, hyp, states, alpha, U, K)
        for in_place in (False, True):
            o, d_hyp = _outputs(U * K), dev(hyp)
            scores = d_hyp if in_place else o[3]
            print("list", V, K, kind, alpha, in_place, flush=True)
            pb.pb_fuse_step_beam(tr, d_x, V, d_hyp, d_st, alpha, U, K, o[0], o[1], o[2], scores, 0)
            torch.cuda.synchronize()
            _compare(o[:3] + [scores], want, list(range(U * K)), (V, K, kind, alpha, in_place))
    pb.pb_free(tr)


@pytest.mark.parametrize("V,K", [(6, 8), (1025, 8), (6000, 12), (33000, 20)])
def test_dead_utterances_with_a_table_of_trees(V, K):
    rng = np.random.default_rng(55000 + V)
    pairs = [_tree(rng, V, V - 1, -1, i % 3, 0.0) for i in range(3)]
    forest = pb.pb_forest_build([p[3] for p in pairs])
    ids = np.array([1, 2, 9, 0], dtype=np.int32)   # (9: no such tree)
    U = len(ids)
    x = _rows(rng, 1, U * K, V, V - 1, pairs[0][0], pairs[0][1])[0]
    states = np.concatenate([rng.integers(0, pairs[i % 3][2].num_states, K) for i in ids]).astype(np.int32)
    states[3 * K + K - 1] = -1                     # a dead utterance with an invalid state
    hyp = np.full(U * K, -np.inf, np.float32)
    hyp[:K] = -1.0
    o = _outputs(U * K)
    print("dead forest", V, K, flush=True)
    pb.pb_fuse_step_beam_forest(forest, dev(x), V, dev(ids), dev(hyp), dev(states), 0.5, U, K, o[0], o[1], o[2], o[3], 0)
    torch.cuda.synchronize()
    for u in (0, 1):
        rows = list(range(u * K, u * K + K))
        want = pairs[ids[u]][2].fuse_step_beam(np.ascontiguousarray(x[rows]), hyp[rows], states[rows], 0.5, 1, K)
        _compare(o, want, rows, (V, K, u))
    assert all(bool((g[2 * K:] == -1).all()) for g in o[:3]) and bool(torch.isnan(o[3][2 * K:]).all())
    pb.pb_forest_free(forest)


@pytest.mark.parametrize("V", [516, 1000, 1024])
@pytest.mark.parametrize("K,U", [(1, 3), (1, 8192), (1, 8193), (2, 512), (2, 513), (2, 2304), (2, 2305), (3, 342), (3, 1536), (3, 1537)])
def test_few_beams_on_both_sides_of_the_dispatch(V, K, U):
    """Aligned rows: a wave per beam or a list of survivors, by the number of utterances; ties, dead beams, a bad state."""
    rng = np.random.default_rng(56000 + V + U)
    blank, eos = int(rng.choice([0, -1, V - 1])), int(rng.choice([-1, V - 2]))
    toks, offs, ot, tr = _tree(rng, V, blank, eos, 1, 0.25)
    x = torch.randn((U * K, V), device=DEV) * 2
    x = torch.round(x * 4) / 4                        # (many exact ties)
    x[rng.integers(0, U * K, 5)] = -float("inf")
    hyp = np.round(-3 * rng.random(U * K) * 4).astype(np.float32) / 4
    hyp[rng.random(U * K) < 0.2] = -np.inf
    states = rng.integers(0, ot.num_states, U * K).astype(np.int32)
    states[K * (U // 2)] = ot.num_states
    o = _outputs(U * K)
    print("few", V, K, U, flush=True)
    pb.pb_fuse_step_beam(tr, x, V, dev(hyp), dev(states), 0.5, U, K, o[0], o[1], o[2], o[3], 0)
    torch.cuda.synchronize()
    assert all(bool((g[K * (U // 2):K * (U // 2 + 1)] == -1).all()) for g in o[:3])
    look = [u for u in sorted({0, 1, U - 1, *rng.integers(0, U, 40).tolist()}) if u != U // 2]
    rows = [u * K + k for u in look for k in range(K)]
    xs = x[torch.tensor(rows, device=DEV)].cpu().numpy()
    _compare(o, ot.fuse_step_beam(xs, hyp[rows], states[rows], 0.5, len(look), K), rows, (V, K, U))
    pb.pb_free(tr)
