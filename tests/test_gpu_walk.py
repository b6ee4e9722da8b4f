"""GPU parity of the second pass of the two-pass multi-frame decoder (frames decided side by side from the states the winners
lead to, then again where that was wrong) at the sizes where it can go wrong, against the CPU oracle: every row shape of the
first pass (up to 256 tokens the CTC rule alone takes the two passes), both sides of the packed winner word, few and many frames a wave, more frames than a block holds, states with
more arcs than a wave has lanes, chains of more than four levels, whole phrases (an arc and the base winner have the same
value), rows that only a pass over them can decide, more of them than are taken at a time; and the segment decoders on calls
that are still theirs.  Ids are exact, scores within 1e-5 (they are the same bits: the oracle's operations in its order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
import test_gpu_segments as seg  # noqa: E402
from gpu_helpers import DEV, dev  # noqa: E402
from oracle import OracleTree  # noqa: E402
from test_gpu_ragged import _check  # noqa: E402
from test_gpu_rows import _near_ties, _outputs  # noqa: E402


def _lists(rng, V, blank, kind):
    ids = np.array([v for v in range(V) if v != blank], dtype=np.int32)
    if kind == "bushy":  # one token with hundreds of arcs behind it, many one-token phrases
        phrases = [[ids[0], t] for t in ids[::2][:600]] + [[ids[0], ids[0], t] for t in ids[1::3][:200]] + [[t] for t in ids[:40]]
    elif kind == "deep":  # runs of one token: every suffix is in the tree, failure chains as long as the run
        phrases = [[ids[3]] * 9 + [ids[5]], [ids[3]] * 7 + [ids[4]], [ids[3], ids[4], ids[3], ids[4], ids[3], ids[6]]]
        phrases += [list(rng.choice(ids[:8], rng.integers(1, 7))) for _ in range(60)]
    else:
        phrases = [list(ids[np.minimum(rng.zipf(1.2, rng.integers(1, 8)) - 1, len(ids) - 1)]) for _ in range(300)]
    offs = np.cumsum([0] + [len(p) for p in phrases]).astype(np.int64)
    return np.concatenate([np.asarray(p, dtype=np.int32) for p in phrases]), offs


def _compare(tr, ot, x, s0, last0, alpha, where):
    T, B, V = x.shape
    d_x = dev(x)
    for mode in (0, 1, 2):
        o = _outputs(T, B)
        print("walk", where, mode, flush=True)
        pb.pb_fuse_frames_select(tr, d_x, B * V, V, dev(s0), dev(last0), alpha, T, B, mode, o[0], o[1], o[2], 0)
        torch.cuda.synchronize()
        _check(o, ot.fuse_frames_select(x, s0, last0, alpha, mode), list(range(B)), (where, mode))


@pytest.mark.parametrize("kind", ["zipf", "bushy", "deep"])
@pytest.mark.parametrize("V,T,B", [(128, 160, 2), (200, 60, 3), (257, 1, 2), (257, 100, 4), (512, 15, 3), (513, 16, 3), (512, 128, 4), (769, 17, 2), (1000, 512, 2),
                                   (1024, 255, 3), (1024, 257, 2), (1025, 1025, 2), (1280, 65, 3), (1281, 1030, 1), (4096, 40, 2),
                                   (32768, 33, 2), (32769, 33, 2)])
def test_phrases_spoken(V, T, B, kind):
    rng = np.random.default_rng(91000 + V + T)
    torch.manual_seed(V + T)
    blank = int(rng.choice([-1, 0, V - 1]))
    toks, offs = _lists(rng, V, blank, kind)
    wmode, alpha = int(rng.integers(0, 3)), float(rng.choice([0.3, 1.0, -0.5]))
    ot = OracleTree(toks, offs, V, blank, weight_mode=wmode)
    tr = pb.pb_build(toks, offs, V, blank, device=0, weight_mode=wmode)
    x = seg._spoken(rng, T, B, V, [(toks, offs)]) if T > 12 else torch.round(torch.randn((T, B, V), device=DEV) * 4) / 2
    if blank >= 0:
        x[torch.rand((T, B), device=DEV) < 0.4, blank] += 14.0
    s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
    _compare(tr, ot, x.cpu().numpy(), s0, rng.integers(-1, V, B).astype(np.int32), alpha, (V, T, B, kind, blank, wmode, alpha))
    pb.pb_free(tr)


@pytest.mark.parametrize("V,T", [(300, 100), (1000, 130), (1100, 130), (20001, 70)])
def test_every_frame_needs_its_row(V, T):
    rng = np.random.default_rng(92000 + V)
    toks, offs = _lists(rng, V, V - 1, "zipf")
    ot = OracleTree(toks, offs, V, V - 1)
    tr = pb.pb_build(toks, offs, V, V - 1, device=0)
    x = _near_ties(rng, tr, T, 2, V, 0.5)
    s0 = rng.integers(0, ot.num_states, 2).astype(np.int32)
    _compare(tr, ot, x, s0, rng.integers(-1, V, 2).astype(np.int32), 0.5, (V, T))
    pb.pb_free(tr)


@pytest.mark.parametrize("V", [1025, 1152, 1280, 1281, 2047, 2048, 2049, 2500, 4095, 4096, 5125, 9217, 16381, 16384])
def test_segment_decoders_on_long_calls(V, monkeypatch):
    monkeypatch.setitem(seg.SEGMENTS, V, (2050, 3))
    seg.test_segment_decoders_past_the_dispatch_line(V, V % 4 == 0, V % 2 == 0)


def test_which_trees_have_a_table_of_arcs():
    """Trees of vocabularies whose calls never take the two passes do without."""
    rng = np.random.default_rng(97000)
    pad = lambda n: (n + 255) // 256 * 256  # noqa: E731
    for V in (100, 127, 128, 1000, 20001):
        for eos in (-1, V - 2):
            toks, offs = _lists(rng, V, V - 1, "deep")
            toks = np.where(toks == eos, 1, toks).astype(np.int32)
            tr = pb.pb_build(toks, offs, V, V - 1, device=0, eos_id=eos)
            n = pb.pb_info(tr)["num_states"]
            arrays = pad(32 * n) + pad(8 * (n - 1)) + 2 * pad(4 * V) + pad(4 * n) + pad(32 * V) + (pad(4 * n) if eos >= 0 else 0)
            slots = 16 * max(16, 2 << (n - 1).bit_length()) if V >= 128 else 0
            assert pb.pb_info(tr)["device_bytes"] == arrays + pad(slots)
            ot = OracleTree(toks, offs, V, V - 1, eos_id=eos)
            s0 = rng.integers(0, n, 2).astype(np.int32)
            x = seg._spoken(rng, 40, 2, V, [(toks, offs)])
            _compare(tr, ot, x.cpu().numpy(), s0, rng.integers(-1, V, 2).astype(np.int32), 0.5, (V, eos))
            pb.pb_free(tr)


@pytest.mark.parametrize("V,T", [(32768, 1030), (32769, 1025), (40961, 1100)])
def test_more_frames_than_a_block_holds_in_one_word_and_in_two(V, T):
    """Past 32768 tokens what the first pass finds of a row lies in two output words, and the frames past the first block
    read both of them."""
    rng = np.random.default_rng(96000 + V)
    torch.manual_seed(V)
    toks, offs = _lists(rng, V, V - 1, "zipf")
    ot = OracleTree(toks, offs, V, V - 1, weight_mode=1)
    tr = pb.pb_build(toks, offs, V, V - 1, device=0, weight_mode=1)
    x = seg._spoken(rng, T, 1, V, [(toks, offs)])
    x[torch.rand((T, 1), device=DEV) < 0.4, V - 1] += 14.0
    s0 = rng.integers(0, ot.num_states, 1).astype(np.int32)
    _compare(tr, ot, x.cpu().numpy(), s0, rng.integers(-1, V, 1).astype(np.int32), 0.5, (V, T))
    pb.pb_free(tr)


@pytest.mark.parametrize("V", [300, 1025, 2500])
def test_zeros_of_both_signs(V):
    """0.0 and -0.0 are equal values: the lower token wins, among arcs and among the tokens of a row that needs a pass."""
    rng = np.random.default_rng(93000 + V)
    toks, offs = _lists(rng, V, V - 1, "bushy")
    weights = np.where(rng.random(len(offs) - 1) < 0.5, 1.0, -1.0).astype(np.float32)
    ot = OracleTree(toks, offs, V, V - 1, weights=weights)
    tr = pb.pb_build(toks, offs, V, V - 1, weights=weights, device=0)
    T, B = 70, 2
    x = np.where(rng.random((T, B, V)) < 0.05, np.where(rng.random((T, B, V)) < 0.5, 0.0, -0.0), -1.0).astype(np.float32)
    x[::3, :, 0] = 0.0                                   # (the token with hundreds of arcs behind it)
    s0 = rng.integers(0, ot.num_states, B).astype(np.int32)
    for alpha in (0.0, -0.0):                            # (times a negative score, or a positive one: -0.0)
        _compare(tr, ot, x, s0, rng.integers(-1, V, B).astype(np.int32), alpha, (V, alpha))
    pb.pb_free(tr)


@pytest.mark.parametrize("V", [300, 1025, 2500])
def test_chains_longer_than_a_turn_and_than_the_levels_counted(V):
    """Runs of one token: failure chains of up to 2100 states, the winning arc in any of them, also where an arc's order has
    counted its last level (2047)."""
    rng = np.random.default_rng(94000 + V)
    n, a = 2100, 3
    depths = [1, 2, 5, 50, 52, 53, 54, 55, 1000, 2095, 2096, 2097, 2099]
    phrases = [[a] * n] + [[a] * k + [20 + i] for i, k in enumerate(depths)]
    offs = np.cumsum([0] + [len(p) for p in phrases]).astype(np.int64)
    toks = np.concatenate([np.asarray(p, dtype=np.int32) for p in phrases])
    weights = np.full(len(phrases), 0.001, dtype=np.float32)
    ot = OracleTree(toks, offs, V, V - 1, weights=weights)
    tr = pb.pb_build(toks, offs, V, V - 1, weights=weights, device=0)
    T, B = 12, len(depths)
    x = np.round(rng.standard_normal((T, B, V)).astype(np.float32) * 4) / 4
    for i in range(B):
        x[int(rng.integers(0, 3)), i, 20 + i] += 12.0
        x[6:, i, a] += 12.0
    deepest = int(np.argmax(pb.pb_host_arrays(tr)["depth"]))
    s0 = np.full(B, deepest, dtype=np.int32)
    s0[::3] -= rng.integers(0, 40, len(s0[::3])).astype(np.int32)
    _compare(tr, ot, x, s0, rng.integers(-1, V, B).astype(np.int32), 0.5, (V,))
    pb.pb_free(tr)


@pytest.mark.parametrize("kind", ["zipf", "bushy", "deep"])
@pytest.mark.parametrize("V,T", [(200, 130), (513, 40), (1000, 510), (1025, 130), (1281, 300), (20001, 70)])
def test_most_frames_surprise_the_winners(V, T, kind):
    """Log-depth weights at alpha 1 on rows without blanks: frames come out otherwise than the winners say, one after the other,
    in states of few arcs and of hundreds, on chains of any length, with and without EOS, one tree and a table of two."""
    rng = np.random.default_rng(95000 + V + T)
    torch.manual_seed(V + T)
    B = 2
    for blank, eos, table in ((V - 1, -1, False), (-1, V - 2, False), (0, -1, True)):
        lists = [_lists(rng, V, blank, kind) for _ in range(2 if table else 1)]
        if eos >= 0:
            lists = [(np.where(t == eos, 1, t).astype(np.int32), o) for t, o in lists]
        ots = [OracleTree(t, o, V, blank, weight_mode=1, eos_id=eos, final_eos_score=0.75) for t, o in lists]
        trs = [pb.pb_build(t, o, V, blank, device=0, weight_mode=1, eos_id=eos, final_eos_score=0.75) for t, o in lists]
        x = seg._spoken(rng, T, B, V, lists)
        s0 = np.array([rng.integers(0, ots[b % len(ots)].num_states) for b in range(B)], dtype=np.int32)
        last0 = rng.integers(-1, V, B).astype(np.int32)
        if not table:
            _compare(trs[0], ots[0], x.cpu().numpy(), s0, last0, 1.0, (V, T, kind, blank, eos))
        else:
            forest = pb.pb_forest_build(trs)
            for mode in (0, 1, 2):
                o = _outputs(T, B)
                print("walk forest", V, T, kind, mode, flush=True)
                pb.pb_fuse_frames_forest(forest, x, B * V, V, dev(np.arange(B, dtype=np.int32)), dev(s0), dev(last0), 1.0, T, B, mode,
                                         o[0], o[1], o[2], 0)
                torch.cuda.synchronize()
                for b in range(B):
                    want = ots[b].fuse_frames_select(np.ascontiguousarray(x[:, b:b + 1].cpu().numpy()), s0[b:b + 1], last0[b:b + 1], 1.0, mode)
                    _check([g[:, b:b + 1] for g in o], want, [0], (V, T, kind, mode, b))
            pb.pb_forest_free(forest)
        for t in trs:
            pb.pb_free(t)
