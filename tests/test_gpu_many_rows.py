"""Calls of more rows than a launch of large workgroups may have threads for (2^32): they are decoded all the same."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_07014_amd as pb  # noqa: E402
from gpu_helpers import DEV, dev  # noqa: E402
from test_gpu_ragged import _tree  # noqa: E402


def test_beams_of_five_million_utterances():
    rng = np.random.default_rng(71000)
    V, K, U = 5, 17, 5_000_000            # (more than 16 beams: the streamed form, 1024 threads an utterance)
    toks, offs, ot, tr = _tree(rng, V, 0, -1, 0, 0.0)
    x = torch.randn((U, K, V), device=DEV)
    hyp = -torch.rand((U, K), device=DEV)
    st = torch.randint(0, ot.num_states, (U, K), dtype=torch.int32, device=DEV)
    o = [torch.full((U, K), -7, dtype=torch.int32, device=DEV) for _ in range(3)] + [torch.zeros((U, K), device=DEV)]
    print("beam", V, K, U, flush=True)
    pb.pb_fuse_step_beam(tr, x, V, hyp, st, 0.5, U, K, o[0], o[1], o[2], o[3], 0)
    torch.cuda.synchronize()
    for u in (0, 1, 4_194_303, 4_194_304, U - 1):
        want = ot.fuse_step_beam(x[u].cpu().numpy(), hyp[u].cpu().numpy(), st[u].cpu().numpy(), 0.5, 1, K)
        for g, w in zip(o[:3], want):
            assert np.array_equal(g[u].cpu().numpy(), np.asarray(w).reshape(-1)), u
    pb.pb_free(tr)


def test_frames_of_one_row_repeated():
    """A frame stride of 0 (every frame the same row) makes as many rows as the outputs have room for."""
    rng = np.random.default_rng(72000)
    V, B, T = 16388, 3000, 7600           # 22.8 million rows
    toks, offs, ot, tr = _tree(rng, V, V - 1, -1, 0, 0.0)
    x = torch.randn((B, V), device=DEV) * 2
    s0 = torch.randint(0, ot.num_states, (B,), dtype=torch.int32, device=DEV)
    o = [torch.full((T, B), -7, dtype=torch.int32, device=DEV) for _ in range(2)] + [torch.zeros((T, B), device=DEV)]
    print("frames", V, T, B, flush=True)
    pb.pb_fuse_frames(tr, x, 0, V, s0, 0.5, T, B, o[0], o[1], o[2], 0)
    torch.cuda.synchronize()
    n = 300                               # frame by frame the same: two calls of few frames meet the long one
    p = [torch.full((n, B), -7, dtype=torch.int32, device=DEV) for _ in range(2)] + [torch.zeros((n, B), device=DEV)]
    for first in (0, T - n):
        start = s0 if first == 0 else o[1][first - 1].clone()
        pb.pb_fuse_frames(tr, x, 0, V, start, 0.5, n, B, p[0], p[1], p[2], 0)
        torch.cuda.synchronize()
        for a, b in zip(o, p):
            assert torch.equal(a[first:first + n], b), first
    want = ot.fuse_frames(np.broadcast_to(x[7].cpu().numpy(), (20, 1, V)).copy(), s0[7:8].cpu().numpy(), 0.5)
    assert np.array_equal(o[0][:20, 7].cpu().numpy(), want[0][:, 0]) and np.array_equal(o[1][:20, 7].cpu().numpy(), want[1][:, 0])
    pb.pb_free(tr)


def test_step_of_seventy_million_hypotheses():
    rng = np.random.default_rng(73000)
    V, B = 5, 70_000_000
    toks, offs, ot, tr = _tree(rng, V, 0, -1, 0, 0.0)
    x = torch.randn((B, V), device=DEV)
    st = torch.randint(0, ot.num_states, (B,), dtype=torch.int32, device=DEV)
    o = [torch.full((B,), -7, dtype=torch.int32, device=DEV) for _ in range(2)] + [torch.zeros(B, device=DEV)]
    print("step", V, B, flush=True)
    pb.pb_fuse_step(tr, x, V, st, 0.5, B, o[0], o[1], o[2], 0)
    torch.cuda.synchronize()
    assert not bool((o[0] == -7).any()) and not bool((o[1] == -7).any())
    rows = np.array([0, 1, 4_194_302, 4_194_303, 4_194_304, 67_108_863, 67_108_864, B - 1])
    d_rows = torch.from_numpy(rows).to(DEV)
    xs, ss = x[d_rows].cpu().numpy(), st[d_rows].cpu().numpy()
    for g, w in zip(o, ot.fuse_step(xs, ss, 0.5)):
        assert np.allclose(g[d_rows].cpu().numpy(), w, atol=1e-5, rtol=0)
    pb.pb_free(tr)
