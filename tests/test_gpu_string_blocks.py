"""Rescore and thresholds take the fidelities of eight strings of a row block
together: numbers of strings around the blocks of 8 and the passes of 24 and 40,
heads and candidates that are missing, windows past one 64-position chunk.
Rescored scores against the FP64 oracle: an FP32 sum over at most N unit terms
and a ratio of three such sums keep F within 5e-6."""
import numpy as np
import pytest

import synth
from oracle import rope

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k_fetch", [1, 6, 7, 8, 15, 16, 23, 24, 31, 39, 40, 64])
@pytest.mark.parametrize("N", [40, 64, 131])
def test_rescored_scores_at_block_edges(k_fetch, N):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(700, seed=7, uniform=True)
    rng = np.random.default_rng(k_fetch)
    n = 6                                                   # one full block of reads and a half
    reads = synth.simulate_reads(ref, np.full(n, N + 3), 0.02, 0.01, 0.01, seed=8)
    off = reads.offsets.copy()
    seq = reads.seq.copy()
    seq[off[2]: off[3]] = 1                                 # degenerate head: no location
    index = mapper.build_index(ref, window_len=N, precision="fp32")
    rb = mapper.upload_reads(index, seq, off)
    bufs = mapper.map_buffers(index, n, k_fetch, k_fetch)
    W = index.n_windows
    cand = np.stack([rng.permutation(W)[:k_fetch] for _ in range(n)]).astype(np.int32)
    cand[1, k_fetch // 2] = -1
    cand[3, 0] = W                                          # past the last window
    bufs.cand_idx.copy_(torch.from_numpy(cand))
    mapper.rescore(index, rb, bufs)
    ti, ts = bufs.top_idx.cpu().numpy(), bufs.top_score.cpu().numpy()
    for r in range(n):
        ids = cand[r][(cand[r] >= 0) & (cand[r] < W)]
        x = rope.encode_raw(seq[off[r]: off[r] + N], N, 32)
        want = {}
        for j in ids:
            c = rope.encode_raw(ref[j: j + N], N, 32)
            X, C = np.sum(np.abs(x) ** 2), np.sum(np.abs(c) ** 2)
            want[int(j)] = 0.0 if X < 1e-4 * N else abs(np.vdot(x, c)) ** 2 / (X * C)
        got = {int(i): float(s) for i, s in zip(ti[r], ts[r]) if i >= 0}
        assert set(got) == {j for j, F in want.items() if F > 0}, r
        assert all(abs(got[j] - want[j]) <= 5e-6 for j in got), r
        assert np.all(np.diff(ts[r]) <= 0) and np.all(ts[r][len(got):] == 0)


@pytest.mark.parametrize("copies", [1, 4, 7, 8, 15, 23, 24, 33, 64])
def test_thresholds_at_block_edges(copies):
    torch_cuda()
    from oracle import thresholds as OT
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(180, seed=9, uniform=True)
    for N, err in ((33, 0.3), (64, 0.05), (100, 0.9)):
        index = mapper.build_index(ref, window_len=N, precision="fp32")
        W = index.n_windows
        thr = mapper.window_thresholds(index, err, copies, copies // 2, seed=5).cpu().numpy()
        for j in sorted({0, W // 2, W - 2, W - 1}):        # the last ones run past the reference
            want = OT.window_threshold(ref, j, 1, N, err, copies, copies // 2, 5)
            assert abs(thr[j] - want) <= 1e-5, (N, copies, j)
