"""Refinement with 1,024-component encodings of 4 factors (changes of a slide side
by side) and of 8 and 16 (one after the other), against the FP64 oracle's
fidelities of every start.  The reference has runs and repeats, so that a slide's
leaving and entering tokens are often of one class.  Tolerance: FP32 sums over a
window's tokens, and compensated sums over the slides, 5e-6 as for the other
refinements."""
import numpy as np
import pytest

import synth
from oracle import mapping, tokens

from gpu_helpers import check_refined_lists, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,m,radius,N", [(4, 4, 31, 40), (5, 4, 7, 60), (4, 4, 0, 150),
                                          (4, 8, 7, 60), (5, 16, 31, 60)])
def test_refinement_by_number_of_factors(s, m, radius, N):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    C = 1024 // m
    token_map = None if 4 ** s == C else (np.arange(4 ** s) % C).astype(np.uint8)
    ref = synth.make_reference(1500, seed=71, uniform=True)
    ref[200:320] = 2                                   # one token over and over
    ref[600:900] = np.resize(ref[600:607], 300)        # period 7
    stride, R, kf = 4, 24, 6
    index = mapper.build_index(ref, window_len=N, stride=stride, precision="fp16", mer_len=s,
                               n_freq=m, n_class=C, token_map=token_map)
    rng = np.random.default_rng(72)
    starts = np.concatenate([rng.integers(0, ref.size - N, R - 4), [210, 250, 620, 700]])
    heads = ref[starts[:, None] + np.arange(N)]
    swap = rng.random(heads.shape) < 0.05
    heads = np.where(swap, rng.integers(0, 4, heads.shape), heads).astype(np.uint8)
    cand = rng.integers(0, index.n_windows, (R, kf)).astype(np.int32)
    cand[:, 0] = np.minimum(starts // stride, index.n_windows - 1)
    cand[0, 1:4] = [0, index.n_windows - 1, -1]
    k = min(8, kf * (2 * radius + 1))
    rb = mapper.upload_reads(index, heads.ravel(), np.arange(R + 1, dtype=np.int64) * N)
    bufs = mapper.map_buffers(index, R, k, kf)
    bufs.cand_idx.copy_(torch.from_numpy(cand).cuda())
    mapper.refine(index, rb, bufs, radius)
    torch.cuda.synchronize()
    Cn, _ = mapping.normalized_rows(
        tokens.encode_windows(ref, np.arange(ref.size - N + 1), N, s, m, C, token_map), N)
    Xn, _ = mapping.normalized_rows(
        np.stack([tokens.encode_raw(h, N, s, m, C, token_map) for h in heads]).reshape(R, -1), N)
    F = mapping.fidelity_matrix(Xn, Cn)
    check_refined_lists(bufs.top_idx.cpu().numpy(), bufs.top_score.cpu().numpy(), cand, F, stride,
                        radius, k, 5e-6)
