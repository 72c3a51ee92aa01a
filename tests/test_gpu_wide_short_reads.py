"""The 1,024-component product with reads that are too short, which score 0 with every
window: the other reads' lists are those of the batch without them, their own are
empty, and they do not hold up the launch.  Keys are exact; no tolerance applies."""
import numpy as np
import pytest

import synth

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _batch(precision, n_windows, n_reads, short, period=0):
    """A function from read numbers to their ReadBatch, and the index; `short` reads
    lack one letter."""
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(n_windows + 149, seed=71, uniform=True)
    if period:
        ref = np.resize(ref[:period], ref.size)
    s, m, n_class, token_map, schedule = synth.token_encoding("s4m4")
    index = mapper.build_index(ref, precision=precision, schedule=schedule, mer_len=s, n_freq=m,
                               n_class=n_class, token_map=token_map)
    at = np.random.default_rng(72).integers(0, n_windows, n_reads)

    def upload(ids):
        lens = np.where(short[ids], 149, 150)
        seq = np.concatenate([ref[at[i]:at[i] + n] for i, n in zip(ids, lens)])
        rb = mapper.upload_reads(index, seq, np.concatenate([[0], np.cumsum(lens)]))
        mapper.encode_reads(index, rb)
        return rb
    return index, upload


@pytest.mark.parametrize("precision,n_windows,n_reads,k_fetch,period", [
    ("fp8", 9_000, 40, 32, 0), ("fp16", 5_000, 300, 8, 0), ("fp8", 300, 5, 16, 0),
    ("fp16", 700, 20, 1, 0), ("fp8", 5_000, 2_100, 32, 97)])
def test_short_reads_leave_the_others_alone(precision, n_windows, n_reads, k_fetch, period):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    short = np.random.default_rng(73).random(n_reads) < 0.3
    short[0], short[1] = True, False
    index, upload = _batch(precision, n_windows, n_reads, short, period)

    def lists(ids):
        bufs = mapper.map_buffers(index, len(ids), 1, k_fetch)
        mapper.score_topk(index, upload(ids), bufs)
        return bufs.cand_idx, bufs.cand_score
    idx, score = lists(np.arange(n_reads))
    own_idx, own_score = lists(np.flatnonzero(~short))
    keep = torch.from_numpy(~short).cuda()
    assert torch.equal(idx[keep], own_idx) and torch.equal(score[keep], own_score)
    assert bool((idx[~keep] == -1).all()) and bool((score[~keep] == 0).all())
    assert bool((own_idx >= 0).all())


def test_short_reads_do_not_hold_up_the_launch():
    """Reads without a score take no turns: with one in ten the launch takes less than
    half as long again (as long without, almost three times when zeros were ranked)."""
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    n = 500
    times = []
    for share in (0.0, 0.1):
        short = np.random.default_rng(74).random(n) < share
        index, upload = _batch("fp8", 75_000, n, short)
        rb, bufs = upload(np.arange(n)), mapper.map_buffers(index, n, 1, 8)
        took = []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            mapper.score_topk(index, rb, bufs)
            b.record()
            b.synchronize()
            took.append(a.elapsed_time(b))
        times.append(min(took))
    assert times[1] < 1.5 * times[0], times
