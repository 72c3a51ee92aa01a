"""The 1,024-component product in many groups of blocks: later groups start from
the k-th best keys of earlier ones.  A read's candidates do not depend on how
many others it is scored with, so the lists of many reads at once are compared
bit for bit with those of the same reads a tile (128) at a time, where every
chunk starts from an empty list.  Keys are exact; no tolerance applies."""
import numpy as np
import pytest

import synth

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n_windows,n_reads,k_fetch,period", [
    ("fp8", 40_000, 3_100, 32, 0),     # four groups of read tiles, 16 chunks
    ("fp16", 10_007, 2_049, 16, 0),    # a last read tile of one read, a ragged last window tile
    ("fp8", 20_000, 2_500, 1, 0),
    ("fp8", 9_000, 2_100, 32, 300),    # repeats: a tile holds more equal scores than slots
    ("fp16", 5_000, 2_100, 8, 97),
])
def test_lists_do_not_depend_on_the_batch(precision, n_windows, n_reads, k_fetch, period):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(n_windows + 149, seed=61, uniform=True)
    if period:
        ref = np.resize(ref[:period], ref.size)
    s, m, n_class, token_map, schedule = synth.token_encoding("s4m4")
    index = mapper.build_index(ref, precision=precision, schedule=schedule, mer_len=s, n_freq=m,
                               n_class=n_class, token_map=token_map)
    reads = synth.simulate_reads(ref, np.full(n_reads, 150), 0.02, 0.01, 0.01, seed=62)

    def lists(a, b):
        off = reads.offsets[a:b + 1] - reads.offsets[a]
        rb = mapper.upload_reads(index, reads.seq[reads.offsets[a]:reads.offsets[b]], off)
        bufs = mapper.map_buffers(index, b - a, min(8, k_fetch), k_fetch)
        for t in (bufs.cand_idx, bufs.cand_score):
            t.fill_(-7)
        mapper.map_reads(index, rb, bufs)
        torch.cuda.synchronize()
        return bufs.cand_idx.cpu().numpy(), bufs.cand_score.cpu().numpy()

    idx, score = lists(0, n_reads)
    assert np.all(idx >= 0) and np.all(np.diff(score, axis=1) <= 0)
    for a in range(0, n_reads, 128):
        b = min(n_reads, a + 128)
        one_idx, one_score = lists(a, b)
        np.testing.assert_array_equal(idx[a:b], one_idx)
        np.testing.assert_array_equal(score[a:b], one_score)
