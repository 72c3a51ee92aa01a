"""The FP32 rescore of lists with missing candidates: where a list's entries stand
does not matter, whether they share a block of eight strings with the head, with
others or with none.  The same kernel forms every score, so lists are equal bit for
bit."""
import numpy as np
import pytest

import synth

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window", [20, 150, 333])
@pytest.mark.parametrize("k_fetch", [8, 16, 24, 31, 33, 48, 64])
def test_place_of_the_candidates(window, k_fetch):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    rng = np.random.default_rng(81)
    ref = synth.make_reference(3_000, seed=82, uniform=True)
    index = mapper.build_index(ref, window, precision="fp16")
    W = index.n_windows
    n, k = 50, min(8, k_fetch)
    at = rng.integers(0, W, n)
    lens = np.full(n, window)
    lens[[3, 17]] = window - 1  # no head
    seq = np.concatenate([ref[a:a + m] for a, m in zip(at, lens)])
    rb = mapper.upload_reads(index, seq, np.concatenate([[0], np.cumsum(lens)]))
    bufs = mapper.map_buffers(index, n, k, k_fetch)

    def rescored(cand):
        bufs.cand_idx.copy_(torch.from_numpy(cand.astype(np.int32)))
        bufs.top_idx.fill_(-7)
        mapper.rescore(index, rb, bufs)
        return bufs.top_idx.clone(), bufs.top_score.clone()
    front = np.full((n, k_fetch), -1)
    for r in range(n):
        own = rng.choice(W, size=int(rng.integers(0, 5)), replace=False)
        front[r, :own.size] = own
    spread = np.full_like(front, -1)
    for r in range(n):
        own = front[r][front[r] >= 0]
        first = int(rng.integers(0, k_fetch - own.size + 1))  # a block of its own, or two
        places = first + np.arange(own.size) if r % 2 else rng.choice(k_fetch, own.size, False)
        spread[r, places] = own
    spread[spread < 0] = rng.choice([-1, -5, W, 2**31 - 1], int((spread < 0).sum()))  # no windows
    a, b = rescored(front), rescored(spread)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    found = (a[0] >= 0).sum(1).cpu().numpy()
    want = np.minimum((front >= 0).sum(1), k)
    want[[3, 17]] = 0
    np.testing.assert_array_equal(found, want)
