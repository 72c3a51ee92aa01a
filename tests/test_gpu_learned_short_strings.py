"""Encodings of many short strings: blocks that take several groups of strings, and
groups whose tokens of a letter share one tile of 16 (up to 16 tokens) or not.
Against the FP64 oracle; a component sums at most n unit terms in FP32, 1e-5 n."""
import numpy as np
import pytest

from oracle import learned as OL

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,longest", [(1, 9), (5, 12), (8, 16), (1030, 11), (2051, 12),
                                       (2600, 40)])
def test_groups_of_short_strings(n, longest):
    torch = torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(n)
    seqs = [rng.integers(0, 4, rng.integers(7, longest + 1)).astype(np.uint8) for _ in range(n)]
    for w in seqs[::7]:
        w[rng.random(w.size) < 0.2] = 5
    seqs[n // 2] = np.full(longest + 8, 2, np.uint8)         # a letter's tokens at the tile's edge
    off = np.concatenate([[0], np.cumsum([w.size for w in seqs])]).astype(np.int64)
    W1, b1, W2, b2 = OL.unpack(OL.init_params(3))
    p = OL.pack(W1, b1, rng.normal(0, 0.05, W2.shape), rng.normal(0, 0.4, b2.shape)).astype(np.float32)
    c = learned.encode(torch.from_numpy(p).cuda(), torch.from_numpy(np.concatenate(seqs)).cuda(),
                       torch.from_numpy(off).cuda(), n, 150).cpu().numpy().astype(np.float64)
    for i in list(range(0, n, max(1, n // 300))) + [n // 2, n - 1]:
        want, _ = OL.forward_string(p.astype(np.float64), seqs[i], 150)
        got = c[i, 0::2] + 1j * c[i, 1::2]
        assert np.max(np.abs(got - want)) <= 1e-5 * seqs[i].size, i
