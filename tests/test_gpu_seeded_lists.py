"""Lists that start from the seed pass's thresholds against lists that cannot: with
64 candidates no threshold is read from the slots, so the first k of those lists
are what k candidates must give, bit for bit (the keys are exact).  Sizes on both
sides of the sample's rules, reads and windows without a location, fewer windows
than a list holds that are not zero, groups of uneven size."""
import numpy as np
import pytest

import synth
from paper_2603_22245_amd import _lib as L

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _lists(indexes, batches, k):
    torch = torch_cuda()
    ci = [torch.full((b.n, k), -7, dtype=torch.int32, device="cuda") for b in batches]
    cs = [torch.full((b.n, k), -7.0, dtype=torch.float32, device="cuda") for b in batches]
    idx, n = [i.idx for i in indexes], [b.n for b in batches]
    nbytes = L.rm_score_groups_workspace_bytes(idx, n, k, None)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    L.rm_score_topk_groups(idx, [b.emb for b in batches], [b.scale for b in batches], n, k, ci, cs,
                           ws, nbytes, None)
    torch.cuda.synchronize()
    return ci, cs


def _reads(index, ref, n, seed, error=0.02):
    from paper_2603_22245_amd import mapper
    N = index.params.window_len
    rng = np.random.default_rng(seed)
    at = rng.integers(0, ref.size - N + 1, n)
    heads = ref[at[:, None] + np.arange(N)]
    heads = np.where(rng.random(heads.shape) < error, rng.integers(0, 4, heads.shape), heads)
    heads[rng.random(n) < 0.05] = 4                          # no letter: the zero vector
    lens = np.full(n, N)
    lens[rng.random(n) < 0.05] = N - 1                       # too short
    keep = np.arange(N) < lens[:, None]
    rb = mapper.upload_reads(index, heads[keep].astype(np.uint8),
                             np.concatenate([[0], np.cumsum(lens)]).astype(np.int64))
    mapper.encode_reads(index, rb)
    return rb


def _check(indexes, batches, ks):
    torch = torch_cuda()
    base_i, base_s = _lists(indexes, batches, 64)
    for k in ks:
        got_i, got_s = _lists(indexes, batches, k)
        for g in range(len(batches)):
            assert torch.equal(got_i[g], base_i[g][:, :k]) and torch.equal(got_s[g], base_s[g][:, :k])


@pytest.mark.parametrize("precision,n_windows,n_reads", [
    ("fp16", 1, 3), ("fp8", 33, 40), ("fp16", 1_000, 700), ("fp32", 1_500, 300), ("fp16", 5_000, 2_000),
    ("fp16", 5_000, 30_000), ("fp8", 20_001, 12_000), ("fp32", 20_001, 900), ("fp32", 3_000, 6_000),
    ("fp8", 150_000, 33), ("fp16", 150_000, 1_100), ("fp32", 150_000, 5)])
def test_seeded_lists_equal_unseeded(precision, n_windows, n_reads):
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(n_windows + 149, seed=41, uniform=True)
    index = mapper.build_index(ref, precision=precision)
    _check([index], [_reads(index, ref, n_reads, n_reads)], (1, 8, 16, 32))


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp8"])
def test_few_windows_that_are_not_zero(precision):
    from paper_2603_22245_amd import mapper
    ref = np.full(149 + 2_000 * 50, 4, np.uint8)
    ref[40_000:40_300] = synth.make_reference(300, seed=43, uniform=True)
    index = mapper.build_index(ref, stride=50, precision=precision)
    rb = _reads(index, ref[39_950:40_350], 60, 44, error=0.0)
    _check([index], [rb], (8, 16, 32))


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp8"])
def test_groups_of_uneven_size(precision):
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(60_000, seed=45, uniform=True)
    indexes = [mapper.build_index(ref[:g], window_len=n, stride=s, precision=precision)
               for g, n, s in ((60_000, 100, 1), (60_000, 200, 2), (3_000, 400, 4), (900, 800, 8))]
    batches = [_reads(i, ref[:i.idx.ref_len], n, n) for i, n in zip(indexes, (500, 30, 1_300, 5))]
    _check(indexes, batches, (8, 16, 32))
