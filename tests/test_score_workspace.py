"""Workspace sizes of the scoring calls (no GPU): a size asked for some reads serves
fewer, alone and in groups, and few reads ask for little.  The default plan gives
fewer reads more chunks of the index, so this does not follow from the plan of
the reads themselves."""
import numpy as np
import pytest

from paper_2603_22245_amd import _lib as L

from gpu_helpers import torch_cuda


def _index(precision, n_windows):
    p = L.make_params(150, 1, 32, "default", precision, 0, 1, 0, None, False)
    idx = L.rm_index(p=p, ref_len=n_windows + 149, n_windows=n_windows)
    for f in ("d_emb", "d_scale", "d_norm2", "d_phase64", "d_phase32", "d_step32"):
        setattr(idx, f, 256)
    return idx


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp8"])
@pytest.mark.parametrize("n_windows", [5_000, 20_000, 64_000, 100_000, 300_000, 10_000_000])
def test_more_reads_never_ask_for_less(precision, n_windows):
    idx = _index(precision, n_windows)
    reads = [1, 32, 33] + [128 * t + d for t in range(1, 160) for d in (0, 1)]
    for k_fetch in (8, 16, 32, 64):
        sizes = [L.rm_score_workspace_bytes(idx, n, k_fetch) for n in reads]
        assert sizes == sorted(sizes)


@pytest.mark.parametrize("n_windows", [1_000, 20_000, 10_000_000])
@pytest.mark.parametrize("k_fetch", [8, 16, 64])
def test_few_reads_ask_for_their_lists(n_windows, k_fetch):
    """At most 512 chunks of 64 windows or more for a handful of reads, a list of
    k_fetch 8-byte keys each, and 1 KB for everything else."""
    idx = _index("fp16", n_windows)
    chunks = min(512, -(-n_windows // 64))
    for n in (1, 8, 32):
        assert L.rm_score_workspace_bytes(idx, n, k_fetch) <= n * (chunks * k_fetch * 8 + 512) + 1024


@pytest.mark.parametrize("precision", ["fp16", "fp8", "fp32"])
def test_groups_with_more_reads_never_ask_for_less(precision):
    rng = np.random.default_rng(3)
    windows = [160_000, 160_000, 80_000, 40_000, 20_000, 10_000, 5_000]
    idxs = [_index(precision, w) for w in windows]
    for _ in range(300):
        n_groups = int(rng.integers(2, 8))
        more = np.exp(rng.uniform(0, np.log(20_000), n_groups)).astype(int)
        fewer = np.maximum(1, (more * rng.choice([0.01, 0.5, 0.97, 1.0], n_groups)).astype(int))
        size = lambda r: L.rm_score_groups_workspace_bytes(idxs[:n_groups], [int(x) for x in r], 16,
                                                           None)
        assert size(fewer) <= size(more)


def test_groups_share_the_chip():
    """Seven groups of 350 reads: eight items of 256 reads for each of 256 CUs and
    seven more, and 64 lists a read, of 16 keys."""
    idxs = [_index("fp16", 16_000_000 // s) for s in (1, 2, 4, 8, 16, 32, 64)]
    got = L.rm_score_groups_workspace_bytes(idxs, [350] * 7, 16, None)
    assert got <= (8 * 263 * 256 + 7 * 350 * 65) * 16 * 8 + 7 * 350 * 260 + 16 * 1024


@pytest.mark.gpu
@pytest.mark.parametrize("precision,n_windows,more,fewer,k_fetch", [
    ("fp16", 20_000, 14_114, 13_372, 16), ("fp16", 64_000, 9_291, 8_920, 16),
    ("fp8", 20_000, 13_825, 13_824, 16), ("fp32", 20_000, 6_913, 6_912, 8)])
def test_buffers_of_more_reads_take_fewer(precision, n_windows, more, fewer, k_fetch):
    torch = torch_cuda()
    import synth
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(n_windows + 149, seed=31, uniform=True)
    index = mapper.build_index(ref, precision=precision)
    at = np.random.default_rng(32).integers(0, n_windows, fewer)
    seq = ref[at[:, None] + np.arange(150)].ravel()
    rb = mapper.upload_reads(index, seq, np.arange(fewer + 1, dtype=np.int64) * 150)
    mapper.encode_reads(index, rb)
    large = mapper.map_buffers(index, more, min(8, k_fetch), k_fetch)
    own = mapper.map_buffers(index, fewer, min(8, k_fetch), k_fetch)
    mapper.score_topk(index, rb, large)
    mapper.score_topk(index, rb, own)
    assert torch.equal(large.cand_idx[:fewer], own.cand_idx)
    assert torch.equal(large.cand_score[:fewer], own.cand_score)
