"""Scoring launches with few reads or few windows: the default plan cuts them
into many chunks and seeds every read's threshold from a sample of the
windows.  Its lists are compared bit for bit with those of one chunk per read
tile (explicit tuning): both hold exact keys, so no tolerance applies."""
import numpy as np
import pytest

import synth
from paper_2603_22245_amd import _lib as L

from gpu_helpers import torch_cuda


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp8"])
@pytest.mark.parametrize("n_windows", [1, 5_000, 200_000, 10_000_000])
def test_workspace_of_more_reads_serves_fewer(precision, n_windows):
    p = L.make_params(150, 1, 32, "default", precision, 0, 1, 0, None, False)
    G = n_windows + 149
    idx = L.rm_index(p=p, ref_len=G, n_windows=n_windows)
    for f in ("d_emb", "d_scale", "d_norm2", "d_phase64", "d_phase32", "d_step32"):
        setattr(idx, f, 256)
    for k_fetch in (8, 16, 32, 64):
        sizes = [L.rm_score_workspace_bytes(idx, n, k_fetch)
                 for n in (1, 8, 32, 33, 100, 128, 129, 200, 300, 500, 1000, 1024, 1025, 1500,
                           2000, 3000, 5000, 8000, 9000, 20_000)]
        assert sizes == sorted(sizes) and sizes[0] > 0
        assert sizes[0] <= L.RM_NOALLOC_SCRATCH_BYTES


def _score(index, rb, k_fetch, ws_bytes, tune=None):
    torch = torch_cuda()
    ci = torch.full((rb.n, k_fetch), -7, dtype=torch.int32, device="cuda")
    cs = torch.full((rb.n, k_fetch), -7.0, dtype=torch.float32, device="cuda")
    ws = torch.full((ws_bytes,), 255, dtype=torch.uint8, device="cuda")
    L.rm_score_topk_groups([index.idx], [rb.emb], [rb.scale], [rb.n], k_fetch, [ci], [cs], ws,
                           ws_bytes, tune)
    torch.cuda.synchronize()
    return ci, cs


# windows: one, a partial tile, a tile and one, past one plan unit, past one
# sample; reads: one, a fragment and one, the 128-read tile's edges, the line
# between the read tiles
@pytest.mark.gpu
@pytest.mark.parametrize("precision,n_windows,n_reads,k_fetch", [
    ("fp16", 1, 1, 16), ("fp8", 31, 17, 8), ("fp32", 33, 129, 16), ("fp16", 65, 128, 32),
    ("fp8", 4097, 1024, 16), ("fp16", 4097, 1025, 8), ("fp32", 20_001, 33, 32),
    ("fp16", 150_000, 5, 16), ("fp8", 150_000, 300, 32), ("fp16", 20_001, 40, 64),
    ("fp8", 700_000, 1, 8)])
def test_default_plan_equals_one_chunk(precision, n_windows, n_reads, k_fetch):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    ref = synth.make_reference(n_windows + 149, seed=95, uniform=True)
    text = ref if ref.size >= 400 else np.concatenate([ref, synth.make_reference(400, seed=97,
                                                                                 uniform=True)])
    reads = synth.simulate_reads(text, np.full(n_reads, 150), 0.01, 0.005, 0.005, seed=96)
    index = mapper.build_index(ref, precision=precision)
    rb = mapper.upload_reads(index, reads.seq, reads.offsets)
    mapper.encode_reads(index, rb)
    one = L.rm_tuning(128, 1 << 20)
    ws = lambda tune: L.rm_score_groups_workspace_bytes([index.idx], [n_reads], k_fetch, tune)
    base = _score(index, rb, k_fetch, ws(one), one)
    got = _score(index, rb, k_fetch, ws(None))
    assert torch.equal(got[0], base[0]) and torch.equal(got[1], base[1])
