"""Read heads on the matrix cores: blocks of 4 or 32 reads, chunks of 64 positions
in steps of four.  Every component is the FP32 sum of the phase table over its
letter's positions in their order, so the FP32 rows are compared with that sum
taken on the CPU; the norm, a reciprocal root and a product round a few times
more: 8 ulps (2^-21) of a component, and 2^-21 of the row's length for those
that cancel."""
import numpy as np
import pytest

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_reads,N", [(1, 33), (3, 64), (4, 65), (5, 130), (33, 150), (7, 1),
                                       (16_385, 40), (16_384, 67)])
def test_rows_are_ordered_sums(n_reads, N):
    torch = torch_cuda()
    from paper_2603_22245_amd import mapper
    rng = np.random.default_rng(N)
    index = mapper.build_index(rng.integers(0, 4, 400 + N).astype(np.uint8), window_len=N,
                               precision="fp32", reduced=False)
    lens = N + rng.integers(0, 9, n_reads)
    lens[rng.random(n_reads) < 0.1] = max(N - 1, 0)          # too short: the zero vector
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    seq = rng.integers(0, 4, off[-1]).astype(np.uint8)
    seq[rng.random(seq.size) < 0.02] = 7                      # unknown letters
    rb = mapper.upload_reads(index, np.concatenate([seq, np.zeros(1, np.uint8)]), off)
    mapper.encode_reads(index, rb)
    rows = rb.emb.view(torch.float32).view(n_reads, 2, 256).cpu().numpy().astype(np.float64)
    base = index.idx.d_phase32 - index.buf.data_ptr()
    tab = index.buf[base: base + N * 64 * 4].view(torch.float32).view(N, 64).cpu().numpy()
    for r in range(0, n_reads, max(1, n_reads // 500)):
        want = np.zeros((4, 64), np.float32)
        if lens[r] >= N:
            for p, L in enumerate(seq[off[r]: off[r] + N]):
                if L < 4:
                    want[L] += tab[p]
        w = want.astype(np.float64)
        norm2 = np.sum(w * w)
        w = w / np.sqrt(norm2) if norm2 >= 1e-4 * N else 0 * w
        w = w.reshape(4, 32, 2).transpose(1, 0, 2).reshape(256)          # (factor, letter), re/im
        im = np.stack([-w[1::2], w[0::2]], 1).reshape(256)
        for got, ref in ((rows[r, 0], w), (rows[r, 1], im)):
            assert np.all(np.abs(got - ref) <= 2.0 ** -21 * (np.abs(ref) + 1.0 / 16)), r
