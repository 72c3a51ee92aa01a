"""The edit-distance kernel's 16 pairs per wavefront, four 64-letter words per
pair, letters staged in LDS when both sides' fit: exact against the oracle's
dynamic programme."""
import numpy as np
import pytest

from oracle import lev

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _pack(seqs):
    off = np.zeros(len(seqs) + 1, np.int64)
    off[1:] = np.cumsum([len(s) for s in seqs])
    return (np.concatenate(seqs).astype(np.uint8) if off[-1] else np.zeros(1, np.uint8)), off


@pytest.mark.parametrize("n,longest", [(1, 20), (15, 64), (16, 65), (17, 128), (33, 256), (18, 3000)])
def test_edit_distance_words_and_staging(n, longest):
    torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(n + longest)
    a = [rng.integers(0, 4, rng.integers(0, min(longest, 256) + 1)).astype(np.uint8)
         for _ in range(n)]
    b = [rng.integers(0, 4, rng.integers(0, longest + 1)).astype(np.uint8) for _ in range(n)]
    for i in range(0, n, 3):  # near pairs
        b[i] = np.concatenate([a[i][:5], a[i][6:], rng.integers(0, 4, 3).astype(np.uint8)])
    for i in range(1, n, 4):  # in either order
        a[i], b[i] = (b[i], a[i]) if len(b[i]) <= 256 else (a[i], b[i])
    want = lev.lev_many(*_pack(a), *_pack(b))
    got = learned.levenshtein(learned.upload_pairs(*_pack(a), *_pack(b))).cpu().numpy()
    np.testing.assert_array_equal(got, want)


def test_edit_distance_unknown_letters_match_nothing():
    torch_cuda()
    from paper_2603_22245_amd import learned
    a = [np.array([0, 4, 2], np.uint8), np.array([200, 1], np.uint8)]
    b = [np.array([0, 4, 2], np.uint8), np.array([1], np.uint8)]
    got = learned.levenshtein(learned.upload_pairs(*_pack(a), *_pack(b))).cpu().numpy()
    assert list(got) == [1, 1]
