"""The edit-distance kernel's blocks of 64 pairs with one, two or four lanes a pair:
exact against the oracle's dynamic programme, and more pairs than one launch has
threads for."""
import numpy as np
import pytest

from oracle import lev

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _pack(seqs):
    off = np.zeros(len(seqs) + 1, np.int64)
    off[1:] = np.cumsum([len(s) for s in seqs])
    return (np.concatenate(seqs).astype(np.uint8) if off[-1] else np.zeros(1, np.uint8)), off


# pattern lengths at the edges of words and of eight-letter loads, texts shorter,
# equal and much longer; the last row mixes blocks of one, two and four lanes
@pytest.mark.parametrize("n,shortest,longest,text", [
    (1, 1, 9, 9), (63, 1, 64, 80), (64, 63, 65, 70), (65, 120, 128, 140), (130, 127, 129, 600),
    (70, 190, 256, 260), (66, 255, 258, 300), (400, 0, 64, 64), (200, 1, 256, 1500)])
def test_blocks_by_longest_pattern(n, shortest, longest, text):
    torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(n + longest)
    a = [rng.integers(0, 4, rng.integers(shortest, longest + 1)).astype(np.uint8) for _ in range(n)]
    b = [rng.integers(0, 4, rng.integers(shortest, text + 1)).astype(np.uint8) for _ in range(n)]
    if n == 200:  # 64 pairs of one word, then 64 of two, the rest of any
        a = [x[:60] if i < 64 else x[:110] if i < 128 else x for i, x in enumerate(a)]
    for i in range(0, n, 3):  # near pairs, in either order
        b[i] = np.concatenate([a[i][:5], a[i][6:], rng.integers(0, 4, 3).astype(np.uint8)])
        if i % 2:
            a[i], b[i] = b[i], a[i]
    for i in range(0, n, 5):  # letters that match nothing
        for s in (a[i], b[i]):
            s[rng.random(s.size) < 0.2] = [4, 7, 8, 64, 128, 255][i % 6]
    # the oracle compares codes: other letters get one that the other string has not
    other = lambda seqs, code: [np.where(s > 3, code, s).astype(np.uint8) for s in seqs]
    want = lev.lev_many(*_pack(other(a, 100)), *_pack(other(b, 200)))
    want[[min(len(x), len(y)) > 256 for x, y in zip(a, b)]] = -1
    got = learned.levenshtein(learned.upload_pairs(*_pack(a), *_pack(b))).cpu().numpy()
    np.testing.assert_array_equal(got, want)


def test_more_pairs_than_a_launch_has_threads():
    """2^30 + 101 pairs of an empty string and one of one or two letters: four
    threads a pair would be more than 2^32."""
    torch = torch_cuda()
    from paper_2603_22245_amd import _lib as L
    n = (1 << 30) + 101
    b_off = torch.arange(n + 1, dtype=torch.int64, device="cuda").mul_(3).div_(2, rounding_mode="floor")
    a_off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    b = torch.zeros(int(b_off[-1]), dtype=torch.uint8, device="cuda")
    out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    L.rm_levenshtein(b, a_off, b, b_off, n, out)
    torch.cuda.synchronize()
    for i in range(0, n, 1 << 28):
        j = min(n, i + (1 << 28))
        assert torch.equal(out[i:j].long(), b_off[i + 1:j + 1] - b_off[i:j])
