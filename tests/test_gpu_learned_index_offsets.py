"""Offsets at the edges of what the learned index takes: angles of any size in the
directly summed windows, and rows of tokens that are none of the four letters."""
import numpy as np
import pytest

from oracle import rope

from gpu_helpers import emb_to_complex, torch_cuda

pytestmark = pytest.mark.gpu


def _index(ref, delta, N, stride, reanchor):
    torch = torch_cuda()
    from paper_2603_22245_amd import _lib as L, mapper
    p = L.make_params(N, stride, 32, "default", "fp32", reanchor, 1, 4, None, False)
    d_ref, d_delta = torch.from_numpy(ref).cuda(), torch.from_numpy(delta).cuda()
    nbytes = L.rm_index_bytes(ref.size, p)
    buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    idx = mapper.Index(p, L.rm_encode_reference_learned(d_ref, ref.size, p, d_delta, buf, nbytes),
                       buf, d_ref)
    torch.cuda.synchronize()
    return emb_to_complex(idx, torch)


@pytest.mark.parametrize("size", [1e6, 1e9, 1e10, 1e14, 1e20, 3e38])
def test_direct_sums_take_offsets_of_any_size(size):
    """Every window its own segment: an FP64 sum of at most 16 terms, rounded to
    FP32, and divided by a norm whose 256 squares are added in FP32 (2^-17)."""
    N, n = 24, 90
    rng = np.random.default_rng(7)
    ref = rng.integers(0, 4, n).astype(np.uint8)
    delta = (rng.uniform(-1, 1, (n - 8, 32)) * size).astype(np.float32)
    delta[::3] = rng.normal(0, 1, delta[::3].shape)
    got = _index(ref, delta, N, 1, 1)
    theta = 2 * np.pi * np.asarray(rope.frequencies(32, "default"), np.float64) / N
    for j in range(n - N + 1):
        C = np.zeros((32, 4), np.complex128)
        for q in range(N - 8):
            C[:, ref[j + q + 4]] += np.exp(1j * q * theta) * np.exp(1j * delta[j + q].astype(np.float64))
        C = C.ravel() / np.linalg.norm(C)
        assert np.max(np.abs(got[j] - C)) <= 2.0 ** -16, j


@pytest.mark.parametrize("stride,reanchor", [(1, 0), (3, 0), (1, 7)])
def test_rows_of_other_letters_are_not_read(stride, reanchor):
    N, n = 40, 400
    rng = np.random.default_rng(8)
    ref = rng.integers(0, 4, n).astype(np.uint8)
    ref[rng.random(n) < 0.1] = 4
    ref[50:70] = 9
    delta = rng.normal(0, 1, (n - 8, 32)).astype(np.float32)
    delta[ref[4:n - 4] > 3] = 0
    want = _index(ref, delta, N, stride, reanchor)
    delta[ref[4:n - 4] > 3] = np.nan
    got = _index(ref, delta, N, stride, reanchor)
    assert np.all(np.isfinite(want))
    np.testing.assert_array_equal(got, want)
