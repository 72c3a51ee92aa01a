"""The learned rolling index over its chunks of 16 slides and its segments, with
given token offsets, against the direct sum in FP64; and the offsets themselves
over tiles of 32 tokens, with other letters.

Tolerances.  A component of a row is a sum kept in FP32 over a segment's slides
and divided by the row's norm: rounding errors of 2^-24 of values that stay
below a few times the norm, a few hundred slides and two terms a slide, each
off by at most 2^-20, that add up like a random walk: 2e-5 is above that by an
order.  FP16 storage adds 2^-11 of the component, FP8 2^-4 of the row's largest.
Offsets of tokens whose middle letter is none of the four are exactly 0."""
import numpy as np
import pytest

from oracle import learned as OL
from oracle import rope

from gpu_helpers import emb_to_complex, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,stride,n,reanchor,schedule,precision", [
    (9, 1, 9, 0, "default", "fp32"),            # one window of one token
    (9, 1, 60, 0, "default", "fp32"),           # each slide replaces the only token
    (17, 1, 17 + 15, 0, "default", "fp32"),     # 15, 16 and 17 slides of a segment
    (24, 1, 24 + 16, 100, "finetuned", "fp32"),
    (24, 1, 24 + 17, 100, "default", "fp16"),
    (40, 5, 700, 7, "default", "fp32"),         # chunks that end inside a stride
    (150, 1, 3000, 1000, "finetuned", "fp32"),
    (150, 2, 4000, 0, "default", "fp8"),
    (150, 23, 4001, 0, "default", "fp32"),      # a stride longer than a chunk
    (233, 1, 2111, 33, "default", "fp16"),
])
def test_index_rows_match_the_direct_sum(N, stride, n, reanchor, schedule, precision):
    torch = torch_cuda()
    from paper_2603_22245_amd import _lib as L, mapper
    rng = np.random.default_rng(N + n)
    ref = rng.integers(0, 4, n).astype(np.uint8)
    ref[rng.random(n) < 0.05] = 4
    ref[4] = 1                                   # the first window is not empty
    delta = rng.normal(0, 0.5, (n - 8, 32)).astype(np.float32)
    delta[rng.random(n - 8) < 0.1] *= 50         # offsets of several turns
    p = L.make_params(N, stride, 32, schedule, precision, reanchor, 1, 4, None, False)
    d_ref, d_delta = torch.from_numpy(ref).cuda(), torch.from_numpy(delta).cuda()
    nbytes = L.rm_index_bytes(n, p)
    buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    idx = mapper.Index(p, L.rm_encode_reference_learned(d_ref, n, p, d_delta, buf, nbytes), buf,
                       d_ref)
    torch.cuda.synchronize()
    got = emb_to_complex(idx, torch)
    theta = 2 * np.pi * np.asarray(rope.frequencies(32, schedule), np.float64) / N
    starts = np.arange(0, n - N + 1, stride)
    assert got.shape[0] == starts.shape[0]
    C = np.zeros((starts.shape[0], 32, 4), np.complex128)
    for q in range(N - 8):
        t = starts + q
        u = np.exp(1j * (q * theta + delta[t].astype(np.float64)))
        for letter in range(4):
            sel = ref[t + 4] == letter
            C[sel, :, letter] += u[sel]
    C = C.reshape(-1, 128)
    norm = np.linalg.norm(C, axis=1, keepdims=True)
    want = np.where(norm > 0, C / np.where(norm > 0, norm, 1), 0)
    tol = 2e-5 * np.ones_like(norm)
    if precision == "fp16":
        tol = tol + 2.0 ** -11 * np.abs(want)
    elif precision == "fp8":
        tol = tol + 2.0 ** -4 * np.max(np.abs(want), axis=1, keepdims=True)
    err = np.abs(got - want)
    assert np.all(err <= tol), float(np.max(err - tol))


@pytest.mark.parametrize("n", [9, 39, 40, 41, 73, 600_000])  # beyond one tile a wavefront
def test_offsets_of_other_letters_and_across_tiles(n):
    torch = torch_cuda()
    from paper_2603_22245_amd import _lib as L
    rng = np.random.default_rng(n)
    W1, b1, W2, b2 = OL.unpack(OL.init_params(5))
    params = OL.pack(W1, b1, rng.normal(0, 0.05, W2.shape),
                     rng.normal(0, 0.4, 128)).astype(np.float32)
    w = rng.integers(0, 6, n).astype(np.uint8)
    d_p, d_w = torch.from_numpy(params).cuda(), torch.from_numpy(w).cuda()
    guard = torch.full((n, 32), float("nan"), device="cuda")  # eight rows beyond the last token
    L.rm_mlp_infer(d_p, d_w, n, guard)
    got = guard.cpu().numpy()
    assert np.all(np.isnan(got[n - 8:])) and np.all(np.isfinite(got[:n - 8]))
    assert np.all(got[:n - 8][w[4:n - 4] > 3] == 0)
    # the same letters in a string of their own give the same bits
    for t in rng.integers(0, n - 8, 8):
        one = torch.empty((1, 32), device="cuda")
        L.rm_mlp_infer(d_p, torch.from_numpy(w[t:t + 9].copy()).cuda(), 9, one)
        np.testing.assert_array_equal(one.cpu().numpy()[0], got[t])
