"""A first-layer weight that is infinite or no number reaches the tokens whose flanks
choose it, and no others: strings without that letter are encoded, and give gradients,
as if it were zero; a unit whose sum is no number is off.  Encodings within 1e-6 per token, gradients within 1e-3 in 2-norm,
the bounds of the sums in FP32."""
import numpy as np
import pytest

from oracle import learned as OL

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("length", [12, 150])
def test_weight_that_no_token_chooses(value, length):
    torch = torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(91)
    W1, b1, W2, b2 = OL.unpack(OL.init_params(5))
    W2, b2 = rng.normal(0, 0.05, W2.shape), rng.normal(0, 0.4, b2.shape)
    n = 40
    a = rng.integers(0, 3, n * length).astype(np.uint8)  # no letter 3
    b = np.where(rng.random(a.size) < 0.1, (a + 1) % 3, a).astype(np.uint8)
    off = np.arange(n + 1, dtype=np.int64) * length
    got = []
    for v in (0.0, value):
        W1[17, 4 * 2 + 3] = v  # unit 17, flank 2, letter 3
        p = OL.pack(W1, b1, W2, b2).astype(np.float32)
        c = learned.encode(torch.from_numpy(p).cuda(), torch.from_numpy(a).cuda(),
                           torch.from_numpy(off).cuda(), n, 150)
        ps = learned.upload_pairs(a, off, b, off, rng.permutation(n) if not got else got[0][2])
        tr = learned.Trainer(params=p, batch=n)
        loss, grad = tr.gradient(ps)
        got.append((c.cpu().numpy(), grad.cpu().numpy().astype(np.float64), ps.ld.cpu().numpy()))
    (c0, g0, _), (c1, g1, _) = got
    assert np.isfinite(c1).all() and np.isfinite(g1).all()
    assert np.max(np.abs(c1 - c0)) <= 1e-6 * (length - 8)
    assert np.linalg.norm(g1 - g0) <= 1e-3 * np.linalg.norm(g0)


@pytest.mark.parametrize("where", ["weight", "bias"])
def test_unit_that_is_no_number_is_off(where):
    torch = torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(92)
    W1, b1, W2, b2 = OL.unpack(OL.init_params(5))
    W2, b2 = rng.normal(0, 0.05, W2.shape), rng.normal(0, 0.4, b2.shape)
    n, length = 40, 60
    a = rng.integers(0, 3, n * length).astype(np.uint8)
    off = np.arange(n + 1, dtype=np.int64) * length
    got = []
    for v in (-1e6, np.nan):  # off for every token
        if where == "weight":
            W1[17, 8:11] = v  # letters 0..2 of flank 2
        else:
            b1[17] = v
        p = OL.pack(W1, b1, W2, b2).astype(np.float32)
        got.append(learned.encode(torch.from_numpy(p).cuda(), torch.from_numpy(a).cuda(),
                                  torch.from_numpy(off).cuda(), n, 150).cpu().numpy())
    assert np.isfinite(got[1]).all()
    assert np.max(np.abs(got[1] - got[0])) <= 1e-6 * (length - 8)
