"""The learned kernels' tiles: 16 tokens of one middle letter, up to eight
strings (four pairs) per block.  Against the FP64 oracle, with the tolerances of
the FP32 kernels: an encoding component sums at most n unit terms (1e-5 n), a
gradient sums token terms with cancellation (2e-3 of the largest component,
1e-3 in 2-norm)."""
import numpy as np
import pytest

from oracle import learned as OL

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _pack(seqs):
    off = np.zeros(len(seqs) + 1, np.int64)
    off[1:] = np.cumsum([len(s) for s in seqs])
    return (np.concatenate(seqs).astype(np.uint8) if off[-1] else np.zeros(1, np.uint8)), off


def _params(seed):
    rng = np.random.default_rng(seed)
    W1, b1, W2, b2 = OL.unpack(OL.init_params(seed))
    return OL.pack(W1, b1, rng.normal(0, 0.05, W2.shape),
                   rng.normal(0, 0.4, b2.shape)).astype(np.float32)


def _strings(kind, n, rng):
    """kind: 'one' letter only (one list full, three empty), 'edge' (a letter's
    tokens at 15, 16, 17 of a tile), 'mixed' lengths, 'unknown' letters."""
    out = []
    for i in range(n):
        if kind == "one":
            w = np.full([9, 24, 25, 256, 300][i % 5], i % 4)
        elif kind == "edge":
            w = np.concatenate([np.full(15 + i % 3 + 4, i % 4), rng.integers(0, 4, 60)])
        else:
            w = rng.integers(0, 4, [0, 8, 9, 150, 257, 40, 180][(i * 3) % 7] + i % 2)
            if kind == "unknown" and w.size:
                w[rng.integers(0, w.size, 1 + w.size // 10)] = [4, 9, 255][i % 3]
        out.append(w.astype(np.uint8))
    return out


@pytest.mark.parametrize("kind,n,nominal", [("one", 1, 150), ("one", 9, 7), ("edge", 8, 150),
                                            ("mixed", 7, 10_000), ("unknown", 17, 150),
                                            ("mixed", 1027, 150)])
def test_encoding_tiles(kind, n, nominal):
    torch = torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(n)
    seqs = _strings(kind, n, rng)
    cat, off = _pack(seqs)
    p = _params(3)
    c = learned.encode(torch.from_numpy(p).cuda(), torch.from_numpy(cat).cuda(),
                       torch.from_numpy(off).cuda(), n, nominal).cpu().numpy().astype(np.float64)
    for i, w in enumerate(seqs):
        want, _ = OL.forward_string(p.astype(np.float64), w[:256], nominal)
        got = c[i, 0::2] + 1j * c[i, 1::2]
        assert np.max(np.abs(got - want)) <= 1e-5 * max(len(w), 1), (kind, i)


@pytest.mark.parametrize("kind,n_pairs", [("one", 2), ("edge", 5), ("mixed", 4), ("unknown", 33),
                                          ("mixed", 513)])
def test_gradient_tiles(kind, n_pairs):
    torch_cuda()
    from paper_2603_22245_amd import learned
    rng = np.random.default_rng(100 + n_pairs)
    a, b = _strings(kind, n_pairs, rng), _strings(kind, n_pairs + 1, rng)[1:]
    ld = rng.permutation(n_pairs).astype(np.int32)
    p = _params(5)
    tr = learned.Trainer(params=p, batch=n_pairs)
    ps = learned.upload_pairs(*_pack(a), *_pack(b), ld)
    loss, grad = tr.gradient(ps)
    loss, grad = float(loss.cpu()[0]), grad.cpu().numpy().astype(np.float64)
    cut = [(x[:256], y[:256]) for x, y in zip(a, b)]
    live = [i for i, (x, y) in enumerate(cut)
            if all(np.any(np.abs(OL.forward_string(p.astype(np.float64), w, 150)[0]) > 0)
                   for w in (x, y))]
    want_loss, want = _oracle(p.astype(np.float64), cut, live, ld)
    assert abs(loss - want_loss) <= 1e-4 * max(1.0, abs(want_loss))
    scale = np.max(np.abs(want))
    assert np.max(np.abs(grad - want)) <= 2e-3 * scale + 1e-12
    assert np.linalg.norm(grad - want) <= 1e-3 * np.linalg.norm(want) + 1e-12


def _oracle(p, pairs, live, ld):
    """Loss and gradient with F = 0 and no gradient for pairs that hold an empty encoding."""
    F = np.zeros(len(pairs))
    fw = {}
    for i in live:
        (ca, ka), (cb, kb) = (OL.forward_string(p, w, 150) for w in pairs[i])
        F[i], Ga, Gb = OL.fidelity_and_grads(ca, cb)
        fw[i] = (ka, kb, Ga, Gb)
    loss, dF = OL.ranking_loss(F, ld)
    grad = np.zeros(OL.N_PARAMS)
    for i, (ka, kb, Ga, Gb) in fw.items():
        grad += OL.backward_string(p, ka, dF[i] * Ga) + OL.backward_string(p, kb, dF[i] * Gb)
    return loss, grad
