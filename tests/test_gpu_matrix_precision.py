"""The matrix-core products keep binary32's precision: sums of one and two terms against
64 bits.  A term leaves out at most 2^-31 of itself and is rounded once at its own size
(2^-24), its smaller parts' sums at 2^-7 of it, cut off by the matrix cores (below
2^-29): 2^-24 (1 + 2^-5) of the absolute terms with one term.  With two, the matrix cores
add the leading products and cut the sum off at 24 bits (2^-23) before that rounding."""

import numpy as np
import pytest

import paper_1702_06943_amd as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ULP = 2.0 ** -24


def _floats(rng, shape):
    """24-bit significands, exponents over 20 binades, both signs."""
    x = (1 + rng.random(shape)) * 2.0 ** rng.integers(-10, 10, shape)
    return (x * rng.choice([-1, 1], shape)).astype(np.float32)


@pytest.mark.parametrize("whole", [False, True])
@pytest.mark.parametrize("terms", [1, 2])
def test_short_sums(terms, whole):
    """150 batches of 16 tuples over 16 columns, `terms` entries to a tuple and a column,
    of 24 bits or of whole numbers below 256 (one part)."""
    nb, n, k = 150, 16, 128
    rng = np.random.default_rng(terms)
    A = np.zeros((nb, n, n), np.float32)
    for t in range(terms):
        i = np.arange(n)
        A[:, i, (i * 3 + 5 * t) % n] = rng.integers(1, 256, (nb, n)) if whole else _floats(rng, (nb, n))
    rp = np.arange(nb * n + 1, dtype=np.int64) * terms
    col, val = np.nonzero(A.reshape(-1, n))[1].astype(np.int32), A[A != 0]
    encs = T.toc_encode_batches(np.full(nb, n, np.int32), n, rp, col, val)
    dev = T.toc_upload(encs, torch.empty(T.toc_upload_size(encs), dtype=torch.uint8, device=DEV))
    W, G = _floats(rng, (n, k)), _floats(rng, (nb * n, k))
    R = torch.empty((nb * n, k), device=DEV)
    out = torch.empty((nb * n, k), device=DEV)

    def ws(op, k):
        return torch.empty(T.toc_workspace_size(dev, op, k)[0], dtype=torch.uint8, device=DEV)

    T.toc_left_mul(dev, torch.from_numpy(G).to(DEV), out, False, ws(T.TOC_OP_LEFT, k))
    A = A.astype(np.float64)
    bound = ULP * (2 * terms - 1 + 2.0 ** -5)
    checks = [("left", out, np.swapaxes(A, 1, 2), G.reshape(nb, n, k))]
    R3 = torch.empty((nb * n, 3), device=DEV)      # (these and the wide ones: other kernels)
    for R, w in ((R, W), (R3, np.ascontiguousarray(W[:, :3]))):
        T.toc_right_mul(dev, torch.from_numpy(w).to(DEV), R, ws(T.TOC_OP_RIGHT, w.shape[1]))
        checks.append((f"right, {w.shape[1]} columns", R, A, w))
    for name, got, X, Y in checks:
        Y = Y.astype(np.float64)
        got = got.cpu().numpy().astype(np.float64).reshape(nb, n, -1)
        e = np.abs(got - X @ Y) / (np.abs(X) @ np.abs(Y))
        print(f"{name}, {terms} terms: largest {e.max():.3e}, RMS {np.sqrt((e ** 2).mean()):.3e}")
        assert e.max() <= bound, name
