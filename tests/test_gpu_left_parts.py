"""The k = 1 products of few batches: a batch's columns dealt to several workgroups
(left), workgroups of 1,024 threads (both), trees of many levels; against the oracle
within 1e-5 * S (sums in blocks of 16, as in the kernels for many batches).  The parts named
beside a case are the left product's."""

import numpy as np
import pytest

import oracle as O
import paper_1702_06943_amd as T
from workloads import Batches, tiny_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nb,rows,cols,kw", [
    (1, 40, 511, dict(density=0.05, n_values=40)),                 # one part
    (1, 40, 512, dict(density=0.05, n_values=40)),                 # two
    (3, 33, 1500, dict(density=0.03, n_values=60)),                # five
    (40, 9, 2304, dict(density=0.02, n_values=60)),                # six
    (300, 4, 1800, dict(density=0.01, n_values=30)),               # one
    (257, 3, 300, dict(density=0.2, n_values=9)),
    (128, 5, 700, dict(density=0.04, n_values=60)),                # two
    (129, 5, 700, dict(density=0.04, n_values=60)),                # one
    (513, 4, 300, dict(density=0.2, n_values=900)),                # 256 threads
    (513, (40, 2), 300, dict(density=0.9, n_values=9000)),         # 1,024: LDS (first batch, others)
    (513, 4, 1025, dict(density=0.03, n_values=900)),              # 1,024: columns
    (2, 120, 60, dict(density=1.0, n_values=2, prefix_copy=0.95)),  # deep trees
    (300, 12, 40, dict(density=1.0, n_values=1, prefix_copy=0.5)),
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_k1(nb, rows, cols, kw, accumulate):
    parts = []
    for b in range(nb):
        n = 0 if b % 7 == 5 else rows if isinstance(rows, int) else rows[b > 0]
        rp, c, v = tiny_batch(5000 + cols + b, n, cols, **kw)
        parts.append(Batches(cols, [n], rp, c, v))
    B = Batches.concat(parts)
    encs = T.toc_encode_batches(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
    dev = T.toc_upload(encs, torch.empty(T.toc_upload_size(encs), dtype=torch.uint8, device=DEV))
    rng = np.random.default_rng(cols + nb)
    n = int(B.row_off[-1])
    W = rng.standard_normal((cols, 1)).astype(np.float32)
    G = rng.standard_normal((n, 1)).astype(np.float32)
    init = rng.standard_normal((nb * cols, 1)).astype(np.float32)
    R = torch.full((n, 1), float("nan"), device=DEV)
    out = torch.from_numpy(init).to(DEV) if accumulate else \
        torch.full((nb * cols, 1), float("nan"), device=DEV)
    T.toc_right_mul(dev, torch.from_numpy(W).to(DEV), R)
    T.toc_left_mul(dev, torch.from_numpy(G).to(DEV), out, accumulate)
    R, out = R.cpu().numpy(), out.cpu().numpy()
    for b in range(nb):
        rn, rp, c, v = B.batch(b)
        tuples = O.canonicalize(rn, cols, rp, c, v)
        r0 = int(B.row_off[b])
        ref, S = O.dense_right(tuples, cols, W)
        assert np.all(np.abs(R[r0:r0 + rn] - ref) <= 1e-5 * S)
        ref, S = O.dense_left(tuples, cols, G[r0:r0 + rn])
        if accumulate:
            ref, S = ref + init[b * cols:(b + 1) * cols], S + np.abs(init[b * cols:(b + 1) * cols])
        assert np.all(np.abs(out[b * cols:(b + 1) * cols] - ref) <= 1e-5 * S)


def test_left_time_does_not_jump():
    """256 image-like batches of few tree codes take little longer than 64, which leave
    three quarters of the CUs idle, or have their columns dealt to several workgroups each."""
    times = []
    for nb in (64, 256):
        rp, c, v = tiny_batch(5600, 250, 784, density=0.2, n_values=40000)
        B = Batches.concat([Batches(784, [250], rp, c, v)] * nb)
        encs = T.toc_encode_batches(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
        dev = T.toc_upload(encs, torch.empty(T.toc_upload_size(encs), dtype=torch.uint8, device=DEV))
        G = torch.randn((250 * nb, 1), device=DEV)
        out = torch.empty((784 * nb, 1), device=DEV)
        best = float("inf")
        for _ in range(10):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            T.toc_left_mul(dev, G, out)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    print(f"64 and 256 batches: {times[0] * 1e3:.0f} and {times[1] * 1e3:.0f} us")
    assert times[1] < 2.5 * times[0]
