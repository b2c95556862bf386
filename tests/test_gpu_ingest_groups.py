"""The image built on the device, byte for byte the host's, where its kernels choose
between LDS and memory: codes held by more than 512 tuples, node counts that fit the
LDS counts, the LDS bits only, or neither, and more columns or levels than the LDS holds."""

import numpy as np
import pytest

import paper_1702_06943_amd as T
from workloads import Batches

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dense(rows, cols, levels, seed, keep=1.0):
    rng = np.random.default_rng(seed)
    A = rng.integers(1, levels + 1, size=(rows, cols)).astype(np.float32)
    A[rng.random(A.shape) >= keep] = 0
    rp = np.concatenate([[0], np.cumsum((A != 0).sum(1))])
    return Batches(cols, [rows], rp, np.nonzero(A)[1].astype(np.int32), A[A != 0])


@pytest.mark.parametrize("parts", [
    [(600, 3, 2, 1.0), (513, 3, 1, 0.5), (512, 3, 1, 1.0), (0, 3, 1, 1.0)],   # large groups
    [(40, 60, 3, 0.7), (1, 60, 9, 1.0)],            # counts in LDS
    [(200, 300, 200, 1.0)],                          # bits only
    [(250, 500, 1000, 1.0), (3, 500, 2, 1.0)],       # neither
    [(320, 320, 1, 1.0)],                            # more than 256 levels
    [(30, 5000, 4, 0.01)],                           # columns beyond the LDS
])
def test_image_equals_host(parts):
    B = Batches.concat([_dense(r, c, n, 77 + i, k) for i, (r, c, n, k) in enumerate(parts)])
    encs = T.toc_encode_batches(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
    size = T.toc_upload_size(encs)
    host = np.zeros(size, np.uint8)
    ref = T.toc_upload(encs, host, T.TOC_UPLOAD_HOST)
    blobs = [T.toc_enc_pack(e) for e in encs]
    infos = [T.toc_phys_info_get(b) for b in blobs]
    off = np.concatenate([[0], np.cumsum([len(b) for b in blobs])])
    data = torch.from_numpy(np.concatenate(blobs)).to(DEV)
    ws = torch.empty(T.toc_ingest_workspace_size(infos, B.n_cols)[0], dtype=torch.uint8, device=DEV)
    n, dev = T.toc_ingest_plan(data, off, infos, B.n_cols, ws)
    assert n == size and T.toc_dev_layout_get(dev) == T.toc_dev_layout_get(ref)
    buf = torch.zeros(size, dtype=torch.uint8, device=DEV)
    T.toc_ingest_build(dev, data, off, buf, ws)
    assert np.array_equal(buf.cpu().numpy(), host)
