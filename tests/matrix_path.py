"""Which kernels took a product with k >= 2: those on the matrix cores leave, at the start
of the workspace, each batch's running sums over the columns of the pairs that its tree
codes stand for."""

import numpy as np

import paper_1702_06943_amd as T


def tree_pairs(B, flags=0):
    """Pairs of each batch that are not a leaf's (from the image's column index)."""
    encs = T.toc_encode_batches(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
    buf = np.zeros(T.toc_upload_size(encs, flags), np.uint8)
    dev = T.toc_upload(encs, buf, flags | T.TOC_UPLOAD_HOST)
    cols = buf[T.toc_dev_layout_get(dev)["cols"]:].view(np.uint32)
    m1 = B.n_cols + 1
    leaf = [int(cols[4 * m1 * b + m1 + B.n_cols]) for b in range(B.n_batches)]
    nnz = [int(T.toc_enc_info_get(e)["nnz"]) for e in encs]
    return np.array(nnz) - np.array(leaf)


def took_matrix_cores(ws, pairs, n_cols):
    """Whether a call of one pass left the running sums in ws (not all zero before it)."""
    stride = (n_cols + 4) // 4 * 4
    words = ws.cpu().numpy().reshape(-1).view(np.uint8)[:4 * stride * len(pairs)]
    if len(words) < 4 * stride * len(pairs):
        return False
    off = words.view(np.uint32).reshape(len(pairs), stride)[:, :n_cols + 1].astype(np.int64)
    return bool(np.all(off[:, 0] == 0) and np.all(np.diff(off, axis=1) >= 0)
                and np.array_equal(off[:, -1], pairs))
