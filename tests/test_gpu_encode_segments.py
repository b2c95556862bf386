"""The device encoder on tuples around and beyond the 256 entries that it looks up at a
time: (I, D) bit for bit the oracle's, with matches that end at, span and skip whole
segments, empty tuples between, and explicit zeros."""

import numpy as np
import pytest

from test_gpu_encode import assert_batches, encode_gpu
from workloads import Batches

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _batch(rows, cols):
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    col = np.concatenate([np.asarray([c for c, _ in r], np.int32) for r in rows] +
                         [np.zeros(0, np.int32)])
    val = np.concatenate([np.asarray([v for _, v in r], np.float32) for r in rows] +
                         [np.zeros(0, np.float32)])
    return Batches(cols, [len(rows)], rp, col, val)


@pytest.mark.parametrize("length", [255, 256, 257, 511, 512, 513, 700])
def test_tuple_lengths(length):
    rng = np.random.default_rng(length)
    rows = []
    for r in range(14):
        cut = int(rng.integers(0, length + 1))       # shares a prefix with the first tuple
        rows.append([(j, float(1 + (0 if j < cut else (j * 7 + r) % 3))) for j in range(length)])
        if r % 4 == 1:
            rows.append([])
        if r % 5 == 2:
            rows.append([(j, 0.0 if j % 3 else 2.0) for j in range(0, length, 2)])
    B = _batch(rows, length)
    got, _ = encode_gpu(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
    assert_batches(B, got)


def test_matches_longer_than_a_segment():
    """Equal tuples: the matches grow by a pair with every repeat, past 512 entries."""
    row = [(j, float(1 + j % 5)) for j in range(600)]
    B = Batches.concat([_batch([row] * 620, 600), _batch([row[:300]] * 310 + [row], 600)])
    got, _ = encode_gpu(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
    assert_batches(B, got)
