"""Physical bytes whose tuples hold a column more than once, or out of order (or values
that the matrix-core products do not take).  The
encoders refuse such tuples, but bytes made elsewhere can describe them: every code
occurs once in a tuple, as the ingest asks, and the bytes are otherwise whole.  The
products sum all pairs of a tuple (at most 100 terms a sum, each rounded to binary32:
within 1e-5 of the absolute terms), and the matrix-core products, whose tiles have one
cell for a tuple and a column, leave such an image to the others."""

import numpy as np
import pytest

import oracle as O
import paper_1702_06943_amd as T

torch = pytest.importorskip("torch")
DEV = "cuda:0"


def _repeated():
    """Three tuples over one column whose five pairs meet in codes of D."""
    one, two, three = (((0, O.f32_bits(float(v)))) for v in (1, 2, 3))
    return [one, two, three], [[1, 2, 3], [4, 3], [6]], 1


def _encoded(rows, cols):
    I, D, _ = O.encode(rows)
    return I, D, cols


def _columns_of_many_pairs():
    """40 tuples of 24 pairs over 4 columns, the same prefixes again and again: more
    pairs from a column's tree codes than tuples, and columns of more leaves than
    tuples before them."""
    rng = np.random.default_rng(5)
    rows = []
    for i in range(40):
        t = [(j % 4, O.f32_bits(float(1 + j))) for j in range(8)]
        t += [(int(rng.integers(0, 2)), O.f32_bits(float(100 + 30 * i + j))) for j in range(16)]
        rows.append(t)
    return _encoded(rows, 4)


def _out_of_order():
    """Each column once, the columns descending in every other tuple."""
    rng = np.random.default_rng(6)
    rows = []
    for i in range(30):
        v = [(j, O.f32_bits(float(rng.integers(1, 4)))) for j in range(9)]
        rows.append(v[::-1] if i % 2 else v)
    return _encoded(rows, 9)


def _values_out_of_range():
    """Whole tuples with a value of 2^-50."""
    rng = np.random.default_rng(7)
    rows = [[(j, O.f32_bits(float(rng.integers(1, 4)) * (2.0 ** -50 if i == j else 1))) for j in range(12)]
            for i in range(30)]
    return _encoded(rows, 12)


def _dense(I, D, cols):
    """Sums of each tuple's values by column, and of their absolute values."""
    rows = O.decode(I, D)
    A, S = np.zeros((2, len(rows), cols))
    for i, t in enumerate(rows):
        for c, b in t:
            A[i, c] += O.bits_f32(b)
            S[i, c] += abs(O.bits_f32(b))
    return A, S


def test_the_bytes_are_accepted():
    for make in (_repeated, _columns_of_many_pairs, _out_of_order, _values_out_of_range):
        I, D, cols = make()
        assert all(len(set(codes)) == len(codes) for codes in D)
        info = T.toc_phys_info_get(np.frombuffer(O.pack_physical(I, D), np.uint8))
        assert info["n_rows"] == len(D) and info["max_col"] == cols - 1


@pytest.mark.gpu
@pytest.mark.parametrize("make", [_repeated, _columns_of_many_pairs, _out_of_order, _values_out_of_range])
@pytest.mark.parametrize("k", [1, 2, 20])
def test_products(make, k):
    I, D, cols = make()
    blob = np.frombuffer(O.pack_physical(I, D), np.uint8).copy()
    infos = [T.toc_phys_info_get(blob)]
    off = np.array([0, len(blob)], np.int64)
    data = torch.from_numpy(blob).to(DEV)
    ws = torch.empty(T.toc_ingest_workspace_size(infos, cols)[0], dtype=torch.uint8, device=DEV)
    size, dev = T.toc_ingest_plan(data, off, infos, cols, ws)
    buf = torch.zeros(size, dtype=torch.uint8, device=DEV)
    T.toc_ingest_build(dev, data, off, buf, ws)
    # what the general kernels ask for these sizes, and no more
    for op in (T.TOC_OP_RIGHT, T.TOC_OP_LEFT):
        n, least = T.toc_workspace_size(dev, op, k)
        assert n == least
    A, S = _dense(I, D, cols)
    rng = np.random.default_rng(k)
    W = rng.standard_normal((cols, k)).astype(np.float32)
    G = rng.standard_normal((len(D), k)).astype(np.float32)
    R = torch.full((len(D), k), float("nan"), device=DEV)
    out = torch.full((cols, k), float("nan"), device=DEV)
    # (a workspace that would hold the matrix-core products' too)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    T.toc_right_mul(dev, torch.from_numpy(W).to(DEV), R, ws)
    T.toc_left_mul(dev, torch.from_numpy(G).to(DEV), out, False, ws)
    assert np.all(np.abs(R.cpu().numpy() - A @ W) <= 1e-5 * (S @ np.abs(W)))
    assert np.all(np.abs(out.cpu().numpy() - A.T @ G) <= 1e-5 * (S.T @ np.abs(G)))
    again = torch.full((cols, k), float("nan"), device=DEV)
    T.toc_left_mul_noalloc(dev, torch.from_numpy(G).to(DEV), again, False)
    assert torch.equal(again, out)
