"""Products with k >= 2 on the matrix cores: against the oracle at the edges of their
tiles (16 and 128 columns, 32 columns of A, 64 / 128 / 256 tuples), on batches whose
tree codes need several levels, and with operands that send them term by term.

Bound: |gpu - oracle| <= 1e-5 * S per element, S the sum of the absolute terms: the
parts' dropped products and the sums' roundings stay below it for any of these
sizes (at most 256 terms, each less 2^-31 of itself at most).
"""

import numpy as np
import pytest

import oracle as O
import paper_1702_06943_amd as T
from matrix_path import took_matrix_cores, tree_pairs
from workloads import Batches, tiny_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 1e-5


def _batches(rows_list, cols, seed, **kw):
    parts = []
    for i, n in enumerate(rows_list):
        rp, c, v = tiny_batch(seed + i, n, cols, **kw)
        parts.append(Batches(cols, [n], rp, c, v))
    return Batches.concat(parts)


def _upload(B, flags=0):
    encs = T.toc_encode_batches(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
    buf = torch.empty(T.toc_upload_size(encs, flags), dtype=torch.uint8, device=DEV)
    return T.toc_upload(encs, buf, flags)


def _ws(dev, op, k):
    n, _ = T.toc_workspace_size(dev, op, k)
    return torch.full((max(n, 4) // 4,), float("nan"), device=DEV)


def _rows(B, b):
    n, rp, c, v = B.batch(b)
    return O.canonicalize(n, B.n_cols, rp, c, v)


def _check_right(B, R, W):
    for b in range(B.n_batches):
        r0, r1 = int(B.row_off[b]), int(B.row_off[b + 1])
        ref, S = O.dense_right(_rows(B, b), B.n_cols, W)
        assert np.all(np.abs(R[r0:r1] - ref) <= TOL * S), f"batch {b}"


def _check_left(B, out, G, init=None):
    m = B.n_cols
    for b in range(B.n_batches):
        r0, r1 = int(B.row_off[b]), int(B.row_off[b + 1])
        ref, S = O.dense_left(_rows(B, b), m, G[r0:r1])
        got = out[b * m:(b + 1) * m].astype(np.float64)
        if init is not None:
            ref = ref + init[b * m:(b + 1) * m]
            S = S + np.abs(init[b * m:(b + 1) * m])
        assert np.all(np.abs(got - ref) <= TOL * S), f"batch {b}"


@pytest.mark.parametrize("rows,cols,k,kw", [
    ([1, 64, 40], 5, 2, dict(density=0.9, n_values=3, prefix_copy=0.6)),
    ([64, 63], 33, 16, dict(density=0.9, n_values=3, prefix_copy=0.6)),
    ([65, 128], 32, 17, dict(density=0.8, n_values=4, prefix_copy=0.5)),
    ([129, 7, 200], 70, 130, dict(density=0.9, n_values=6, prefix_copy=0.5)),
    ([256, 0, 255], 97, 300, dict(density=0.7, n_values=5, prefix_copy=0.5)),
    ([250], 64, 128, dict(density=1.0, n_values=2, prefix_copy=0.9)),
    ([250, 31], 40, 20, dict(density=0.9, n_values=3, prefix_copy=0.6, integer=True)),
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_left(rows, cols, k, kw, accumulate):
    B = _batches(rows, cols, 7000 + cols, **kw)
    dev = _upload(B)
    rng = np.random.default_rng(cols * k)
    G = rng.standard_normal((int(B.row_off[-1]), k)).astype(np.float32)
    Gd = torch.zeros((len(G), k + 3), device=DEV)
    Gd[:, :k] = torch.from_numpy(G)
    init = rng.standard_normal((B.n_batches * cols, k)).astype(np.float32)
    out = torch.full((len(init), k + 5), float("nan"), device=DEV)
    out[:, :k] = torch.from_numpy(init)
    ws = _ws(dev, T.TOC_OP_LEFT, k)
    T.toc_left_mul(dev, Gd[:, :k], out[:, :k], accumulate, ws)
    assert took_matrix_cores(ws, tree_pairs(B), cols)
    _check_left(B, out[:, :k].cpu().numpy(), G, init if accumulate else None)
    assert torch.isnan(out[:, k:]).all()          # the padding stays untouched
    # the same bits without a workspace of the caller's
    again = torch.zeros((len(init), k), device=DEV)
    again += torch.from_numpy(init).to(DEV)
    T.toc_left_mul_noalloc(dev, Gd[:, :k], again, accumulate)
    assert torch.equal(again, out[:, :k].contiguous())


@pytest.mark.parametrize("rows,cols,k,kw", [
    ([1, 64, 40], 5, 2, dict(density=0.9, n_values=3, prefix_copy=0.6)),
    ([65, 128, 1], 33, 3, dict(density=0.5, n_values=4, prefix_copy=0.5)),
    ([129, 0, 256], 96, 3, dict(density=0.3, n_values=50, prefix_copy=0.3)),
    ([20, 64] * 55, 40, 150, dict(density=0.6, n_values=400, prefix_copy=0.0)),
    ([128, 30] * 30, 65, 257, dict(density=0.7, n_values=900, prefix_copy=0.0)),
    ([250, 256, 131] * 25, 31, 200, dict(density=0.9, n_values=2000, prefix_copy=0.0)),
    ([250, 17] * 30, 50, 300, dict(density=0.8, n_values=3000, prefix_copy=0.02)),
])
def test_right(rows, cols, k, kw):
    B = _batches(rows, cols, 8000 + cols, **kw)
    dev = _upload(B)
    W = np.random.default_rng(cols * k).standard_normal((cols, k)).astype(np.float32)
    Wd = torch.zeros((cols, k + 2), device=DEV)
    Wd[:, :k] = torch.from_numpy(W)
    R = torch.full((int(B.row_off[-1]), k + 1), float("nan"), device=DEV)
    ws = _ws(dev, T.TOC_OP_RIGHT, k)
    T.toc_right_mul(dev, Wd[:, :k], R[:, :k], ws)
    assert took_matrix_cores(ws, tree_pairs(B), cols)
    _check_right(B, R[:, :k].cpu().numpy(), W)
    assert torch.isnan(R[:, k:]).all()


def test_dead_codes_and_other_workspaces():
    """An image that keeps unused codes; and workspaces that the matrix-core kernels do not
    take (none, too small, not 16-byte aligned), whose calls the general kernels take."""
    B = _batches([64, 63], 33, 8800, density=0.9, n_values=3, prefix_copy=0.6)
    rng = np.random.default_rng(1)
    G = rng.standard_normal((127, 16)).astype(np.float32)
    W = rng.standard_normal((33, 3)).astype(np.float32)
    Gd, Wd = torch.from_numpy(G).to(DEV), torch.from_numpy(W).to(DEV)
    for flags in (0, T.TOC_UPLOAD_KEEP_DEAD):
        dev = _upload(B, flags)
        pairs = tree_pairs(B, flags)
        n, least = T.toc_workspace_size(dev, T.TOC_OP_LEFT, 16)
        need = 2 * 4 * 36 + 2 * 8 * int(pairs.max())     # offsets and pairs of both batches
        assert n >= need and (least == 0 or flags)     # (with all codes, the tables need memory)
        base = torch.full((n + 64,), 255, dtype=torch.uint8, device=DEV)
        others = [(None, False), (base[:need - 16], False), (base[4:4 + n], False)]
        for ws, matrix in [(base[:n], True)] + (others if least == 0 else []):
            base.fill_(255)
            out = torch.full((2 * 33, 16), float("nan"), device=DEV)
            T.toc_left_mul(dev, Gd, out, False, ws)
            assert took_matrix_cores(base if ws is None else ws, pairs, 33) == matrix
            _check_left(B, out.cpu().numpy(), G)
        n, least = T.toc_workspace_size(dev, T.TOC_OP_RIGHT, 3)
        base = torch.full((max(n, least) + 64,), 255, dtype=torch.uint8, device=DEV)
        for size, matrix in ((n, True), (least, least >= need)):
            base.fill_(255)
            R = torch.full((127, 3), float("nan"), device=DEV)
            T.toc_right_mul(dev, Wd, R, base[:size])
            assert took_matrix_cores(base[:size], pairs, 33) == matrix
            _check_right(B, R.cpu().numpy(), W)


@pytest.mark.parametrize("left", [False, True])
def test_passes_of_a_smaller_workspace(left):
    """A workspace for fewer batches than the image has: passes of nearly one size, the same
    bits; and where a pass would not fill the chip, the general kernels."""
    kw = dict(n_values=400, prefix_copy=0.0) if left else dict(n_values=3, prefix_copy=0.6)
    B = _batches([70, 66, 90, 128] * 60 + [100], 40, 8850, density=0.9, **kw)
    dev, k, n = _upload(B), 300 if left else 3, int(B.row_off[-1])
    pairs = tree_pairs(B)
    X = np.random.default_rng(2).standard_normal((n if left else 40, k)).astype(np.float32)
    Xd = torch.from_numpy(X).to(DEV)
    one = 4 * 44 + 8 * int(pairs.max())
    outs = []
    for batches in (241, 100, 64, 63):          # (64 are the least that a pass may have)
        ws = torch.full((batches * one + 15,), 255, dtype=torch.uint8, device=DEV)
        out = torch.full((241 * 40 if left else n, k), float("nan"), device=DEV)
        if left:
            T.toc_left_mul(dev, Xd, out, False, ws)
        else:
            T.toc_right_mul(dev, Xd, out, ws)
        outs.append(out)
        # the last pass's sums: the batches are dealt evenly over the passes
        per = -(-241 // -(-241 // batches))
        last = pairs[(241 - 1) // per * per:]
        assert took_matrix_cores(ws, last, 40) == (batches >= 64)
    for out in (outs[0], outs[3]):
        (_check_left if left else _check_right)(B, out.cpu().numpy(), X)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    if left:
        out = torch.full((241 * 40, k), float("nan"), device=DEV)
        T.toc_left_mul_noalloc(dev, Xd, out, False)
        assert torch.equal(outs[0], out)


@pytest.mark.parametrize("ingested", [False, True])
@pytest.mark.parametrize("rows,whole", [(130, False), (250, True)])
def test_padding_and_parts_decide(rows, whole, ingested):
    """Batches of mostly leaves: 130 tuples of a tile of 256 and values of three parts go to the
    general kernels, which take two thirds of the time; full tiles of one part do not."""
    rp, c, v = tiny_batch(8870, rows, 400, density=0.4, n_values=200 if whole else 40000,
                          integer=whole)
    B = Batches.concat([Batches(400, [rows], rp, c, v)] * 60)
    if ingested:
        encs = T.toc_encode_batches(B.n_rows, B.n_cols, B.rowptr, B.col, B.val)
        blobs = [T.toc_enc_pack(e) for e in encs]
        infos = [T.toc_phys_info_get(b) for b in blobs]
        off = np.concatenate([[0], np.cumsum([len(b) for b in blobs])]).astype(np.int64)
        bytes_ = torch.from_numpy(np.concatenate(blobs)).to(DEV)
        ws = torch.empty(T.toc_ingest_workspace_size(infos, 400)[0], dtype=torch.uint8, device=DEV)
        size, dev = T.toc_ingest_plan(bytes_, off, infos, 400, ws)
        T.toc_ingest_build(dev, bytes_, off, torch.empty(size, dtype=torch.uint8, device=DEV), ws)
    else:
        dev = _upload(B)
    k, rng = 300, np.random.default_rng(8870)
    W = rng.standard_normal((400, k)).astype(np.float32)
    G = rng.standard_normal((60 * rows, k)).astype(np.float32)
    R, out = torch.empty((60 * rows, k), device=DEV), torch.empty((60 * 400, k), device=DEV)
    room = torch.zeros(16 << 20, dtype=torch.uint8, device=DEV)      # (more than the kernels ask)
    for product in (lambda: T.toc_right_mul(dev, torch.from_numpy(W).to(DEV), R, room),
                    lambda: T.toc_left_mul(dev, torch.from_numpy(G).to(DEV), out, False, room)):
        room.fill_(255)
        product()
        assert took_matrix_cores(room, tree_pairs(B), 400) == whole
    B = Batches(400, [rows], rp, c, v)
    _check_right(B, R[-rows:].cpu().numpy(), W)
    _check_left(B, out[-400:].cpu().numpy(), G[-rows:])


@pytest.mark.parametrize("bad", [np.inf, np.nan, 1e-41, 1e-38, 1e-30, 1e-25, 1e12, 1e30, 3e38])
def test_operands_outside_the_split(bad):
    """A non-finite or extreme entry of W or G reaches only what it multiplies."""
    k = 2
    B = _batches([70, 130], 37, 8900, density=0.6, n_values=6, prefix_copy=0.4)
    dev = _upload(B)
    rng = np.random.default_rng(5)
    W = rng.standard_normal((37, k)).astype(np.float32)
    G = rng.standard_normal((200, k)).astype(np.float32)
    W[4, 1] = bad
    G[9, 0] = bad
    G[150] = bad
    R = torch.empty((200, k), device=DEV)
    out = torch.empty((2 * 37, k), device=DEV)
    ws = _ws(dev, T.TOC_OP_RIGHT, k)
    T.toc_right_mul(dev, torch.from_numpy(W).to(DEV), R, ws)
    assert took_matrix_cores(ws, tree_pairs(B), B.n_cols)
    ws = _ws(dev, T.TOC_OP_LEFT, k)
    T.toc_left_mul(dev, torch.from_numpy(G).to(DEV), out, False, ws)
    assert took_matrix_cores(ws, tree_pairs(B), B.n_cols)
    R, out = R.cpu().numpy(), out.cpu().numpy()
    for b in range(2):
        r0, r1 = int(B.row_off[b]), int(B.row_off[b + 1])
        A = np.zeros((r1 - r0, 37))
        n, rp, c, v = B.batch(b)
        for i in range(n):
            A[i, c[rp[i]:rp[i + 1]]] = v[rp[i]:rp[i + 1]]
        for got, X, Y in ((R[r0:r1], A, W), (out[b * 37:(b + 1) * 37], A.T, G[r0:r1])):
            Y = Y.astype(np.float64)
            held = (X != 0).astype(np.float64) @ (~np.isfinite(Y)).astype(np.float64) > 0
            safe = np.where(np.isfinite(Y), Y, 0)
            ref, S = X @ safe, np.abs(X) @ np.abs(safe)
            ok = ~held & (S < 1e38)
            assert np.all(np.abs(got - ref)[ok] <= TOL * S[ok])
            assert not np.isfinite(got[held]).any()


@pytest.mark.parametrize("mapped", [False, True])
@pytest.mark.parametrize("scale", [2.0 ** -40, 2.0 ** 55])
def test_values_outside_the_split(scale, mapped):
    """An image of such values goes to the general kernels; values that toc_map_values has
    moved outside are taken term by term."""
    B = _batches([66, 40], 35, 8950, density=0.9, n_values=5, prefix_copy=0.5)
    if not mapped:
        B.val = (B.val * np.float32(scale)).astype(np.float32)
    dev = _upload(B)
    if mapped:
        T.toc_map_values(dev, T.TOC_MAP_SCALE, scale)
        B.val = (B.val * np.float32(scale)).astype(np.float32)
    rng = np.random.default_rng(6)
    for k in (3, 20):
        W = rng.standard_normal((35, k)).astype(np.float32)
        G = rng.standard_normal((106, k)).astype(np.float32)
        R = torch.empty((106, k), device=DEV)
        out = torch.empty((70, k), device=DEV)
        for op, call, X, Y in ((T.TOC_OP_RIGHT, T.toc_right_mul, W, R),
                               (T.TOC_OP_LEFT, lambda d, x, y, w: T.toc_left_mul(d, x, y, False, w), G, out)):
            ws = _ws(dev, op, k)
            call(dev, torch.from_numpy(X).to(DEV), Y, ws)
            if op == T.TOC_OP_LEFT or k == 3:       # (wider right products of so few codes: the general)
                assert took_matrix_cores(ws, tree_pairs(B), 35) == mapped
        _check_right(B, R.cpu().numpy(), W)
        _check_left(B, out.cpu().numpy(), G)


def test_small_values_are_not_slow():
    """Values of G and W far below the others (saturated gradients, decayed weights) take the
    matrix cores too: within three times the time without them (a tile taken term by term
    takes twenty times)."""
    B = _batches([250] * 64, 100, 8990, density=0.9, n_values=400, prefix_copy=0.0)
    dev, k = _upload(B), 300
    W, G = torch.randn(100, k, device=DEV), torch.randn(64 * 250, k, device=DEV)
    R, out = torch.empty_like(G), torch.empty(64 * 100, k, device=DEV)
    ws = [_ws(dev, op, k) for op in (T.TOC_OP_RIGHT, T.TOC_OP_LEFT)]

    def time(call):
        best = float("inf")
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            call()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    calls = (lambda: T.toc_right_mul(dev, W, R, ws[0]), lambda: T.toc_left_mul(dev, G, out, False, ws[1]))
    usual = [time(c) for c in calls]
    for ws_op in ws:
        assert took_matrix_cores(ws_op, tree_pairs(B), 100)
    for x in (W, G):
        x[torch.rand_like(x) < 0.01] = 1e-25
    for c, t in zip(calls, usual):
        assert time(c) < 3 * t
