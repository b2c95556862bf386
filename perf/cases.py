"""The calls whose speed matters to a user of this library, as measurable cases.

A case is a matrix family (the five workloads of workloads/gen.py, drawn here on
the GPU so that making them is quick), an operation and its sizes:

  products  toc_right_mul then toc_left_mul: one gradient of a linear model on
            every mini-batch (k = 1)
  right     toc_right_mul (the first layer of a network, forward)
  left      toc_left_mul (the first layer's weight gradient)
  decode    toc_decode_csr
  dense     toc_decode_dense
  mgd       toc_mgd_epoch_split: logistic regression steps
  mlp       toc_mlp_epoch: neural network steps
  encode    toc_encode_device: Algorithm 1 from CSR on the device
  ingest    toc_ingest_plan + toc_ingest_build: physical bytes to the image

Mini-batches have 50 to 250 rows, the range of the paper's section 5; the last
one of a data set may be shorter.
"""

import math

import numpy as np
import torch

import paper_1702_06943_amd as T

DEVICE = "cuda"
HOST_THREADS = 16
ONEHOT_FIELDS, ONEHOT_NUMERIC = 40, 10
TEXT_CANDIDATES, TEXT_MEAN = 256, 75.0
H2, CLASSES = 50, 10          # the network of section 5.1: h1 -> 50 -> 10
LEARNING_RATE = {"image": 1e-6, "text": 0.5, "onehot": 0.1, "census": 0.1}

# canonical compressed bytes (4 |D| + 10 live codes + offsets) and codes of D per
# nonzero, measured on the families' 250-row batches
BYTES_PER_NNZ = {"census": 3.1, "text": 8.9, "image": 10.1, "quant": 9.1, "onehot": 4.9}
CODES_PER_NNZ = {"census": 0.21, "text": 0.85, "image": 0.98, "quant": 0.95, "onehot": 0.61}


def _case(name, family, op, batches, rows=250, last=250, cols=0, k=1, scaled=False):
    return dict(name=name, family=family, op=op, batches=batches, rows=rows, last=last,
                cols=cols, k=k, scaled=scaled)


def listed():
    return [
        # one Census-width mini-batch of logistic regression: launch latency
        _case("census_step", "census", "products", 1, cols=68),
        # a linear model on sparse text (Rcv1 width), ragged last batch
        _case("text_products", "text", "products", 300, last=113, cols=47236),
        # a linear model on one-hot fields (ImageNet width)
        _case("onehot_products", "onehot", "products", 2000, cols=900),
        # a network's first layer on images: forward and weight gradient
        _case("image_right", "image", "right", 400, cols=784, k=300),
        _case("image_left", "image", "left", 400, cols=784, k=300),
        # the same on dense quantised features, ragged last batch
        _case("quant_right", "quant", "right", 100, cols=1000, k=200),
        _case("quant_left", "quant", "left", 100, last=191, cols=1000, k=200),
        # images back to CSR, for an operation that needs the pairs
        _case("image_decode", "image", "decode", 400, cols=784),
        # steps of logistic regression, one after another
        _case("image_mgd", "image", "mgd", 64, cols=784),
        # steps of the paper's network (784-200-50-10) on pixels in [0, 1]
        _case("image_mlp", "image", "mlp", 64, cols=784, k=200, scaled=True),
        # compressing a block of image mini-batches on the GPU
        _case("image_encode", "image", "encode", 256, cols=784),
        # bringing compressed bytes back into a form the products can use
        _case("onehot_ingest", "onehot", "ingest", 1000, cols=900),
    ]


def draw(rng):
    def log(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    family, op = rng.choice([
        ("census", "products"), ("text", "products"), ("onehot", "products"),
        ("image", "products"), ("image", "right"), ("image", "left"), ("quant", "right"),
        ("quant", "left"), ("census", "right"), ("census", "left"), ("image", "decode"),
        ("onehot", "decode"), ("quant", "decode"), ("image", "dense"),
        ("onehot", "dense"), ("image", "mgd"), ("onehot", "mgd"), ("image", "mlp"),
        ("image", "encode"), ("onehot", "encode"), ("census", "encode"),
        ("onehot", "ingest"), ("image", "ingest")])
    most, cols, k = {
        "census": (400, rng.randint(20, 100), 20),
        "text": (250, log(2000, 47236), 20),
        "image": (400, rng.randint(16, 28) ** 2, 300),
        "quant": (100, log(64, 1000), 200),
        "onehot": (2000, rng.randint(300, 1000), 20),
    }[family]
    batches = log(1, most)
    wide = op in ("right", "left")
    if op in ("mgd", "mlp"):
        batches = log(2, 64)
    elif op == "encode":
        batches = log(16, 256)
    elif op == "ingest":
        batches = log(8, 300 if family == "image" else 1000)
    rows = rng.randint(50, 250)
    return dict(family=family, op=op, batches=batches, rows=rows, last=rng.randint(1, rows),
                cols=cols, k=log(2, k) if wide else 4 * rng.randint(8, 50) if op == "mlp" else 1,
                scaled=op == "mlp" or (family == "image" and rng.random() < 0.5))


# --- inputs -------------------------------------------------------------------


def _total_rows(case):
    return (case["batches"] - 1) * case["rows"] + case["last"]


def _zipf(n, s):
    p = np.arange(1, n + 1, dtype=np.float64) ** -s
    c = np.cumsum(p)
    return torch.from_numpy(c / c[-1]).to(DEVICE)


def _ranks(cdf, shape, g):
    u = torch.rand(shape, generator=g, device=DEVICE, dtype=torch.float64)
    return torch.searchsorted(cdf, u, right=True).clamp_(max=len(cdf) - 1)


def _copy_prefixes(A, p, width, g):
    """A[b, r, :width] becomes that of an earlier row of batch b with probability p."""
    nb, rows = A.shape[:2]
    copy = torch.rand((nb, rows), generator=g, device=DEVICE) < p
    u = torch.rand((nb, rows), generator=g, device=DEVICE)
    b = torch.arange(nb, device=DEVICE)
    for r in range(1, rows):
        src = (u[:, r] * r).long().clamp_(max=r - 1)
        A[:, r, :width] = torch.where(copy[:, r, None], A[b, src, :width], A[:, r, :width])


def _dense_to_csr(A):
    mask = A != 0
    rowptr = torch.zeros(A.shape[0] + 1, dtype=torch.int64, device=DEVICE)
    rowptr[1:] = mask.sum(1).cumsum(0)
    return rowptr, mask.nonzero()[:, 1].to(torch.int32), A[mask]


def _census(case, g):
    vocab = torch.rand((case["cols"], 8), generator=g, device=DEVICE) * 2 - 1
    vocab[vocab == 0] = 0.5
    ranks = _ranks(_zipf(8, 1.2), (case["batches"], case["rows"], case["cols"]), g)
    A = vocab[torch.arange(case["cols"], device=DEVICE), ranks]
    _copy_prefixes(A, 0.6, case["cols"] * 40 // 68, g)
    return _dense_to_csr(A.reshape(-1, case["cols"])[:_total_rows(case)])


def _quant(case, g):
    cols = case["cols"]
    levels = torch.randn((cols, 256), generator=g, device=DEVICE).sort(1).values
    levels[levels == 0] = 0.5
    z = torch.randn((cols, case["batches"] * case["rows"]), generator=g, device=DEVICE)
    at = (torch.searchsorted(levels, z, right=True) - 1).clamp_(min=0)
    A = levels.gather(1, at).t().reshape(case["batches"], case["rows"], cols).contiguous()
    _copy_prefixes(A, 0.3, min(200, cols), g)
    return _dense_to_csr(A.reshape(-1, cols)[:_total_rows(case)])


def _image(case, g):
    n, side = _total_rows(case), int(round(math.sqrt(case["cols"])))
    at = torch.arange(side, device=DEVICE, dtype=torch.float32)
    x, y = at.repeat(side), at.repeat_interleave(side)
    centre = torch.randn((2, n, 1), generator=g, device=DEVICE) * (side / 14) + (side - 1) / 2
    width = 2 * (side / 7) ** 2
    f = torch.exp(-((x - centre[0]) ** 2 + (y - centre[1]) ** 2) / width)
    f *= 1 + 0.3 * torch.randn(f.shape, generator=g, device=DEVICE)
    kept, at = f.topk(int(round(0.2 * case["cols"])), dim=1)
    hi, lo = kept[:, :1], kept[:, -1:]
    q = (255 * (kept - lo) / (hi - lo)).round().clamp(1, 255)
    if case["scaled"]:
        q /= 255
    return _dense_to_csr(torch.zeros_like(f).scatter_(1, at, q))


def _text(case, g):
    n, cols = _total_rows(case), case["cols"]
    perm = torch.randperm(cols, generator=g, device=DEVICE)
    c = perm[_ranks(_zipf(cols, 1.1), (n, TEXT_CANDIDATES), g)]
    mean = torch.full((n, 1), TEXT_MEAN, device=DEVICE)
    nnz = torch.poisson(mean, generator=g)
    by_col, order = c.sort(dim=1, stable=True)
    first = torch.ones_like(by_col, dtype=torch.bool)
    first[:, 1:] = by_col[:, 1:] != by_col[:, :-1]
    drawn_first = torch.zeros_like(first).scatter_(1, order, first)
    keep = drawn_first & (drawn_first.cumsum(1) <= nnz)
    c = torch.where(keep, c, cols).sort(1).values
    keep = c < cols
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    rowptr[1:] = keep.sum(1).cumsum(0)
    col = c[keep].to(torch.int32)
    q = torch.randint(1, 17, col.shape, generator=g, device=DEVICE)
    return rowptr, col, q.float() / 16


def _onehot(case, g):
    n, n_cat = _total_rows(case), case["cols"] - ONEHOT_NUMERIC
    u = torch.rand(ONEHOT_FIELDS, generator=g, device=DEVICE, dtype=torch.float64).cpu().numpy()
    raw = np.rint(np.exp(np.log(2.0) + u * np.log(50.0)))
    card = np.maximum(2, np.floor(raw * n_cat / raw.sum())).astype(np.int64)
    card[np.argmax(card)] += n_cat - card.sum()
    col = torch.empty((n, ONEHOT_FIELDS + ONEHOT_NUMERIC), dtype=torch.int32, device=DEVICE)
    off = 0
    for f, c in enumerate(card):
        col[:, f] = off + _ranks(_zipf(int(c), 1.2), (n,), g)
        off += int(c)
    col[:, ONEHOT_FIELDS:] = n_cat + torch.arange(ONEHOT_NUMERIC, device=DEVICE)
    val = torch.ones(col.shape, device=DEVICE)
    q = torch.randint(1, 65, (n, ONEHOT_NUMERIC), generator=g, device=DEVICE)
    val[:, ONEHOT_FIELDS:] = q / 64
    rowptr = torch.arange(n + 1, device=DEVICE) * col.shape[1]
    return rowptr, col.reshape(-1), val.reshape(-1)


_MAKE = {"census": _census, "text": _text, "image": _image, "quant": _quant, "onehot": _onehot}


def _inputs(case, seed):
    """The matrix as CSR on the GPU, and the operands of the operation."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    rowptr, col, val = _MAKE[case["family"]](case, g)
    x = {"rowptr": rowptr, "col": col, "val": val,
         "n_rows": np.array([case["rows"]] * (case["batches"] - 1) + [case["last"]], np.int32)}
    n, m, k, op = len(rowptr) - 1, case["cols"], case["k"], case["op"]

    def normal(shape, sigma):
        return torch.randn(shape, generator=g, device=DEVICE) * sigma

    if op in ("products", "right"):
        x["W"] = normal((m, k), 0.05)
    if op in ("products", "left"):
        x["G"] = normal((n, k), 1.0)
    if op == "mgd":      # labels of a planted model, with noise
        row = torch.repeat_interleave(torch.arange(n, device=DEVICE), rowptr.diff())
        w = normal(m, 1.0).double()
        r = torch.zeros(n, dtype=torch.float64, device=DEVICE)
        r.index_add_(0, row, val.double() * w[col.long()])
        r += 0.1 * r.std() * normal(n, 1.0).double()
        x["y"] = torch.where(r > r.median(), 1.0, -1.0).float()
        x["h"] = normal(m, 0.01)
    if op == "mlp":
        x["labels"] = torch.randint(0, CLASSES, (n,), generator=g, device=DEVICE,
                                    dtype=torch.int32)
        sizes = [m, k, H2, CLASSES]
        x["params"] = {}
        for i in (1, 2, 3):
            x["params"][f"W{i}"] = normal((sizes[i - 1], sizes[i]), sizes[i - 1] ** -0.5)
            x["params"][f"b{i}"] = normal(sizes[i], 0.1)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    op, m, nb = case["op"], case["cols"], case["batches"]
    n, nnz = len(x["rowptr"]) - 1, len(x["col"])

    def empty(shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device=DEVICE)

    s = {"op": op, "x": x, "cols": m}
    if op == "encode":
        first = torch.from_numpy(np.concatenate([[0], np.cumsum(x["n_rows"])])).to(DEVICE)
        starts = x["rowptr"][first]
        sizes = starts.diff()
        s["max_nnz"] = int(sizes.max())
        s["ws"] = empty(T.toc_encode_device_workspace_size(nb, s["max_nnz"]), torch.uint8)
        s["out"] = [empty(nnz, torch.int32), empty(nnz), empty(nnz, torch.int32),
                    empty(n + nb, torch.int64), empty(4 * nb, torch.int64),
                    empty(nb, torch.int32)]
        s["batch_of"] = torch.repeat_interleave(torch.arange(nb, device=DEVICE), sizes)
        s["place"] = torch.arange(nnz, device=DEVICE) - starts[s["batch_of"]]
        return s
    encs = T.toc_encode_batches(x["n_rows"], m, x["rowptr"].cpu().numpy(), x["col"].cpu().numpy(),
                                x["val"].cpu().numpy(), HOST_THREADS)
    if op == "ingest":
        blobs = [T.toc_enc_pack(e) for e in encs]
        s["infos"] = [T.toc_phys_info_get(b) for b in blobs]
        s["blob_off"] = np.concatenate([[0], np.cumsum([len(b) for b in blobs])]).astype(np.int64)
        s["blobs"] = torch.from_numpy(np.concatenate(blobs)).to(DEVICE)
        s["ws"] = empty(T.toc_ingest_workspace_size(s["infos"], m)[0], torch.uint8)
        # the same bytes for every seed: 40 a nonzero and the per-batch arrays are enough
        size = 40 * nnz + 256 * n + 64 * nb * (m + 1) + 4096
        assert size >= T.toc_upload_size(encs)
        s["buf"] = torch.zeros(size, dtype=torch.uint8, device=DEVICE)
        return s
    s["dev"] = T.toc_upload(encs, empty(T.toc_upload_size(encs), torch.uint8))
    if op in ("products", "right"):
        s["R"] = empty((n, case["k"]))
        s["ws_right"] = empty(T.toc_workspace_size(s["dev"], T.TOC_OP_RIGHT, case["k"])[0],
                              torch.uint8)
    if op in ("products", "left"):
        s["out"] = empty((nb * m, case["k"]))
        s["ws_left"] = empty(T.toc_workspace_size(s["dev"], T.TOC_OP_LEFT, case["k"])[0],
                             torch.uint8)
    if op == "decode":
        s["csr"] = [empty(n + 1, torch.int64), empty(nnz, torch.int32), empty(nnz)]
    if op == "dense":
        s["A"] = empty((n, m))
    if op == "mgd":
        s["lr"] = LEARNING_RATE[case["family"]]
        s["h"] = empty(m)
        s["ws"] = empty(T.toc_mgd_workspace_size(s["dev"]), torch.uint8)
    if op == "mlp":
        s["params"] = {name: torch.empty_like(p) for name, p in x["params"].items()}
        s["ws"] = empty(T.toc_mlp_workspace_size(s["dev"], case["k"], H2, CLASSES), torch.uint8)
    return s


# --- one pass -----------------------------------------------------------------


def run(s):
    op, x = s["op"], s["x"]
    out = []
    if op in ("products", "right"):
        T.toc_right_mul(s["dev"], x["W"], s["R"], s["ws_right"])
        out.append(s["R"])
    if op in ("products", "left"):
        T.toc_left_mul(s["dev"], x["G"], s["out"], False, s["ws_left"])
        out.append(s["out"])
    if op == "decode":
        T.toc_decode_csr(s["dev"], *s["csr"])
        out = s["csr"]
    if op == "dense":
        T.toc_decode_dense(s["dev"], s["A"], 1.0)
        out.append(s["A"])
    if op == "mgd":          # from the same model each time
        s["h"].copy_(x["h"])
        T.toc_mgd_epoch_split(s["dev"], x["y"], s["h"], T.TOC_MGD_LOGISTIC, s["lr"], s["ws"])
        out.append(s["h"])
    if op == "mlp":
        names = list(s["params"])
        torch._foreach_copy_([s["params"][p] for p in names], [x["params"][p] for p in names])
        T.toc_mlp_epoch(s["dev"], s["params"], x["labels"], 0.1, s["ws"])
        out = s["params"]
    if op == "encode":
        I_col, I_val, codes, rowptr, counts, status = s["out"]
        T.toc_encode_device(x["n_rows"], s["cols"], x["rowptr"], x["col"], x["val"],
                            s["max_nnz"], *s["out"], s["ws"])
        # a batch's slot holds |I| pairs and |D| codes; what follows them is not defined
        n_first, n_codes = counts[0::4][s["batch_of"]], counts[1::4][s["batch_of"]]
        is_pair, is_code = s["place"] < n_first, s["place"] < n_codes
        out = [I_col * is_pair, torch.where(is_pair, I_val, 0), codes * is_code, rowptr, counts,
               status]
    if op == "ingest":
        size, dev = T.toc_ingest_plan(s["blobs"], s["blob_off"], s["infos"], s["cols"], s["ws"])
        T.toc_ingest_build(dev, s["blobs"], s["blob_off"], s["buf"], s["ws"])
        s["dev"] = dev
        out.append(s["buf"])
    return out


# --- what a pass cannot do without, and what it should give -----------------------


def _nnz(case):
    per_row = {"census": case["cols"], "quant": case["cols"], "image": round(0.2 * case["cols"]),
               "text": min(TEXT_MEAN, 0.04 * case["cols"]),
               "onehot": ONEHOT_FIELDS + ONEHOT_NUMERIC}[case["family"]]
    return per_row * _total_rows(case)


def work(case):
    op, n, m, k, nb = case["op"], _total_rows(case), case["cols"], case["k"], case["batches"]
    nnz = _nnz(case)
    packed = nnz * BYTES_PER_NNZ[case["family"]]
    codes = nnz * CODES_PER_NNZ[case["family"]]
    right = {"bytes": packed + 4 * k * (n + m), "flops": 2 * codes * k}
    left = {"bytes": packed + 4 * k * (n + nb * m), "flops": 2 * codes * k}
    if op == "right":
        return right
    if op == "left":
        return left
    if op == "products":
        return {"bytes": right["bytes"] + left["bytes"], "flops": 4 * codes}
    if op == "decode":
        return {"bytes": packed + 8 * nnz + 8 * n, "flops": 0}
    if op == "dense":
        return {"bytes": packed + 4 * n * m, "flops": n * m}
    if op == "mgd":
        return {"bytes": packed + 4 * n + 8 * m, "flops": 4 * codes}
    if op == "mlp":
        params = m * k + k * H2 + H2 * CLASSES
        return {"bytes": packed + 4 * n + 8 * params,
                "flops": 4 * codes * k + 6 * n * (k * H2 + H2 * CLASSES)}
    if op == "encode":
        return {"bytes": 8 * nnz + 8 * n + packed, "flops": 0}
    return {"bytes": 1.4 * packed, "flops": 0}       # ingest: bytes in, codes and keys out


def tolerance(case):
    """Sums in binary32 (about four times what another order of summation gives);
    a step's error travels through the steps that follow it."""
    op = case["op"]
    if op in ("products", "right", "left"):
        return {"rel": 1e-6, "max": 2e-5}
    if op == "dense":
        return {"rel": 1e-7, "max": 1e-6}
    if op in ("mgd", "mlp"):
        return {"rel": 4e-6, "max": 4e-5}
    return "exact"


def exact(case, seed):
    op, m, k = case["op"], case["cols"], case["k"]
    if op in ("encode", "ingest"):
        return None
    x = _inputs(case, seed)
    rowptr, col, val = x["rowptr"], x["col"].long(), x["val"].double()
    n = len(rowptr) - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE), rowptr.diff())
    first = [min(b * case["rows"], n) for b in range(case["batches"])] + [n]

    def dense(b):
        p, q = (int(rowptr[first[i]]) for i in (b, b + 1))
        A = torch.zeros((first[b + 1] - first[b], m), dtype=torch.float64, device=DEVICE)
        A[row[p:q] - first[b], col[p:q]] = val[p:q]
        return A

    if op == "decode":
        return [rowptr, x["col"], val]
    if op == "dense":
        return [torch.cat([dense(b) for b in range(case["batches"])]) + 1.0]
    if op == "products":
        W, G = x["W"][:, 0].double(), x["G"][:, 0].double()
        R = torch.zeros(n, dtype=torch.float64, device=DEVICE).index_add_(0, row, val * W[col])
        out = torch.zeros(case["batches"] * m, dtype=torch.float64, device=DEVICE)
        out.index_add_(0, row // case["rows"] * m + col, val * G[row])
        return [R[:, None], out[:, None]]
    if op == "right":
        W = x["W"].double()
        return [torch.cat([dense(b) @ W for b in range(case["batches"])])]
    if op == "left":
        G = x["G"].double()
        return [torch.cat([dense(b).t().contiguous() @ G[first[b]:first[b + 1]]
                           for b in range(case["batches"])])]
    if op == "mgd":
        h, y = x["h"].double(), x["y"].double()
        lr = float(np.float32(LEARNING_RATE[case["family"]]))
        for b in range(case["batches"]):
            A, yb = dense(b), y[first[b]:first[b + 1]]
            g = -yb * torch.sigmoid(-yb * (A @ h))
            h = h - lr / len(yb) * (A.t().contiguous() @ g)
        return [h]
    p = {name: t.double() for name, t in x["params"].items()}
    lr = float(np.float32(0.1))
    for b in range(case["batches"]):
        A, c = dense(b), x["labels"][first[b]:first[b + 1]].long()
        H1 = torch.sigmoid(A @ p["W1"] + p["b1"])
        Hh = torch.sigmoid(H1 @ p["W2"] + p["b2"])
        d3 = torch.softmax(Hh @ p["W3"] + p["b3"], 1)
        d3[torch.arange(len(c), device=DEVICE), c] -= 1
        d3 = d3 / len(c)
        d2 = (d3 @ p["W3"].t().contiguous()) * Hh * (1 - Hh)
        d1 = (d2 @ p["W2"].t().contiguous()) * H1 * (1 - H1)
        for i, (left, d) in enumerate(((A, d1), (H1, d2), (Hh, d3)), 1):
            p[f"W{i}"] = p[f"W{i}"] - lr * (left.t().contiguous() @ d)
            p[f"b{i}"] = p[f"b{i}"] - lr * d.sum(0)
    return p
