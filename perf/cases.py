"""Workloads of the double-quantization library, for measuring it.

A case is a dict of plain values.  ``prepare(case, seed)`` makes on the GPU what a program holds before the call,
``run(state)`` is one pass through the public entry points, ``exact(case, seed)`` the same numbers in 64 bits from
plain torch where they have such a value.  Five kinds of work, all of them what a run of the method consists of:

``epoch``      one epoch of Alg. 1, 2 or 3 from a given snapshot through ``DoubleQuantTrainer``: the full gradient and
               m rounds.  This is what the library is for.
``objective``  ``dq_full_grad``: the gradient, the margins and P(x) at a point (epoch prologue; evaluation of a model)
``worker``     one ``dq_worker_step`` with the caller's own mini-batches, as a program with its own round loop calls it
``quantize``   ``dq_quantize_pack`` of whole vectors, the scale included
``aggregate``  ``dq_unpack_dequant_sum``: the master's receive side
``message``    the sparse message on its own: sparsify, quantize, encode, decode
"""
from __future__ import annotations

import math

import torch

import paper_1805_10111_amd as dq
from paper_1805_10111_amd.driver import DoubleQuantTrainer

DEV = "cuda"


def listed():
    return [
        # The small dense problem (2000 x 1000, four workers, 16 rows each): nothing but launches and latency.
        dict(name="epoch_dense_small", kind="epoch", feat="dense", n=2000, d=1000, algo="asylpg", M=4, B=16, b_x=8, b=8,
             m=32, each=False, tau=0, wire=False, cached=True),
        # A dense problem of 784 columns (28 x 28 images) with a model message of 6 bits, one of the widths that the
        # study of the model precision goes through.
        dict(name="epoch_dense_medium", kind="epoch", feat="dense", n=60000, d=784, algo="asylpg", M=10, B=100, b_x=6, b=8,
             m=60, each=False, tau=0, wire=False, cached=True),
        # The large dense problem (200000 x 4096, 3.3 GB) with momentum: 134 MB of feature rows per round.
        dict(name="epoch_dense_large", kind="epoch", feat="dense", n=200000, d=4096, algo="acc", M=32, B=256, b_x=8, b=8,
             m=25, each=False, tau=0, wire=False, cached=True),
        # Bag-of-words features in the shape of real-sim: Alg. 1 ...
        dict(name="epoch_text", kind="epoch", feat="csr", n=72000, d=20958, nnz=52, algo="asylpg", M=8, B=32, b_x=8, b=8,
             m=282, each=False, tau=0, wire=False, cached=True),
        # ... and Alg. 2 (sparsified gradients of 4 bits).
        dict(name="epoch_text_sparse", kind="epoch", feat="csr", n=72000, d=20958, nnz=52, algo="sparse", M=16, B=64, b_x=8,
             b=4, m=71, each=False, tau=0, wire=False, cached=True),
        # rcv1's width (47236 columns), the gradients really crossing as (position, value) messages.
        dict(name="epoch_text_wide_wire", kind="epoch", feat="csr", n=20242, d=47236, nnz=75, algo="sparse", M=8, B=32, b_x=8,
             b=4, m=79, each=False, tau=0, wire=True, cached=True),
        # Objective and gradient of a model on dense rows of a width that is no power of two.
        dict(name="objective_dense", kind="objective", feat="dense", n=50000, d=3000),
        # The same on the real-sim shape.
        dict(name="objective_text", kind="objective", feat="csr", n=72000, d=20958, nnz=52),
        # A program's own round loop: its own mini-batches of a size that divides nothing, no cached margins, the
        # gradient wanted beside the message.
        dict(name="worker_dense_ragged", kind="worker", feat="dense", n=40000, d=2500, M=12, B=90, b_x=8, b=4, sparsify=True,
             own=True, cached=False, alpha=True),
        # The quantizer on a long gradient vector (2^28 coordinates, 1 GiB).
        dict(name="quantize_long", kind="quantize", d=1 << 28, M=1, b=8),
        # The master's receive side over 16 workers' 4-bit messages of 2^27 coordinates.
        dict(name="aggregate_long", kind="aggregate", d=1 << 27, M=16, b=4),
        # One round's sparse messages on their own.
        dict(name="message_sparse", kind="message", d=20958, M=16, b=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["epoch", "epoch", "epoch", "objective", "worker", "quantize", "aggregate", "message"])
    if kind == "quantize":
        b, M = rng.choice([2, 3, 4, 6, 8, 8, 11]), rng.choice([1, 1, 4, 16])
        return dict(kind=kind, d=_log(rng, 1000, (1 << 27) // M), M=M, b=b)
    if kind == "aggregate":
        b, M = rng.choice([2, 4, 8, 8, 5]), rng.choice([1, 3, 8, 16, 32])
        return dict(kind=kind, d=_log(rng, 1000, (1 << 29) // (M * b)), M=M, b=b)
    if kind == "message":
        return dict(kind=kind, d=_log(rng, 500, 48000), M=rng.randint(2, 32), b=rng.choice([2, 4, 4]))
    dense = rng.random() < 0.5
    M, B = rng.randint(2, 32), _log(rng, 8, 256)
    if dense:
        d = _log(rng, 50, 8192)
        c = dict(kind=kind, feat="dense", n=_log(rng, 1000, min(200000, 400000000 // d)), d=d)
    else:
        d = _log(rng, 1000, 60000)
        c = dict(kind=kind, feat="csr", n=_log(rng, 2000, 80000), d=d, nnz=_log(rng, 8, 100))
        B = min(B, 128)
    if kind == "objective":
        return c
    if kind == "worker":
        c.update(M=M, B=B, b_x=rng.choice([2, 4, 8, 8, 8, 11]), b=rng.choice([2, 4, 8, 8]), sparsify=rng.random() < 0.4,
                 own=rng.random() < 0.5, cached=rng.random() < 0.7, alpha=True)
        return c
    algo = rng.choice(["asylpg", "sparse", "acc"])
    wide = rng.random() < 0.2                              # not quantized at all: the full-precision comparison runs
    c.update(algo=algo, M=M, B=B, b_x=32 if wide else rng.choice([4, 8, 8, 8, 6]), b=32 if wide else rng.choice([4, 8, 8]),
             m=rng.randint(8, 60), each=rng.random() < 0.2, tau=rng.choice([0, 0, 0, 1]), wire=False, cached=rng.random() < 0.8)
    c["m"] = min(c["m"], max(8, int(8e8 / (c["M"] * c["B"] * (c["d"] if dense else 500)))))
    c["wire"] = algo == "sparse" and c["b"] == 4 and c["d"] <= 48000 and rng.random() < 0.5
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _pad4(d):
    return (d + 3) // 4 * 4


def _labels(margins, g):
    y = torch.where(margins >= 0, 1.0, -1.0).float()
    return torch.where(torch.rand(y.shape[0], device=DEV, generator=g) < 0.05, -y, y)


def _dense(case, g):
    """Rows N(0,1)/sqrt(d), labels from a planted vector, five in a hundred of them flipped."""
    n, d = case["n"], case["d"]
    X = torch.empty((n, _pad4(d)), device=DEV)
    w = torch.randn(d, device=DEV, generator=g)
    margins = torch.empty(n, device=DEV)
    for r in range(0, n, 32768):
        rows = torch.randn((min(32768, n - r), d), device=DEV, generator=g) / math.sqrt(d)
        X[r:r + rows.shape[0], :d] = rows
        if d < X.shape[1]:
            X[r:r + rows.shape[0], d:] = 0.0
        margins[r:r + rows.shape[0]] = (rows * w).sum(1)
    x0 = 0.5 * w + 0.1 * torch.randn(d, device=DEV, generator=g)
    return dict(n=n, d=d, y=_labels(margins, g), dense=X[:, :d]), x0


def _csr(case, g):
    """Bag-of-words rows: lognormal/Poisson lengths, columns ~ 1/(j+1) without repeats, tf-idf values of unit norm."""
    n, d, mean = case["n"], case["d"], float(case["nnz"])
    rand = lambda k: torch.rand(k, device=DEV, generator=g, dtype=torch.float64)          # noqa: E731
    sigma = 0.6
    logn = torch.exp(torch.randn(n, device=DEV, generator=g, dtype=torch.float64) * sigma + math.log(mean) - 0.5 * sigma * sigma)
    pois = torch.poisson(torch.full((n,), mean, device=DEV, dtype=torch.float64), generator=g)
    lens = torch.where(rand(n) < 0.5, logn.round(), pois).long().clamp(1, min(d, 8 * int(mean) + 8))
    cdf = torch.cumsum(1.0 / torch.arange(1, d + 1, dtype=torch.float64), 0)              # (on the host: the same every time)
    cdf = (cdf / cdf[-1]).to(DEV)
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), 2 * lens + 8)
    cols = torch.searchsorted(cdf, rand(rows.numel()), right=True).clamp_(max=d - 1)
    key = torch.unique(rows * d + cols)                                                   # sorted: by row, then column
    rows = key // d
    order = torch.argsort(rows.double() + 0.999 * rand(key.numel()))                      # by row, then by lot
    first = torch.searchsorted(rows, torch.arange(n, device=DEV))
    rank = torch.arange(key.numel(), device=DEV) - first[rows]                            # (rows of `order` are `rows` again)
    key = key[order[rank < lens[rows]].sort().values]
    rows, cols = key // d, key % d
    counts = torch.bincount(rows, minlength=n)
    indptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    indptr[1:] = torch.cumsum(counts, 0)
    idf = torch.log1p(n / torch.bincount(cols, minlength=d).double().clamp(min=1.0))
    tf = (torch.log(rand(key.numel()).clamp(min=1e-12)) / math.log(0.4)).ceil().clamp(min=1.0)      # geometric, p = 0.6
    vals = (1.0 + torch.log(tf)) * idf[cols]
    norm = torch.segment_reduce(vals * vals, "sum", lengths=counts).sqrt()
    vals = (vals / norm[rows]).float()
    support = (rand(d) < 0.05).double()
    support[:64] = 1.0
    w = torch.randn(d, device=DEV, generator=g, dtype=torch.float64) * support
    margins = torch.segment_reduce(vals.double() * w[cols], "sum", lengths=counts)
    margins = margins - margins.sort().values[n // 2]
    x0 = (0.5 * w + 0.02 * torch.randn(d, device=DEV, generator=g, dtype=torch.float64)).float()
    return dict(n=n, d=d, y=_labels(margins, g), indptr=indptr, indices=cols.int(), values=vals), x0


L2, L1 = 1e-4, 1e-5


def _problem(case, g):
    p, x0 = _dense(case, g) if case["feat"] == "dense" else _csr(case, g)
    return p, x0


def _codes(case, x0, g):
    """The b_x-bit message of a model near the snapshot x0, and its scale: (codes, words, scale)."""
    b, d = case["b_x"], x0.numel()
    x = x0 + 0.05 * torch.randn(d, device=DEV, generator=g)
    top = (1 << (b - 1)) - 1
    scale = (x.abs().max() / top).reshape(1)
    codes = (x / scale).round().clamp(-top, top).int()
    bits = ((codes[:, None] >> torch.arange(b, device=DEV)) & 1).reshape(-1).to(torch.int64)
    words = torch.zeros((_pad4((d * b + 31) // 32), 32), dtype=torch.int64, device=DEV)
    words.view(-1)[:bits.numel()] = bits
    words = (words << torch.arange(32, device=DEV)).sum(1)
    words = torch.where(words >= 1 << 31, words - (1 << 32), words).int()
    return codes, words, scale


def _vector(d, g):
    """Gradient-like coordinates: one in ten N(0, 1), the others N(0, 1e-4)."""
    v = torch.randn(d, device=DEV, generator=g)
    return v.mul_(torch.where(torch.rand(d, device=DEV, generator=g) < 0.1, 1.0, 0.01))


def _matrix(M, d, g):
    v = torch.zeros((M, _pad4(d)), device=DEV)
    for m in range(M):
        v[m, :d] = _vector(d, g)
    return v[:, :d]


def _row_words(d, b):
    return _pad4(d if b == 32 else dq.packed_words(d, b))


def _ints(*shape):
    return torch.zeros(shape, dtype=torch.int32, device=DEV)


def _sums(case, g):
    M, words = case["M"], _row_words(case["d"], case["b"])
    packed = torch.randint(-(1 << 31), 1 << 31, (M, words), dtype=torch.int32, device=DEV, generator=g)
    return packed, 0.01 + 0.05 * torch.rand(M, device=DEV, generator=g)


def _own_batches(case, g):
    return torch.randint(0, case["n"], (case["M"], case["B"]), dtype=torch.int32, device=DEV, generator=g)


def _worker_inputs(case, seed):
    g = _gen(seed)
    p, x0 = _problem(case, g)
    codes, words, scale = _codes(case, x0, g)
    return p, x0, codes, words, scale, _own_batches(case, g)


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    s = dict(kind=kind, case=case, seed=seed)
    if kind == "epoch":
        p, x0 = _problem(case, g)
        tr = DoubleQuantTrainer(dq.DeviceProblem(l2=L2, l1=L1 if case["feat"] == "csr" else 0.0, **p), case["algo"], case["M"],
                                case["B"], case["b_x"], case["b"], case["m"], 0.1, seed=seed, x0=x0, tau=case["tau"],
                                each=case["each"], sparse_wire=case["wire"], cache_margins=case["cached"])
        if case["algo"] == "acc":
            tr.epoch_index = 1                             # (the second epoch: its first model is not the snapshot)
            s["y0"] = x0 + 0.02 * torch.randn(x0.numel(), device=DEV, generator=g)
        s["trainer"] = tr
    elif kind == "objective":
        p, x0 = _problem(case, g)
        prob = dq.DeviceProblem(l2=L2, l1=L1, **p)
        s.update(prob=prob, x=x0, g=torch.zeros(prob.d, device=DEV), z=torch.zeros(prob.n, device=DEV),
                 obj=torch.zeros(1, dtype=torch.float64, device=DEV), ws=dq.new_workspace(dq.OP_FULL_GRAD, prob))
    elif kind == "worker":
        p, x0, _, words, scale, idx = _worker_inputs(case, seed)
        prob = dq.DeviceProblem(l2=L2, l1=L1, **p)
        M, d = case["M"], case["d"]
        z = None
        if case["cached"]:
            z = torch.zeros(prob.n, device=DEV)
            dq.dq_full_grad(prob, x0, torch.zeros(d, device=DEV), z, None, dq.new_workspace(dq.OP_FULL_GRAD, prob))
        s.update(prob=prob, idx=idx if case["own"] else None, words=words, scale=scale, x0=x0, z=z,
                 packed=_ints(M, _row_words(d, case["b"])), delta=torch.zeros(M, device=DEV),
                 alpha=torch.zeros((M, _pad4(d)), device=DEV) if case["alpha"] else None, status=_ints(1),
                 ws=dq.new_workspace(dq.OP_WORKER_STEP, prob, M, case["B"]))
    elif kind == "quantize":
        M, d = case["M"], case["d"]
        s.update(v=_matrix(M, d, g), absmax=torch.zeros(M, device=DEV), delta=torch.zeros(M, device=DEV),
                 packed=_ints(M, _row_words(d, case["b"])))
    elif kind == "aggregate":
        packed, delta = _sums(case, g)
        s.update(packed=packed, delta=delta, out=torch.zeros(case["d"], device=DEV))
    else:
        M, d, b = case["M"], case["d"], case["b"]
        s.update(alpha=_matrix(M, d, g), beta=torch.zeros((M, _pad4(d)), device=DEV)[:, :d], absmax=torch.zeros(M, device=DEV),
                 kept=_ints(M), packed=_ints(M, _row_words(d, b)), delta=torch.zeros(M, device=DEV),
                 stream=_ints(M, _pad4(dq.dq_sparse_stream_words(d, b))), nnz=_ints(M), back=_ints(M, _row_words(d, b)))
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = s["kind"]
    if kind == "epoch":
        tr = s["trainer"]
        if "y0" in s:
            tr.y.copy_(s["y0"])                            # every pass is the same epoch
        tr.epoch_prologue()
        tr.rounds(0, tr.m)
        out = dict(x=tr.x, g=tr.g_snap, objective=tr.obj, model=tr.xq, model_scale=tr.delta_x, messages=tr.packed, scales=tr.delta)
        if tr.z_snap is not None:
            out["z"] = tr.z_snap
        if tr.algo == "acc":
            out.update(y=tr.y, xsum=tr.xsum)
        if tr.algo == "sparse":
            out["nonzeros"] = tr.nnz
        if tr.b == 32:
            out["messages"] = tr.packed.view(torch.float32)
        if tr.b_x == 32:
            out["model"] = tr.xq.view(torch.float32)
        return out
    if kind == "objective":
        dq.dq_full_grad(s["prob"], s["x"], s["g"], s["z"], s["obj"], s["ws"])
        return dict(g=s["g"], z=s["z"], objective=s["obj"])
    if kind == "worker":
        dq.dq_worker_step(s["prob"], s["idx"], case["M"], case["B"], s["words"], s["scale"], case["b_x"], 0, s["x0"], s["z"],
                          case["sparsify"], case["b"], s["seed"], 3, 0, s["packed"], s["delta"], None, s["alpha"], s["status"],
                          s["ws"])
        return dict(messages=s["packed"], scales=s["delta"], alpha=s["alpha"])
    if kind == "quantize":
        dq.dq_quantize_pack(s["v"], case["b"], s["absmax"], False, s["seed"], 5, dq.TAG_GRAD, 0, s["packed"], s["delta"])
        return dict(messages=s["packed"], scales=s["delta"], absmax=s["absmax"])
    if kind == "aggregate":
        dq.dq_unpack_dequant_sum(s["packed"], s["delta"], case["d"], case["b"], 1.0 / case["M"], s["out"])
        return s["out"]
    dq.dq_sparsify(s["alpha"], None, s["seed"], 7, 0, s["beta"], s["absmax"], s["kept"])
    dq.dq_quantize_pack(s["beta"], case["b"], s["absmax"], True, s["seed"], 7, dq.TAG_GRAD, 0, s["packed"], s["delta"])
    dq.dq_sparse_encode(s["packed"], case["d"], case["b"], s["stream"], s["nnz"])
    dq.dq_sparse_decode(s["stream"], s["nnz"], case["d"], case["b"], s["back"])
    return dict(beta=s["beta"], kept=s["kept"], messages=s["packed"], scales=s["delta"], stream=s["stream"], nnz=s["nnz"],
                received=s["back"])


# ------------------------------------------------------------------------------------------------ what a pass needs
def _entries(case):
    return case["n"] * case["d"] if case["feat"] == "dense" else case["n"] * case["nnz"]


def _full_work(case):
    e, n, d = _entries(case), case["n"], case["d"]
    rows = 4 * e if case["feat"] == "dense" else 8 * e + 8 * n
    return rows + 4 * n + 4 * n + 8 * d, 4 * e


def _worker_work(case):
    M, B, d = case["M"], case["B"], case["d"]
    e = M * B * (d if case["feat"] == "dense" else case["nnz"])
    rows = 4 * e if case["feat"] == "dense" else 8 * e
    return rows + 16 * M * B + d * case["b_x"] // 8 + 4 * d + M * d * case["b"] // 8, 4 * e + 4 * M * d


def work(case):
    kind = case["kind"]
    if kind == "objective":
        nbytes, flops = _full_work(case)
    elif kind == "worker":
        nbytes, flops = _worker_work(case)
        nbytes += 4 * case["M"] * case["d"] if case["alpha"] else 0
    elif kind == "epoch":
        nbytes, flops = _full_work(case)
        rb, rf = _worker_work(case)
        M, d = case["M"], case["d"]
        rb += M * d * case["b"] // 8 + 12 * d + d * case["b_x"] // 8 + (16 * d if case["algo"] == "acc" else 0)
        nbytes, flops = nbytes + case["m"] * rb, flops + case["m"] * (rf + 2 * M * d)
    elif kind == "quantize":
        nbytes, flops = case["M"] * case["d"] * (4 + case["b"] / 8), 3 * case["M"] * case["d"]
    elif kind == "aggregate":
        nbytes, flops = case["d"] * (4 + case["M"] * case["b"] / 8), 2 * case["M"] * case["d"]
    else:
        d, M, b = case["d"], case["M"], case["b"]
        nbytes = M * (8 * d + 3 * d * b // 8 + 4 * dq.dq_sparse_stream_words(d, b))
        flops = 6 * M * d
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """Relative error that another correct implementation in the same types would show: about four times what the
    features changed by one unit in their last place make of the outputs (or what they are off 64 bits, if more)."""
    kind = case["kind"]
    if kind in ("quantize", "message"):
        return "exact"                                     # addressed random streams, elementwise float32
    if kind == "aggregate":
        return {"rel": 3e-7, "max": 3e-6}                  # float32 sums over the workers
    if kind == "objective":
        return {"rel": 5e-6, "max": 5e-5}
    # A difference below all of these can still flip the rounding (or the drop) of a coordinate whose random number
    # lies that close to its threshold: one level of one coordinate of one message, and through the rounds of an epoch
    # that coordinate of the model, by a step times the scale over the number of workers.
    if kind == "worker":
        return {"rel": 2e-6, "max": 1e-5, "differ": 1e-3}
    return {"rel": 2e-5, "max": 5e-3, "differ": 1e-3}


# ------------------------------------------------------------------------------------------------ 64 bits
def _dots(p, rows, v):
    """a_i . v over the given rows (None: all), 64 bits."""
    if "dense" in p:
        out = []
        for r in range(0, p["n"] if rows is None else rows.numel(), 8192):
            A = (p["dense"][r:r + 8192] if rows is None else p["dense"][rows[r:r + 8192]]).double()
            out.append((A * v).sum(1))
        return torch.cat(out)
    at, row = _flat(p, rows)
    out = torch.zeros(p["n"] if rows is None else rows.numel(), dtype=torch.float64, device=DEV)
    return out.index_add_(0, row, p["values"][at].double() * v[p["indices"][at].long()])


def _flat(p, rows):
    """Entry numbers of the given CSR rows, one after the other, and the number in `rows` of the row of each."""
    if rows is None:
        rows = torch.arange(p["n"], device=DEV)
    lens = p["indptr"][rows + 1] - p["indptr"][rows]
    row = torch.repeat_interleave(torch.arange(rows.numel(), device=DEV), lens)
    before = torch.cumsum(lens, 0) - lens
    return p["indptr"][rows][row] + torch.arange(row.numel(), device=DEV) - before[row], row


def _combine(p, rows, coef):
    """sum_i coef_i a_i over the given rows (None: all), 64 bits."""
    if "dense" in p:
        out = torch.zeros(p["d"], dtype=torch.float64, device=DEV)
        for r in range(0, coef.numel(), 8192):
            A = (p["dense"][r:r + 8192] if rows is None else p["dense"][rows[r:r + 8192]]).double()
            out += (A * coef[r:r + 8192, None]).sum(0)
        return out
    at, row = _flat(p, rows)
    out = torch.zeros(p["d"], dtype=torch.float64, device=DEV)
    return out.index_add_(0, p["indices"][at].long(), p["values"][at].double() * coef[row])


def _full(p, x, l2, l1):
    y, x = p["y"].double(), x.double()
    z = _dots(p, None, x)
    g = _combine(p, None, -y / (1.0 + torch.exp(y * z)) / p["n"]) + l2 * x
    obj = torch.nn.functional.softplus(-y * z).mean() + 0.5 * l2 * (x * x).sum() + l1 * x.abs().sum()
    return g, z, obj.reshape(1)


def _f32(v):
    """The value that a float argument has once it is a float32."""
    return float(torch.tensor(v, dtype=torch.float32).double())


def exact(case, seed):
    kind, g = case["kind"], _gen(seed)
    if kind == "message":
        return None
    if kind == "quantize":
        v = _matrix(case["M"], case["d"], g)
        top = v.abs().amax(1).double()
        return dict(messages=None, scales=top / ((1 << (case["b"] - 1)) - 1), absmax=top)
    if kind == "aggregate":
        packed, delta = _sums(case, g)
        b, d, M = case["b"], case["d"], case["M"]
        if 32 % b:
            return None
        per = 32 // b
        out = torch.zeros((packed.shape[1], per), dtype=torch.float64, device=DEV)
        for m in range(M):
            for k in range(per):
                out[:, k] += delta[m].double() * ((packed[m] << (32 - b * (k + 1))) >> (32 - b)).double()
        return (out.reshape(-1)[:d] * (_f32(1.0 / M)))
    if kind == "worker":
        p, x0, codes, _, scale, idx = _worker_inputs(case, seed)
        if not case["own"]:
            return None
        x0d, q = x0.double(), codes.double() * scale.double()
        alpha = torch.zeros((case["M"], _pad4(case["d"])), dtype=torch.float64, device=DEV)
        for m in range(case["M"]):
            rows = idx[m].long()
            y, zs, dz = p["y"][rows].double(), _dots(p, rows, x0d), _dots(p, rows, q - x0d)
            slope = lambda z: -y / (1.0 + torch.exp(y * z))                                # noqa: E731
            alpha[m, :case["d"]] = _combine(p, rows, (slope(zs + dz) - slope(zs)) / case["B"]) + _f32(L2) * (q - x0d)
        return dict(messages=None, scales=None, alpha=alpha)
    p, x0 = _problem(case, g)
    if kind == "objective":
        gr, z, obj = _full(p, x0, _f32(L2), _f32(L1))
        return dict(g=gr, z=z, objective=obj)
    gr, z, obj = _full(p, x0, _f32(L2), _f32(L1) if case["feat"] == "csr" else 0.0)        # the rounds have no such value
    out = dict(x=None, g=gr, objective=obj, model=None, model_scale=None, messages=None, scales=None)
    if case["cached"]:
        out["z"] = z
    return out
