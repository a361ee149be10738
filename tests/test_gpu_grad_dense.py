"""GPU parity: dense full gradient, variance-reduced gradient and fused worker step versus the oracle.

Floating-point results are compared at 1e-5 relative to the largest entry of the oracle's
vector (the oracle accumulates in double, the kernels in float32).  Integer results (codes)
are compared bit-exactly against the library's own unfused chain, and against the oracle
up to the rounding decisions that a sub-tolerance difference of alpha can flip.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, host, words

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def dq():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_1805_10111_amd as dq
    return dq


def _ws(dq, op, P, M=1, B=1):
    return dq.new_workspace(op, P, M, B)


def _close(got, want, tol=TOL):
    scale = np.abs(want).max()
    assert np.abs(got.astype(np.float64) - want).max() <= tol * scale + 1e-30, \
        (np.abs(got.astype(np.float64) - want).max(), scale)


def _model(rng, d, b_x, x_snap, spread=0.05):
    """A model near the snapshot and its b_x-bit message (packed words, delta, dequantized q) from the oracle."""
    x = (x_snap + spread * rng.standard_normal(d)).astype(np.float32)
    if b_x == 32:
        return x.view(np.uint32).copy(), np.float32(1.0), x
    k, dx, _ = oracle.quantize(x, b_x, 3, 1, oracle.MASTER_ID, oracle.TAG_MODEL)
    return oracle.pack(k, b_x), dx, oracle.dequantize(k, dx)


# (the last two give a block more rows than one chunk of labels/margins holds: 1024, then a ragged remainder)
PROBLEMS = [(2000, 1000), (37, 13), (300, 4096), (129, 2048), (64, 1027), (150, 6000), (90, 16384), (70, 12003),
            (600011, 8), (1100000, 5)]


@pytest.mark.parametrize("n,d", PROBLEMS)
def test_full_grad(dq, n, d):
    p = synth.dense_logistic(n, d, seed=n + d, l2=1e-3, l1=1e-4)
    lda = (d + 3) // 4 * 4
    if lda != d:                                   # padded rows: padding must be ignored
        Xp = np.full((n, lda), 7.0, dtype=np.float32)
        Xp[:, :d] = p.dense
    else:
        Xp = p.dense
    P = dq.DeviceProblem(n=n, d=d, y=dev(p.y), l2=p.l2, l1=p.l1, dense=dev(Xp)[:, :d])
    rp = oracle.RefProblem(p)
    x = (0.5 * np.random.default_rng(1).standard_normal(d)).astype(np.float32)
    g = torch.zeros(d, device="cuda")
    z = torch.zeros(n, device="cuda")
    obj = torch.zeros(1, dtype=torch.float64, device="cuda")
    ws = _ws(dq, dq.OP_FULL_GRAD, P)
    dq.dq_full_grad(P, dev(x), g, z, obj, ws)
    g_ref, z_ref = oracle.full_grad(rp, x, want_margins=True)
    _close(host(g), g_ref.astype(np.float64))
    _close(host(z), z_ref.astype(np.float64))
    assert abs(host(obj)[0] - oracle.objective(rp, x)) <= TOL * oracle.objective(rp, x)
    # deterministic: a second call gives the same bits
    g2 = torch.zeros(d, device="cuda")
    dq.dq_full_grad(P, dev(x), g2, None, None, ws)
    assert torch.equal(g, g2)


@pytest.mark.parametrize("have_z", [True, False])
@pytest.mark.parametrize("b_x", [8, 4, 32])
@pytest.mark.parametrize("n,d,M,B", [(2000, 1000, 4, 16), (300, 4096, 3, 40), (64, 1027, 2, 5), (500, 2048, 33, 7),
                                     (150, 6000, 3, 40), (90, 16384, 2, 9), (70, 12003, 2, 33)])
def test_vr_grad(dq, n, d, M, B, b_x, have_z):
    p = synth.dense_logistic(n, d, seed=d, l2=1e-3)
    P = dq.DeviceProblem.from_host(p) if d % 4 == 0 else None
    if P is None:
        lda = (d + 3) // 4 * 4
        Xp = np.zeros((n, lda), dtype=np.float32)
        Xp[:, :d] = p.dense
        P = dq.DeviceProblem(n=n, d=d, y=dev(p.y), l2=p.l2, l1=p.l1, dense=dev(Xp)[:, :d])
    rp = oracle.RefProblem(p)
    rng = np.random.default_rng(5)
    x_snap = (0.3 * rng.standard_normal(d)).astype(np.float32)
    xq, dx, q = _model(rng, d, b_x, x_snap)
    idx = np.stack([oracle.sample_indices(n, B, 11, 2, w) for w in range(M)])
    z_snap = None
    if have_z:
        _, z_ref = oracle.full_grad(rp, x_snap, want_margins=True)
        z_snap = dev(z_ref)
    ld = (d + 3) // 4 * 4
    alpha = torch.full((M, ld), 5.0, device="cuda")[:, :d]
    amax = torch.zeros(M, device="cuda")
    l1n = torch.zeros(M, device="cuda")
    ws = _ws(dq, dq.OP_VR_GRAD, P, M, B)
    dq.dq_vr_grad(P, dev(idx), M, B, dev(xq.view(np.int32)), dev(np.array([dx], dtype=np.float32)), b_x, False,
                  dev(x_snap), z_snap, alpha, amax, l1n, ws)
    for w in range(M):
        want = oracle.vr_grad(rp, idx[w], q, x_snap).astype(np.float64)
        got = host(alpha)[w]
        _close(got, want)
        assert host(amax)[w] == np.abs(got).max()
        assert abs(host(l1n)[w] - np.abs(got.astype(np.float64)).sum()) <= 1e-6 * np.abs(got).sum()


def test_vr_grad_flag_bit_and_bad_index(dq):
    n, d, M, B = 200, 1000, 3, 8
    p = synth.dense_logistic(n, d, seed=2)
    P = dq.DeviceProblem.from_host(p)
    x_snap = dev(np.random.default_rng(0).standard_normal(d).astype(np.float32))
    idx = torch.zeros((M, B), dtype=torch.int32, device="cuda")
    alpha = torch.full((M, d), 5.0, device="cuda")
    amax = torch.full((M,), 5.0, device="cuda")
    ws = _ws(dq, dq.OP_VR_GRAD, P, M, B)
    dq.dq_vr_grad(P, idx, M, B, None, None, 8, True, x_snap, None, alpha, amax, None, ws)
    assert not host(alpha).any() and not host(amax).any()
    # worker step in the flag-bit round: zero codes, delta = 0
    packed = torch.full((M, 252), -1, dtype=torch.int32, device="cuda")
    delta = torch.full((M,), 5.0, device="cuda")
    nnz = torch.full((M,), 5, dtype=torch.int32, device="cuda")
    dq.dq_worker_step(P, idx, M, B, None, None, 8, True, x_snap, None, False, 8, 1, 1, 0, packed, delta, nnz, None, None, ws)
    assert not words(packed)[:, :250].any() and not host(delta).any() and not host(nnz).any()
    # indices outside [0, n) are skipped, not dereferenced
    bad = torch.tensor([[0, -1, n, 2 ** 31 - 1, 1, 2, 3, 4]] * M, dtype=torch.int32, device="cuda")
    xq = torch.zeros(250, dtype=torch.int32, device="cuda")
    dq.dq_vr_grad(P, bad, M, B, xq, torch.ones(1, device="cuda"), 8, False, x_snap, None, alpha, amax, None, ws)
    assert np.isfinite(host(alpha)).all()


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("d,M,B", [(4096, 2, 256), (4096, 1, 71), (3000, 2, 70), (4096, 32, 64), (2052, 3, 44),
                                   (2048, 2, 70), (1500, 3, 64), (8192, 2, 40), (6000, 2, 70), (16384, 2, 36),
                                   (12000, 1, 33), (4096, 1, 65536), (2048, 1, 40000),
                                   (1024, 3, 64), (1028, 2, 40), (4100, 2, 40), (8196, 2, 36), (16380, 1, 34)])
def test_vr_grad_row_streaming_paths(dq, d, M, B, bad):
    """Rows wider than 1024 floats are streamed with two row buffers when a block owns whole pairs of batches of valid
    rows, with one buffer when it owns whole batches, and through the checked loop otherwise (ragged last block,
    indices outside [0, n)).  Every path against the oracle; a skipped index contributes nothing but still counts
    in the 1/B of the mean."""
    n = 400
    p = synth.dense_logistic(n, d, seed=d + B, l2=1e-3)
    P = dq.DeviceProblem.from_host(p)
    rp = oracle.RefProblem(p)
    rng = np.random.default_rng(B)
    x_snap = (0.3 * rng.standard_normal(d)).astype(np.float32)
    xq, dx, q = _model(rng, d, 8, x_snap)
    idx = np.stack([oracle.sample_indices(n, B, 17, 3, w) for w in range(M)]).astype(np.int64)
    if bad:                                              # a few rows of every worker are out of range
        for w in range(M):
            pos = rng.choice(B, size=max(1, B // 9), replace=False)
            idx[w, pos] = rng.choice([-1, n, n + 5, 2 ** 31 - 1], size=pos.size)
    _, z_ref = oracle.full_grad(rp, x_snap, want_margins=True)
    alpha = torch.full((M, d), 5.0, device="cuda")
    amax = torch.zeros(M, device="cuda")
    ws = _ws(dq, dq.OP_VR_GRAD, P, M, B)
    dq.dq_vr_grad(P, dev(idx.astype(np.int32)), M, B, dev(xq.view(np.int32)), dev(np.array([dx], dtype=np.float32)), 8, False,
                  dev(x_snap), dev(z_ref), alpha, amax, None, ws)
    dense_part = p.l2 * (q.astype(np.float64) - x_snap.astype(np.float64))
    for w in range(M):
        ok = idx[w][(idx[w] >= 0) & (idx[w] < n)]
        want = (oracle.vr_grad(rp, ok.astype(np.int32), q, x_snap).astype(np.float64) - dense_part) * (ok.size / B) + dense_part
        _close(host(alpha)[w], want, tol=2e-5 if bad else TOL)   # (the oracle's float32 output is rescaled here)
        assert host(amax)[w] == np.abs(host(alpha)[w]).max()


@pytest.mark.parametrize("sparsify", [False, True])
@pytest.mark.parametrize("b", [8, 4, 2])
@pytest.mark.parametrize("n,d,M,B", [(2000, 1000, 4, 16), (300, 4096, 5, 64), (64, 1027, 2, 5), (150, 6000, 3, 40),
                                     (90, 16384, 2, 9)])
def test_worker_step(dq, n, d, M, B, b, sparsify):
    p = synth.dense_logistic(n, d, seed=d + 1, l2=1e-3)
    lda = (d + 3) // 4 * 4
    Xp = np.zeros((n, lda), dtype=np.float32)
    Xp[:, :d] = p.dense
    P = dq.DeviceProblem(n=n, d=d, y=dev(p.y), l2=p.l2, l1=p.l1, dense=dev(Xp)[:, :d])
    rp = oracle.RefProblem(p)
    rng = np.random.default_rng(6)
    x_snap = (0.3 * rng.standard_normal(d)).astype(np.float32)
    xq, dx, q = _model(rng, d, 8, x_snap)
    seed, it, w0 = 77, 9, 100
    idx = np.stack([oracle.sample_indices(n, B, seed, it, w0 + w) for w in range(M)])
    xs_d, xq_d, dx_d, idx_d = dev(x_snap), dev(xq.view(np.int32)), dev(np.array([dx], dtype=np.float32)), dev(idx)
    ws = _ws(dq, dq.OP_VR_GRAD, P, M, B)
    nw = dq.packed_words(d, b)
    ldw = (nw + 3) // 4 * 4
    # fused
    packed = torch.full((M, ldw), -1, dtype=torch.int32, device="cuda")
    delta = torch.zeros(M, device="cuda")
    nnz = torch.zeros(M, dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    alpha_f = torch.zeros((M, lda), device="cuda")[:, :d]
    dq.dq_worker_step(P, idx_d, M, B, xq_d, dx_d, 8, False, xs_d, None, sparsify, b, seed, it, w0, packed, delta, nnz,
                      alpha_f, status, ws)
    # unfused chain of the same library: must agree bit for bit
    alpha = torch.zeros((M, lda), device="cuda")[:, :d]
    amax = torch.zeros(M, device="cuda")
    dq.dq_vr_grad(P, idx_d, M, B, xq_d, dx_d, 8, False, xs_d, None, alpha, amax, None, ws)
    assert torch.equal(alpha, alpha_f)
    v = alpha
    if sparsify:
        beta = torch.zeros((M, lda), device="cuda")[:, :d]
        kept = torch.zeros(M, dtype=torch.int32, device="cuda")
        dq.dq_sparsify(alpha, None, seed, it, w0, beta, amax, kept)
        v = beta
    packed2 = torch.full((M, ldw), -1, dtype=torch.int32, device="cuda")
    delta2 = torch.zeros(M, device="cuda")
    dq.dq_quantize_pack(v, b, amax, True, seed, it, dq.TAG_GRAD, w0, packed2, delta2)
    assert torch.equal(packed[:, :nw], packed2[:, :nw]) and torch.equal(delta, delta2)
    assert np.all(words(packed)[:, nw:] == 0xFFFFFFFF)
    assert host(status)[0] == 0
    # against the oracle: the decoded message is an unbiased rounding of the oracle's vector
    flips = 0
    for w in range(M):
        a_ref = oracle.vr_grad(rp, idx[w], q, x_snap)
        _close(host(alpha_f)[w], a_ref.astype(np.float64))
        v_ref = oracle.sparsify(a_ref, seed, it, w0 + w)[0] if sparsify else a_ref
        k_ref, d_ref, _ = oracle.quantize(v_ref, b, seed, it, w0 + w)
        k = oracle.unpack(words(packed)[w, :nw], d, b)
        assert host(nnz)[w] == np.count_nonzero(k)
        assert abs(host(delta)[w] - d_ref) <= 2e-5 * d_ref
        diff = np.abs(k.astype(np.int32) - k_ref.astype(np.int32))
        if not sparsify:
            assert diff.max() <= 1
            flips += int(diff.sum())
        else:
            # a flipped keep decision changes a code by the full level; count them
            flips += int(np.count_nonzero(diff))
    assert flips <= max(3, 2e-3 * M * d), flips          # decisions flipped by sub-tolerance differences
    # the direct check: the oracle's sparsifier and quantizer applied to the gradient the GPU itself computed give
    # the GPU's message word for word (identical quantizer inputs => identical codes, no flips)
    for w in range(M):
        a_gpu = host(alpha_f)[w]
        v_o = oracle.sparsify(a_gpu, seed, it, w0 + w)[0] if sparsify else a_gpu
        k_o, d_o, _ = oracle.quantize(v_o, b, seed, it, w0 + w)
        assert host(delta)[w] == d_o
        assert np.array_equal(words(packed)[w, :nw], oracle.pack(k_o, b))
        assert host(nnz)[w] == np.count_nonzero(k_o)


def test_worker_step_samples_its_own_minibatch(dq):
    """idx = None: the kernel draws the mini-batch itself, identically to dq_sample_indices."""
    n, d, M, B = 2000, 1000, 4, 16
    p = synth.dense_logistic(n, d, seed=8)
    P = dq.DeviceProblem.from_host(p)
    rng = np.random.default_rng(2)
    x_snap = (0.3 * rng.standard_normal(d)).astype(np.float32)
    xq, dx, _ = _model(rng, d, 8, x_snap)
    seed, it, w0 = 5, 17, 3
    idx = torch.zeros((M, B), dtype=torch.int32, device="cuda")
    dq.dq_sample_indices(n, M, B, seed, it, w0, idx)
    ws = _ws(dq, dq.OP_VR_GRAD, P, M, B)
    outs = []
    for use_idx in (idx, None):
        packed = torch.zeros((M, 252), dtype=torch.int32, device="cuda")
        delta = torch.zeros(M, device="cuda")
        dq.dq_worker_step(P, use_idx, M, B, dev(xq.view(np.int32)), dev(np.array([dx], dtype=np.float32)), 8, False,
                          dev(x_snap), None, False, 8, seed, it, w0, packed, delta, None, None, None, ws)
        outs.append((packed, delta))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    assert outs[0][0].any()


def test_worker_step_full_precision_message(dq):
    """b = 32: the worker sends alpha itself (AsyFPG / QSVRG-style comparison modes)."""
    n, d, M, B = 300, 1000, 2, 8
    p = synth.dense_logistic(n, d, seed=3)
    P = dq.DeviceProblem.from_host(p)
    rng = np.random.default_rng(1)
    x_snap = (0.3 * rng.standard_normal(d)).astype(np.float32)
    x = (x_snap + 0.05 * rng.standard_normal(d)).astype(np.float32)
    idx = dev(np.stack([oracle.sample_indices(n, B, 1, 1, w) for w in range(M)]))
    ws = _ws(dq, dq.OP_VR_GRAD, P, M, B)
    out = torch.zeros((M, d), dtype=torch.float32, device="cuda")
    delta = torch.zeros(M, device="cuda")
    alpha = torch.zeros((M, d), device="cuda")
    dq.dq_worker_step(P, idx, M, B, dev(x).view(torch.int32), None, 32, False, dev(x_snap), None, False, 32, 1, 1, 0,
                      out.view(torch.int32), delta, None, alpha, None, ws)
    assert torch.equal(out, alpha) and host(delta).tolist() == [1.0, 1.0]
    rp = oracle.RefProblem(p)
    for w in range(M):
        _close(host(out)[w], oracle.vr_grad(rp, host(idx)[w], x, x_snap).astype(np.float64))


def test_unsupported_and_invalid(dq):
    p = synth.dense_logistic(20, 16388, seed=0)
    P = dq.DeviceProblem.from_host(p)
    x = torch.zeros(16388, device="cuda")
    with pytest.raises(dq.DqError) as e:
        dq.dq_full_grad(P, x, x.clone(), None, None, torch.zeros(1 << 20, device="cuda"))
    assert e.value.code == dq.ERR_UNSUPPORTED             # dense rows wider than 16384 floats have no kernel
    p = synth.dense_logistic(20, 64, seed=0)
    P = dq.DeviceProblem.from_host(p)
    x = torch.zeros(64, device="cuda")
    with pytest.raises(dq.DqError) as e:
        dq.dq_full_grad(P, x, x.clone(), None, None, torch.zeros(4, device="cuda"))
    assert e.value.code == dq.ERR_WORKSPACE


@pytest.mark.parametrize("n,d", [(3001, 1), (4097, 54), (2500, 64), (999, 65), (700, 128), (1203, 131), (4100, 256), (900, 257),
                                 (400, 1025), (300, 1290), (1100, 2045), (41000, 2047), (77, 2500), (130, 3000), (90, 4099), (40, 7397), (33, 8200), (50, 12002),
                                 (40, 8193), (33, 8197), (50, 8957), (33, 10243), (40, 12290), (33, 12291), (21, 16383),
                                 (1, 54), (2, 3000)])
def test_full_gradient_over_widths(dq, n, d):
    """Rows on 16, 32 and 64 lanes, and every count of threads and columns per thread, with ragged last quads whose padding is
    not a number."""
    rng = np.random.default_rng(n + d)
    lda = (d + 3) // 4 * 4 + 4
    X = np.full((n, lda), np.nan, dtype=np.float32)
    X[:, :d] = rng.standard_normal((n, d)).astype(np.float32) / np.sqrt(d)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    x = rng.standard_normal(d).astype(np.float32)
    P = dq.DeviceProblem(n=n, d=d, y=dev(y), l2=1e-3, l1=1e-4, dense=dev(X)[:, :d])
    g, z, obj = torch.zeros(d, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    dq.dq_full_grad(P, dev(x), g, z, obj, dq.new_workspace(dq.OP_FULL_GRAD, P))
    ref = oracle.RefProblem(synth.Problem(n=n, d=d, y=y, l2=1e-3, l1=1e-4, dense=np.ascontiguousarray(X[:, :d])))
    want_g, want_z = oracle.full_grad(ref, x, want_margins=True)
    assert np.abs(host(z) - want_z).max() <= 1e-5 * np.abs(want_z).max() + 1e-7
    assert np.abs(host(g) - want_g).max() <= 1e-5 * np.abs(want_g).max() + 1e-9
    assert abs(host(obj)[0] - oracle.objective(ref, x)) <= 1e-5 * abs(oracle.objective(ref, x))


@pytest.mark.parametrize("d,M,B", [(54, 3, 5), (1000, 2, 5), (1000, 3, 33), (1500, 2, 5), (2500, 2, 5), (5000, 2, 3), (12002, 2, 7),
                                   (2500, 12, 90)])
def test_an_infinite_feature_reaches_its_own_column_only(dq, d, M, B):
    """A row with an infinite feature, the last of a block's: the gradient is infinite in that column and finite in all others.
    (A row that is requested twice to fill up a batch must not be added a second time: 0 * Inf is not a number.)"""
    n, j = 7, d // 2
    rng = np.random.default_rng(d)
    X = (rng.standard_normal((n, (d + 3) // 4 * 4)) / np.sqrt(d)).astype(np.float32)
    X[n - 1, j] = np.inf
    x_snap = np.zeros(d, dtype=np.float32)
    q = rng.standard_normal(d).astype(np.float32)
    q[j] = 1.0
    y = -np.ones(n, dtype=np.float32)
    P = dq.DeviceProblem(n=n, d=d, y=dev(y), l2=0.0, l1=0.0, dense=dev(X)[:, :d])
    idx = np.full((M, B), n - 1, dtype=np.int32)
    idx[:, :-1] = rng.integers(0, n - 1, (M, B - 1))
    ld = (d + 3) // 4 * 4
    alpha, amax = torch.zeros((M, ld), device="cuda")[:, :d], torch.zeros(M, device="cuda")
    dq.dq_vr_grad(P, dev(idx).view(-1), M, B, dev(q).view(torch.int32), None, 32, False, dev(x_snap), torch.zeros(n, device="cuda"),
                  alpha, amax, None, dq.new_workspace(dq.OP_VR_GRAD, P, M, B))
    a = host(alpha)
    assert np.isinf(host(amax)).all() and np.isinf(a[:, j]).all() and np.isfinite(np.delete(a, j, 1)).all()


@pytest.mark.parametrize("d", [1, 54, 100, 200, 256])
def test_an_infinite_feature_in_the_full_gradient_of_narrow_rows(dq, d):
    n, j = 37, d // 2
    rng = np.random.default_rng(d)
    X = rng.standard_normal((n, (d + 3) // 4 * 4)).astype(np.float32)
    X[n - 1, j] = np.inf
    x = np.ones(d, dtype=np.float32)
    y = -np.ones(n, dtype=np.float32)                      # (margin +Inf with label -1: slope 1)
    P = dq.DeviceProblem(n=n, d=d, y=dev(y), l2=0.0, l1=0.0, dense=dev(X)[:, :d])
    g = torch.zeros(d, device="cuda")
    dq.dq_full_grad(P, dev(x), g, None, None, dq.new_workspace(dq.OP_FULL_GRAD, P))
    assert host(g)[j] == np.inf and np.isfinite(np.delete(host(g), j)).all()


@pytest.mark.parametrize("d", [16, 33, 64, 100, 128, 256, 1000])
def test_all_columns_of_a_row_get_the_same_coefficient(dq, d):
    """One row of powers of two: the gradient divided by the feature is exact, and is the row's coefficient in every column,
    whatever the order in which the lanes added up the margin."""
    rng = np.random.default_rng(d)
    g = torch.zeros(d, device="cuda")
    for _ in range(30):
        X = np.ldexp(rng.choice([-1.0, 1.0], (1, (d + 3) // 4 * 4)), rng.integers(-3, 3, (1, (d + 3) // 4 * 4))).astype(np.float32)
        x = (0.1 * rng.standard_normal(d)).astype(np.float32)
        P = dq.DeviceProblem(n=1, d=d, y=torch.ones(1, device="cuda"), l2=0.0, l1=0.0, dense=dev(X)[:, :d])
        dq.dq_full_grad(P, dev(x), g, None, None, dq.new_workspace(dq.OP_FULL_GRAD, P))
        coef = host(g) / X[0, :d]
        assert np.unique(coef).size == 1 and coef[0] < 0


@pytest.mark.parametrize("n,d", [(40000, 2500), (30000, 5000), (12000, 10000)])
def test_full_gradient_is_no_coarser_than_512_float32_sums(dq, n, d):
    """With several columns per thread there are 256 blocks; the gradient is all the same as close to 64 bits as 512 float32
    sums over n/512 rows each, one row after the other, leave it.  Beside those sums it has the roundings of the
    coefficients and of the sum of the blocks' vectors, 2^-24 of their values each: two of them, in quadrature."""
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, (d + 3) // 4 * 4), device="cuda", generator=g)[:, :d] / d ** 0.5
    X = torch.nn.functional.pad(X, (0, -d % 4))[:, :d]
    x = 0.5 * torch.randn(d, device="cuda", generator=g)
    y = torch.where(torch.rand(n, device="cuda", generator=g) < 0.5, 1.0, -1.0)
    out = torch.zeros(d, device="cuda")
    P = dq.DeviceProblem(n=n, d=d, y=y, l2=0.0, l1=0.0, dense=X)
    dq.dq_full_grad(P, x, out, None, None, dq.new_workspace(dq.OP_FULL_GRAD, P))
    exact, parts, per = torch.zeros(d, dtype=torch.float64, device="cuda"), torch.zeros((512, d), device="cuda"), -(-n // 512)
    z = torch.cat([(X[r:r + 4096].double() * x.double()).sum(1) for r in range(0, n, 4096)])
    coef = -y.double() / (1.0 + torch.exp(y.double() * z)) / n
    for r in range(0, n, 4096):
        exact += (X[r:r + 4096].double() * coef[r:r + 4096, None]).sum(0)
    first = torch.arange(512, device="cuda") * per
    for k in range(per):
        rows = first + k
        live = (rows < n).float()[:, None]
        parts += coef.float()[rows.clamp(max=n - 1), None] * X[rows.clamp(max=n - 1)] * live
    plain = (parts.double().sum(0).float().double() - exact).norm() / exact.norm()
    mine = (out.double() - exact).norm() / exact.norm()
    assert mine <= (plain ** 2 + (2 * 2.0 ** -24) ** 2) ** 0.5


@pytest.mark.parametrize("M,B,P", [(2, 4, 1), (2, 8, 1), (2, 12, 1), (2, 16, 1), (2, 20, 1), (2, 24, 1), (2, 28, 1), (2, 33, 9), (2, 40, 10),
                                   (2, 44, 11), (2, 48, 12), (2, 52, 13), (2, 56, 14), (2, 60, 15), (2, 64, 16), (2, 72, 18), (2, 76, 19),
                                   (2, 150, 10), (2, 240, 15), (256, 40, 2), (32, 40, 3), (32, 56, 4), (16, 70, 5), (2, 90, 6), (2, 100, 7),
                                   (2, 120, 8)])
@pytest.mark.parametrize("b_x", [8, 32])
def test_any_number_of_partial_sums(dq, M, B, P, b_x):
    """A worker's mini-batch on P blocks: the second kernel adds their partial sums eight at a time, then a rest of any size
    (P = 1: no second kernel; else every rest of eight occurs, with eight sums before it and without; P is seen in the workspace,
    of which the step writes M P rows)."""
    n, d = 300, 260
    p = synth.dense_logistic(n, d, seed=d, l2=1e-3)
    prob, rp, rng = dq.DeviceProblem.from_host(p), oracle.RefProblem(p), np.random.default_rng(6)
    x_snap = (0.3 * rng.standard_normal(d)).astype(np.float32)
    xq, dx, q = _model(rng, d, b_x, x_snap)
    idx = np.stack([oracle.sample_indices(n, B, 11, 2, w) for w in range(M)])
    _, z_ref = oracle.full_grad(rp, x_snap, want_margins=True)
    alpha, amax = torch.full((M, d), 5.0, device="cuda"), torch.zeros(M, device="cuda")
    ws = _ws(dq, dq.OP_VR_GRAD, prob, M, B).fill_(-77.0)
    dq.dq_vr_grad(prob, dev(idx), M, B, dev(xq.view(np.int32)), dev(np.array([dx], dtype=np.float32)), b_x, False,
                  dev(x_snap), dev(z_ref), alpha, amax, None, ws)
    rows = ws[:ws.numel() // d * d].reshape(-1, d)
    assert int((rows != -77.0).all(1).sum()) == (M * P if P > 1 else 0)
    for w in range(M):
        _close(host(alpha)[w], oracle.vr_grad(rp, idx[w], q, x_snap).astype(np.float64))
