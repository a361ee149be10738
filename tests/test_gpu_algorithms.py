"""GPU parity of whole rounds and epochs (Alg. 1-3) against the oracle's loops.

Two protocols.  Lock-step: before every round the GPU state is overwritten with the
oracle's, the GPU runs the round, and its outputs are compared with the oracle's round
(codes up to decisions flipped by sub-tolerance differences of alpha; the new model to
1e-5).  Free run: both sides run whole epochs independently from the same seed and the
objectives at the snapshots are compared.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import algorithms as alg
import synth
from gpu_util import dev, host, launches, words

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def dq():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_1805_10111_amd as dq
    return dq


def _trainer(dq, p, cfg, m, seed):
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    P = dq.DeviceProblem.from_host(p)
    return DoubleQuantTrainer(P, cfg.algo, cfg.M, cfg.B, cfg.b_x, cfg.b, m, cfg.lr, seed=seed)


def _small(cfg_name):
    cfg = synth.CONFIGS[cfg_name]
    if cfg_name == "C1":
        return cfg, synth.make_problem(cfg), 40
    if cfg_name == "C4":
        return cfg, synth.make_problem(cfg, n=3000), 6
    return cfg, synth.make_problem(cfg, n=4000), 12


@pytest.mark.parametrize("name", ["C1", "C4", "C2", "C3"])
def test_lock_step_rounds(dq, name):
    cfg, p, m = _small(name)
    seed = 3
    tr = _trainer(dq, p, cfg, m, seed)
    rp = oracle.RefProblem(p)
    d, M, B, b, bx = p.d, cfg.M, cfg.B, cfg.b, cfg.b_x
    acc = cfg.algo == "acc"
    x_snap = np.zeros(d, dtype=np.float32)
    y = x_snap.copy()
    flips = total = 0
    for e in range(2):
        # ---- oracle epoch start
        if acc:
            theta = np.float32(2.0 / (e + 3))
            eta = np.float32(np.float32(cfg.lr) / theta)
            x = oracle.acc_mix(y, x_snap, theta)
            xsum = np.zeros(d, dtype=np.float32)
        else:
            theta, eta = np.float32(0), np.float32(cfg.lr)
            x = x_snap.copy()
        g_snap = oracle.full_grad(rp, x_snap)
        # ---- GPU epoch start from the oracle's state
        tr.epoch_index = e
        tr.x_snap.copy_(dev(x_snap)); tr.y.copy_(dev(y))
        tr.epoch_prologue()
        assert np.abs(host(tr.g_snap) - g_snap).max() <= TOL * np.abs(g_snap).max()
        assert np.array_equal(host(tr.x), x)
        for t in range(m):
            it = e * m + t
            q, xq_words, dx, bits = alg.model_message(x, x_snap, bx, seed, it)
            flag = bits == 1
            # overwrite the GPU state with the oracle's
            tr.x.copy_(dev(x)); tr.g_snap.copy_(dev(g_snap))
            if acc:
                tr.y.copy_(dev(y)); tr.xsum.copy_(dev(xsum))
            if not flag:
                tr.xq[: xq_words.size].copy_(dev(xq_words.view(np.int32)))
                tr.delta_x.copy_(dev(np.array([dx], dtype=np.float32)))
            assert tr.round(t) == flag
            # ---- oracle round
            codes = np.zeros((M, d), dtype=np.int8)
            deltas = np.zeros(M, dtype=np.float32)
            for w in range(M):
                wd, dl, _, _, _, _ = alg.worker_message(rp, q, x_snap, flag, B, b, seed, it, w, cfg.algo == "sparse")
                codes[w] = oracle.unpack(wd, d, b)
                deltas[w] = dl
            if acc:
                oracle.master_update(codes, deltas, np.float32(1.0 / M), g_snap, x, y, x_snap, xsum, eta=eta,
                                     theta=theta, l1=rp.l1)
            else:
                oracle.master_update(codes, deltas, np.float32(1.0 / M), g_snap, x, eta=eta, l1=rp.l1)
            # ---- compare the round
            got_codes = np.stack([oracle.unpack(words(tr.packed)[w], d, b) for w in range(M)])
            diff = np.abs(got_codes.astype(np.int32) - codes)
            assert diff.max() <= 1
            flips += int(diff.sum()); total += diff.size
            assert np.all(np.abs(host(tr.delta) - deltas) <= 2e-5 * deltas + 1e-30)
            scale = max(np.abs(x).max(), 1e-30)
            # a flipped code moves a coordinate by eta*delta/M; everything else agrees to rounding
            bound = TOL * scale + float(eta) * float(deltas.max()) / M * (diff.max(axis=0) > 0)
            assert np.all(np.abs(host(tr.x) - x) <= bound + 1e-7 * scale)
        if acc:
            x_snap = oracle.acc_snapshot(xsum, m)
        else:
            x_snap = x.copy()
        tr.x.copy_(dev(x))
        if acc:
            tr.xsum.copy_(dev(xsum)); tr.y.copy_(dev(y))
        tr.epoch_epilogue()
        assert np.array_equal(host(tr.x_snap), x_snap)
    assert flips <= max(2, 1e-3 * total), (flips, total)


@pytest.mark.parametrize("name", ["C1", "C4", "C2", "C3"])
def test_free_run_objectives(dq, name):
    cfg, p, m = _small(name)
    S = 2
    tr = _trainer(dq, p, cfg, m, seed=0)
    log = tr.run(S)
    ref = alg.run(p, cfg.algo, cfg.M, cfg.B, cfg.b_x, cfg.b, m, S, cfg.lr, seed=0)
    assert len(log.objectives) == len(ref.objectives) == S + 1
    for a, b in zip(log.objectives, ref.objectives):
        assert abs(a - b) <= TOL * abs(b), (log.objectives, ref.objectives)
    assert log.objectives[-1] < log.objectives[0]
    assert log.bits_up == ref.bits_up and log.bits_down == ref.bits_down
    rel = np.abs(host(tr.x_snap) - ref.x_snap).max() / np.abs(ref.x_snap).max()
    assert rel < 1e-3, rel       # free-running trajectories differ by a few flipped roundings


def test_flag_bit_rule_when_an_update_leaves_the_model_at_the_snapshot(dq):
    """Section 4.1 sends one flag bit when the model equals the snapshot.  The library decides that from where a round
    stands in the epoch (first round of an epoch that starts at the snapshot); the oracle compares the two vectors bit
    for bit at every round.  The two rules part only when an update returns the model to the snapshot exactly -- here a
    prox that zeroes every step from a zero start.  What must hold then: the same iterates and gradient messages
    (the quantized model of an all-zero vector is the snapshot itself, so the workers' gradients vanish either way),
    and a download count that differs by exactly the model messages the library sends where the oracle sends flags."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    n, d, M, B, m, S = 400, 256, 4, 8, 6, 2
    p = synth.dense_logistic(n, d, seed=4, l2=1e-4, l1=10.0)          # l1 far above any gradient entry: prox gives 0
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), "asylpg", M, B, 8, 8, m, 0.1, seed=2)
    log = tr.run(S)
    ref = alg.run(p, "asylpg", M, B, 8, 8, m, S, 0.1, seed=2)
    assert not host(tr.x).any() and not ref.x.any()                    # the model never leaves the snapshot
    assert not host(tr.delta).any() and not words(tr.packed).any()     # all-zero gradient messages, scale 0
    for a, b in zip(log.objectives, ref.objectives):
        assert abs(a - b) <= TOL * abs(b)
    assert log.bits_up == ref.bits_up
    assert ref.bits_down == S * m                                      # the oracle: a flag bit every round
    assert log.bits_down == S * (1 + (m - 1) * (32 + 8 * d))           # the library: a flag at the epoch start only


def test_runs_are_reproducible(dq):
    cfg, p, m = _small("C1")
    a = _trainer(dq, p, cfg, 10, seed=5); a.run(2)
    b = _trainer(dq, p, cfg, 10, seed=5); b.run(2)
    c = _trainer(dq, p, cfg, 10, seed=6); c.run(2)
    assert torch.equal(a.x_snap, b.x_snap) and torch.equal(a.packed, b.packed)
    assert not torch.equal(a.x_snap, c.x_snap)


@pytest.mark.parametrize("algo,b,d,M,B,b_x", [("acc", 8, 4096, 32, 256, 8), ("asylpg", 4, 4096, 16, 64, 8),
                                              ("sparse", 4, 3000, 8, 128, 8), ("acc", 2, 2048, 32, 128, 8),
                                              ("asylpg", 8, 1500, 4, 64, 8), ("asylpg", 8, 4096, 8, 64, 4),
                                              ("acc", 4, 2048, 16, 64, 2), ("acc", 8, 8192, 8, 32, 8),
                                              ("asylpg", 8, 6004, 8, 16, 4), ("acc", 8, 4096, 32, 256, 11)])
def test_rounds_enqueued_together_equal_rounds_enqueued_one_by_one(dq, algo, b, d, M, B, b_x):
    """How the rounds of an epoch are spread over dq_run_rounds calls (3 + 4 rounds, or one round per call) must not
    matter: every vector and every message comes out identical, bit for bit.  (Between the rounds of one call the
    model is quantized by the next round's row-streaming kernel instead of the master's: one round per call never
    takes that path, several rounds per call do wherever the shape allows it.)"""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.dense_logistic(600, d, seed=d + M, l2=1e-3)
    P = dq.DeviceProblem.from_host(p)
    m = 7
    runs = []
    for together in (True, False):
        tr = DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.1, seed=9)
        for _ in range(2):
            tr.epoch_prologue()
            if together:
                tr.rounds(0, 3)
                tr.rounds(3, m - 3)
            else:
                for t in range(m):
                    tr.rounds(t, 1)
            tr.epoch_epilogue()
        torch.cuda.synchronize()
        runs.append(tr)
    a, c = runs
    for name in ("x", "x_snap", "packed", "delta", "xq", "delta_x", "absmax_x"):
        assert torch.equal(getattr(a, name), getattr(c, name)), name
    if algo == "acc":
        assert torch.equal(a.y, c.y) and torch.equal(a.xsum, c.xsum)
    assert np.isfinite(host(a.x)).all() and host(a.x).any()


@pytest.mark.parametrize("algo,b,M,B,b_x,cache", [
    ("asylpg", 8, 8, 32, 8, True), ("sparse", 4, 16, 64, 8, True), ("asylpg", 4, 3, 20, 4, True),
    ("sparse", 8, 40, 16, 2, True), ("asylpg", 8, 8, 32, 11, True),
    ("asylpg", 8, 4, 88, 8, True),        # about 4500 entries per mini-batch: more than a thread stages in one go
    ("asylpg", 8, 2, 128, 8, True),       # about 6500: more than the staging buffer holds, nothing is prepared ahead
    ("asylpg", 8, 2, 300, 8, True),       # more rows than one pass takes
    ("sparse", 4, 64, 8, 8, True),        # many workers: one block each
    ("asylpg", 8, 8, 32, 8, False), ("sparse", 4, 16, 64, 8, False),     # margins at the snapshot recomputed
    ("asylpg", 8, 4, 88, 8, False),       # ... with their smaller staging buffer: not prepared ahead
    ("acc", 8, 8, 32, 8, True), ("acc", 4, 16, 64, 4, True)])            # Alg. 3 on the same features
def test_rounds_enqueued_together_equal_rounds_enqueued_one_by_one_sparse_features(dq, algo, b, M, B, b_x, cache):
    """The same for CSR features (the shape of configs C2 and C3).  With several rounds per call the master leaves
    (decoded model) - snapshot for the next round's workers, may quantize the sparsified gradients itself, and every
    worker launch draws, reads and lays out the next round's mini-batches in blocks of its own; rounds enqueued one
    per call do none of that.  Messages, scales and iterates must agree bit for bit."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.make_problem(synth.CONFIGS["C2"], n=3000)
    P = dq.DeviceProblem.from_host(p)
    m = 6
    runs = []
    for together in (True, False):
        tr = DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.5, seed=4, cache_margins=cache)
        for _ in range(2):
            tr.epoch_prologue()
            if together:
                tr.rounds(0, 4)
                tr.rounds(4, m - 4)
            else:
                for t in range(m):
                    tr.rounds(t, 1)
            tr.epoch_epilogue()
        torch.cuda.synchronize()
        runs.append(tr)
    a, c = runs
    for name in ("x", "x_snap", "packed", "delta", "xq", "delta_x", "absmax_x", "nnz") + (("y", "xsum") if algo == "acc" else ()):
        assert torch.equal(getattr(a, name), getattr(c, name)), name
    assert np.isfinite(host(a.x)).all() and host(a.x).any() and host(a.status)[0] == 0


@pytest.mark.parametrize("b,M,each,b_x,counts", [(4, 16, False, 8, True), (8, 24, False, 8, True), (4, 5, True, 4, True),
                                                  (8, 32, True, 32, True), (2, 8, False, 8, True), (2, 8, False, 8, False),
                                                  (4, 20, False, 8, False)])
@pytest.mark.parametrize("shape", ["C3", "ragged"])
def test_master_that_quantizes_the_sparsified_gradients_equals_the_separate_steps(dq, b, M, each, b_x, counts, shape):
    """Alg. 2 on CSR features wide enough for the sparsifier to be split over several blocks per worker: inside
    dq_run_rounds the master kernel quantizes the workers' sparsified gradients while it aggregates them.  A round
    enqueued that way must leave messages, scales, nonzero counts, the model and the model's message bit for bit
    as dq_worker_step followed by dq_master_step do, which quantize in a launch of their own (M = 20, 24 and 32: more
    workers than one pass of the kernel takes; b = 2 with nonzero counts: the route is not taken, both sides are the
    separate steps; without counts (`nnz` null in the run state) 2-bit messages take it too)."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    # ("ragged": 4099 columns, the narrowest kind of model the route is taken for, its last quad one coordinate long)
    p = synth.make_problem(synth.CONFIGS["C3"], n=3000) if shape == "C3" else \
        synth.sparse_text_logistic(500, 4099, mean_nnz=30.0, seed=3)
    P = dq.DeviceProblem.from_host(p)
    B, m, seed = 32, 4, 9
    one = DoubleQuantTrainer(P, "sparse", M, B, b_x, b, m, 0.5, seed=seed, each=each)
    two = DoubleQuantTrainer(P, "sparse", M, B, b_x, b, m, 0.5, seed=seed, each=each)
    if not counts:
        one.state.nnz = None
        two.state.nnz = None
    one.epoch_prologue(); two.epoch_prologue()
    one.rounds(0, 3)
    idx = torch.empty(M * B, dtype=torch.int32, device="cuda")
    for t in range(3):
        if t == 0:
            two.rounds(0, 1)                               # (the model is the snapshot: all-zero messages)
            continue
        dq.dq_sample_indices(P.n, M, B, seed, t, 0, idx)
        dq.dq_worker_step(P, idx, M, B, two.xq, two.delta_x, b_x, False, two.x_snap, two.z_snap, True, b, seed, t, 0,
                          two.packed, two.delta, nnz_out=two.nnz[t] if counts else None, status=two.status, ws=two.ws)
        step = dq.dq_master_step_each if each else dq.dq_master_step
        args = (two.packed, two.delta, M, b) + (() if each else (float(np.float32(1) / np.float32(M)),))
        step(*args, two.g_snap, two.x, None, two.x_snap, None, two.eta, 0.0, P.l1, b_x, seed, t + 1,
             two.xq, two.delta_x, two.absmax_x[t & 1:], two.status)
    torch.cuda.synchronize()
    for name in ("packed", "delta", "nnz", "x", "xq", "delta_x", "status"):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    assert host(one.x).any() and host(one.packed).any() and host(one.status)[0] == 0
    assert host(one.nnz)[1:3].all() if counts else not host(one.nnz).any()


@pytest.mark.parametrize("name", ["C1", "C4", "C2"])
def test_kernel_events_time_the_worker_kernel_and_change_nothing(dq, name):
    """dq_run_rounds with worker_events: each pair receives the start and end of the row-streaming kernel's launch
    (a positive duration far below a millisecond on these sizes) and the round computes exactly what it computes
    without events."""
    cfg, p, m = _small(name)
    m = min(m, 6)
    a = _trainer(dq, p, cfg, m, seed=3)
    b = _trainer(dq, p, cfg, m, seed=3)
    a.epoch_prologue(); b.epoch_prologue()
    pairs = []
    for t in range(m):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(); e1.record()                       # creates the HIP events
        a.rounds(t, 1, [e0.cuda_event, e1.cuda_event])
        pairs.append((e0, e1, a.is_flag_round(t)))
    b.rounds(0, m)
    torch.cuda.synchronize()
    assert torch.equal(a.x, b.x) and torch.equal(a.packed, b.packed) and torch.equal(a.delta, b.delta)
    timed = [e0.elapsed_time(e1) for e0, e1, flag in pairs if not flag]
    assert len(timed) >= m - 1
    assert all(1e-4 < ms < 1.0 for ms in timed), timed


@pytest.mark.parametrize("algo,b_x,b", [("asylpg", 32, 32), ("acc", 32, 32), ("asylpg", 32, 8), ("asylpg", 8, 32),
                                        ("sparse", 32, 4)])
def test_unquantized_modes_free_run(dq, algo, b_x, b):
    """b = 32 / b_x = 32: AsyFPG, Acc-AsyFPG and QSVRG-style runs through the same kernels."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    cfg = synth.CONFIGS["C1"]
    p = synth.make_problem(cfg, n=600, d=200)
    m, S = 12, 2
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), algo, cfg.M, cfg.B, b_x, b, m, cfg.lr, seed=4)
    log = tr.run(S)
    ref = alg.run(p, algo, cfg.M, cfg.B, b_x, b, m, S, cfg.lr, seed=4)
    for a, r in zip(log.objectives, ref.objectives):
        assert abs(a - r) <= TOL * abs(r)
    assert log.bits_down == ref.bits_down
    if algo != "sparse":
        assert log.bits_up == ref.bits_up
    else:
        assert abs(log.bits_up - ref.bits_up) <= 0.01 * ref.bits_up      # a flipped keep decision moves a few codes
    rel = np.abs(host(tr.x_snap) - ref.x_snap).max() / np.abs(ref.x_snap).max()
    assert rel < (2e-5 if (b, b_x) == (32, 32) else 2e-3), rel


def test_comparison_of_the_six_algorithms(dq):
    from paper_1805_10111_amd.compare import run_comparison
    cfg = synth.CONFIGS["C1"]
    p = synth.make_problem(cfg, n=1000, d=400)
    res = run_comparison(cfg, p, epochs=3, threshold=0.69, b=8, m=40)
    assert set(res) == {"AsyFPG", "Acc-AsyFPG", "QSVRG", "AsyLPG", "Sparse-AsyLPG", "Acc-AsyLPG"}
    fp, lp, qs, sp = res["AsyFPG"], res["AsyLPG"], res["QSVRG"], res["Sparse-AsyLPG"]
    assert lp["bits_total"] < qs["bits_total"] < fp["bits_total"]
    assert sp["bits_total"] < lp["bits_total"]
    assert abs(lp["objectives"][-1] - fp["objectives"][-1]) < 0.01 * fp["objectives"][-1]
    assert 3.5 < fp["bits_total"] / lp["bits_total"] < 4.1        # (32 d) / (32 + 8 d) per message


def test_mu_trace_follows_the_papers_observation(dq):
    """Fig. 2 of the paper: the mu needed for condition (2) is largest right after the snapshot
    (x is still close to it) and falls as x moves away within the epoch."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    cfg = synth.CONFIGS["C1"]
    p = synth.make_problem(cfg, n=600, d=200)
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), "asylpg", cfg.M, cfg.B, 8, 8, 30, cfg.lr, seed=1)
    tr.run_epoch(record_mu=True)
    tr.run_epoch(record_mu=True)
    assert len(tr.mu_trace) == 60
    # (in the very first epoch the snapshot is 0 and both sides scale with ||x||^2: the ratio is flat)
    mus = [r[2] / r[3] for r in tr.mu_trace if r[0] == 1 and r[3] > 0]
    assert all(np.isfinite(mus))
    assert mus[0] == max(mus) and mus[0] > 10 * mus[-1]


@pytest.mark.parametrize("name,algo,tau,b_x,b", [("C1", "asylpg", 1, 8, 8), ("C1", "asylpg", 3, 8, 8), ("C1", "acc", 2, 8, 8),
                                                 ("C1", "asylpg", 3, 32, 32), ("C2", "asylpg", 3, 8, 8), ("C3", "sparse", 5, 8, 4)])
def test_bounded_delay_free_run(dq, name, algo, tau, b_x, b):
    """Emulated staleness (Assumption 3): worker group g reads the model of g rounds ago."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    cfg = synth.CONFIGS[name]
    p = synth.make_problem(cfg, n=1500) if cfg.csr else synth.make_problem(cfg, n=600, d=200)
    m, S = 10, 2
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), algo, cfg.M, cfg.B, b_x, b, m, cfg.lr, seed=2, tau=tau)
    log = tr.run(S)
    ref = alg.run(p, algo, cfg.M, cfg.B, b_x, b, m, S, cfg.lr, seed=2, tau=tau)
    sync = alg.run(p, algo, cfg.M, cfg.B, b_x, b, m, S, cfg.lr, seed=2)
    for a, r in zip(log.objectives, ref.objectives):
        assert abs(a - r) <= TOL * abs(r)
    rel = np.abs(host(tr.x_snap) - ref.x_snap).max() / np.abs(ref.x_snap).max()
    assert rel < 2e-3, rel
    # the delay is visible: the delayed trajectory differs from the synchronous one by more than that
    assert np.abs(ref.x_snap - sync.x_snap).max() / np.abs(ref.x_snap).max() > 5 * max(rel, 1e-6)
    assert log.bits_down == ref.bits_down


def test_delay_argument_checks(dq):
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    cfg = synth.CONFIGS["C1"]
    p = synth.make_problem(cfg, n=100, d=64)
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), "asylpg", cfg.M, cfg.B, 8, 8, 4, cfg.lr, tau=cfg.M)
    with pytest.raises(dq.DqError) as e:          # at most one delay group per worker
        tr.run_epoch()
    assert e.value.code == dq.ERR_INVALID_ARG


@pytest.mark.parametrize("algo,b_x,b,tau", [("asylpg", 8, 8, 0), ("asylpg", 32, 32, 0), ("acc", 8, 8, 0), ("sparse", 8, 4, 0),
                                             ("asylpg", 8, 8, 3)])
def test_one_master_update_per_gradient_free_run(dq, algo, b_x, b, tau):
    """Alg. 1 taken literally at the master: every message is its own update; with tau = M - 1 on top, worker w
    computes on a model that is w rounds old -- the paper's asynchronous picture on one GPU."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    cfg = synth.CONFIGS["C1"]
    p = synth.make_problem(cfg, n=600, d=200)
    m, S, lr = 10, 2, 0.03
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), algo, cfg.M, cfg.B, b_x, b, m, lr, seed=5, tau=tau, each=True)
    log = tr.run(S)
    ref = alg.run(p, algo, cfg.M, cfg.B, b_x, b, m, S, lr, seed=5, tau=tau, each=True)
    for a, r in zip(log.objectives, ref.objectives):
        assert abs(a - r) <= TOL * abs(r)
    assert log.bits_down == ref.bits_down
    mean_mode = alg.run(p, algo, cfg.M, cfg.B, b_x, b, m, S, lr, seed=5, tau=tau)
    assert abs(mean_mode.objectives[-1] - ref.objectives[-1]) > 1e-4          # the two aggregation rules differ


@pytest.mark.parametrize("algo,b", [("asylpg", 8), ("sparse", 4)])
def test_free_run_on_a_model_wider_than_the_on_chip_buffer(dq, algo, b):
    """rcv1-like width (47,236 features): the CSR worker builds its gradient in two column windows."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.sparse_text_logistic(1500, 47236, mean_nnz=75.0, seed=4, l2=1e-4, l1=1e-5)
    M, B, m, S, lr = 4, 16, 6, 2, 0.1
    tr = DoubleQuantTrainer(dq.DeviceProblem.from_host(p), algo, M, B, 8, b, m, lr, seed=2)
    log = tr.run(S)
    ref = alg.run(p, algo, M, B, 8, b, m, S, lr, seed=2)
    for a, r in zip(log.objectives, ref.objectives):
        assert abs(a - r) <= TOL * abs(r)
    assert log.bits_down == ref.bits_down
    if algo == "asylpg":
        assert log.bits_up == ref.bits_up


def test_sparse_messages_through_the_wire_format(dq):
    """Alg. 2 with every message really encoded as (position, value) entries (Section 4.2) and decoded again
    before the master uses it: same trajectory bit for bit, and the entry counts are the ones the bit counter uses."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    cfg = synth.CONFIGS["C3"]
    p = synth.make_problem(cfg, n=3000)
    P = dq.DeviceProblem.from_host(p)
    m, S = 6, 2
    a = DoubleQuantTrainer(P, "sparse", cfg.M, cfg.B, cfg.b_x, cfg.b, m, cfg.lr, seed=3)
    b = DoubleQuantTrainer(P, "sparse", cfg.M, cfg.B, cfg.b_x, cfg.b, m, cfg.lr, seed=3, sparse_wire=True)
    la, lb = a.run(S), b.run(S)
    assert torch.equal(a.x_snap, b.x_snap) and la.bits_up == lb.bits_up and la.objectives == lb.objectives
    assert torch.equal(b.wire_nnz, b.nnz[m - 1])                       # entries of the last round's messages
    used = (host(b.wire_nnz).astype(np.int64) * (15 + cfg.b) + 31) // 32      # ceil(log2 20958) = 15 position bits
    w = words(b.wire)
    for r in range(cfg.M):
        assert not w[r, used[r]:].any() and (used[r] == 0 or w[r, :used[r]].any())


@pytest.mark.parametrize("d,M,B,b,nnz,l2,infinite,kernels", [
    (47236, 8, 32, 4, 60.0, 1e-4, False, 6), (36003, 5, 24, 8, 30.0, 1e-4, False, 6), (40001, 40, 9, 4, 30.0, 50.0, False, 6),
    (36001, 85, 3, 4, 30.0, 1e-4, False, 6), (36001, 130, 3, 4, 30.0, 1e-4, False, 5), (47233, 3, 16, 8, 30.0, 50.0, False, 6),
    (47236, 4, 32, 4, 30.0, 1e-4, True, 6), (47236, 8, 32, 2, 60.0, 1e-4, False, 5), (20958, 8, 32, 4, 30.0, 1e-4, False, 6)])
def test_messages_encoded_by_the_worker_step_equal_the_separate_encoder(dq, d, M, B, b, nnz, l2, infinite, kernels):
    """Models wider than the on-chip buffer, Alg. 2: the launch that quantizes also encodes (4 and 8 bits).  Streams are those of
    dq_sparse_encode on the messages, every word; messages and models those of a run without streams.  Eight slices a worker
    down to two, few entries and rows of which most is kept, ragged ends; an infinite feature: no entries; and what keeps the separate
    encoder: more workers than are split, 2 bits, a model that a block holds.  `kernels` of a round: worker, sparsifier, quantizer
    and encoder, decoder, update, the model's message; without the split the worker has the sparsifier and (130 workers, 2 bits)
    the quantizer, and the encoder is one of its own."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.sparse_text_logistic(400, d, mean_nnz=nnz, seed=8)
    if infinite:
        p.values[p.indptr[37]] = np.inf
    P = dq.DeviceProblem.from_host(p)
    P = dq.DeviceProblem(n=P.n, d=P.d, y=P.y, indptr=P.indptr, indices=P.indices, values=P.values, l2=l2, l1=1e-5)
    plain, wired = (DoubleQuantTrainer(P, "sparse", M, B, 8, b, 4, 0.01, seed=3, sparse_wire=w) for w in (False, True))
    for tr in (plain, wired):
        tr.epoch_prologue()
        tr.rounds(0, 2)                                    # (one-time function attributes are set outside a capture)
    assert launches(lambda: wired.rounds(1, 1)) == kernels
    seen = 0
    for tr in (plain, wired):
        tr.epoch_prologue()
    for t in range(4):
        wired.wire.fill_(-1)
        plain.rounds(t, 1); wired.rounds(t, 1)
        for name in ("packed", "delta", "x", "xq", "delta_x", "nnz", "status"):
            a, c = getattr(plain, name), getattr(wired, name)
            assert torch.equal(a.view(torch.int32), c.view(torch.int32)), (t, name)
        stream, count = torch.full_like(wired.wire, -1), torch.full_like(wired.wire_nnz, -1)
        dq.dq_sparse_encode(wired.packed, d, b, stream, count)
        assert torch.equal(stream, wired.wire) and torch.equal(count, wired.wire_nnz), t
        seen += int(count.sum())
    assert (seen == 0) == infinite


@pytest.mark.parametrize("name", ["C1", "C4", "C3", "C2"])
def test_rounds_replayed_from_a_captured_graph(dq, name):
    """dq_run_rounds only enqueues kernels (no allocation, no memset), so a caller may capture an epoch's rounds
    into a graph.  Every replay -- with eager work of the program between replays -- must give what the same
    rounds give when enqueued directly."""
    cfg, p, m = _small(name)
    m = min(m, 8)
    eager = _trainer(dq, p, cfg, m, seed=4)
    graph = _trainer(dq, p, cfg, m, seed=4)
    for tr in (eager, graph):
        tr.epoch_prologue()
        tr.rounds(0, m)                                  # warm-up: one-time function attributes are set outside the capture
    torch.cuda.synchronize()
    assert (launches(lambda: graph.rounds(0, m)) <= 3) == (name in ("C1", "C2")), "all rounds in one launch"
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            graph.rounds(0, m)
    torch.cuda.synchronize()
    scratch = torch.zeros(1 << 16, device="cuda")
    for rep in range(3):
        eager.rounds(0, m)
        g.replay()
        scratch.add_(1.0)                                # the program's own eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(eager.x, graph.x) and torch.equal(eager.packed, graph.packed), rep
        assert torch.equal(eager.delta, graph.delta) and torch.equal(eager.xq, graph.xq), rep
    assert np.isfinite(host(graph.x)).all()


@pytest.mark.parametrize("algo,b,M,each,b_x", [("asylpg", 8, 8, False, 8), ("asylpg", 2, 17, True, 6), ("acc", 8, 8, False, 8),
                                               ("asylpg", 8, 64, False, 8), ("acc", 4, 33, True, 4), ("sparse", 4, 5, False, 8), ("sparse", 8, 40, True, 8)])
@pytest.mark.parametrize("d,B,cache", [(4099, 24, True), (20958, 32, True), (36001, 24, True), (47236, 260, True),
                                       (20958, 32, False), (34400, 8, False), (34400, 32, False), (47236, 155, False)])
def test_worker_steps_split_over_the_columns_equal_the_separate_calls(dq, algo, b, M, each, b_x, d, B, cache):
    """CSR features: inside dq_run_rounds the blocks of a worker share the columns of the gradient and the master quantizes
    it, and wide models are split the same way in any call.  Messages, scales and iterates must be those of dq_vr_grad,
    dq_sparsify, dq_quantize_pack and the master step, one after the other, bit for bit.  (Ragged last quads, several
    LDS windows, more rows than one pass takes, 17, 33 and 40 workers: fewer slices each.  Without cached margins: batches
    on either side of what the workspace has room to prepare ahead, 650 entries at 34,400 columns and 4244 at 47,236, and
    no more than the step itself can stage, 4788 and 5151.)  Nothing is written past the workspace."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.sparse_text_logistic(600, d, mean_nnz=30.0, seed=3)
    P = dq.DeviceProblem.from_host(p)
    m, seed = 4, 9
    one = DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.5, seed=seed, each=each, cache_margins=cache)
    two = DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.5, seed=seed, each=each, cache_margins=cache)
    sentinel, size = 0x5A5A5A5A, one.ws.numel()
    roomy = torch.full((size + 16384,), sentinel, dtype=torch.int32, device="cuda")
    one.state.ws = roomy.data_ptr()                        # (of which the call is told the first `size` words)
    one.epoch_prologue(); two.epoch_prologue()
    one.rounds(0, 3)
    assert bool((roomy[size:] == sentinel).all())
    ld = (d + 3) // 4 * 4
    idx = torch.empty(M * B, dtype=torch.int32, device="cuda")
    alpha, beta = torch.zeros((M, ld), device="cuda")[:, :d], torch.zeros((M, ld), device="cuda")[:, :d]
    amax, kept = torch.zeros(M, device="cuda"), torch.zeros(M, dtype=torch.int32, device="cuda")
    acc = algo == "acc"
    for t in range(3):
        if t == 0:
            two.rounds(0, 1)                               # (the model is the snapshot: all-zero messages)
            continue
        dq.dq_sample_indices(P.n, M, B, seed, t, 0, idx)
        dq.dq_vr_grad(P, idx, M, B, two.xq, two.delta_x, b_x, False, two.x_snap, two.z_snap, alpha, amax, None, two.ws)
        if algo == "sparse":
            dq.dq_sparsify(alpha, None, seed, t, 0, beta, amax, kept)
            assert torch.equal(kept, one.nnz[t])
        dq.dq_quantize_pack(beta if algo == "sparse" else alpha, b, amax, True, seed, t, dq.TAG_GRAD, 0, two.packed, two.delta,
                            two.status)
        step = dq.dq_master_step_each if each else dq.dq_master_step
        args = (two.packed, two.delta, M, b) + (() if each else (float(np.float32(1) / np.float32(M)),))
        step(*args, two.g_snap, two.x, two.y if acc else None, two.x_snap, two.xsum if acc else None, two.eta, two.theta, P.l1,
             b_x, seed, t + 1, two.xq, two.delta_x, two.absmax_x[t & 1:], two.status)
    torch.cuda.synchronize()
    for name in ("packed", "delta", "x", "xq", "delta_x", "status") + (("y", "xsum") if acc else ()):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    assert host(one.x).any() and host(one.packed).any() and host(one.status)[0] == 0


@pytest.mark.parametrize("algo,b,M,B,b_x,each", [("asylpg", 8, 4, 16, 8, False), ("acc", 4, 3, 9, 6, False), ("asylpg", 2, 1, 1, 2, True),
                                                 ("acc", 8, 4, 16, 11, True), ("asylpg", 4, 2, 15, 16, False)])
@pytest.mark.parametrize("n,d", [(2000, 1000), (300, 54), (77, 1), (500, 1024), (400, 257), (600, 1021)])
def test_small_dense_rounds_in_one_launch_equal_the_separate_calls(dq, algo, b, M, B, b_x, each, n, d):
    """Up to four workers of sixteen rows and 1024 columns: dq_run_rounds runs all rounds of a call in one block.  Messages,
    scales, model, message of the model and largest magnitudes are those of dq_worker_step and the master step, round by
    round, bit for bit, however the rounds are cut into calls, in the first epoch and in a later one."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.dense_logistic(n, d, seed=2, l2=1e-2, l1=1e-5)
    lda = (d + 3) // 4 * 4 + 4
    X = np.full((n, lda), np.nan, dtype=np.float32)         # (padding that is not a number)
    X[:, :d] = p.dense
    P = dq.DeviceProblem(n=n, d=d, y=dev(p.y), l2=float(p.l2), l1=float(p.l1), dense=dev(X)[:, :d])
    m, seed = 6, 5
    x0 = torch.randn(d, device="cuda") * 0.3
    one = DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.5, seed=seed, each=each, x0=x0)
    two = DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.5, seed=seed, each=each, x0=x0)
    acc = algo == "acc"
    idx = torch.empty(M * B, dtype=torch.int32, device="cuda")
    for e in range(2):
        one.epoch_prologue(); two.epoch_prologue()
        one.rounds(0, 3); one.rounds(3, 1); one.rounds(4, 2)
        for t in range(m):
            it = e * m + t
            if t == 0 and two.is_flag_round(0):
                two.packed.zero_(); two.delta.zero_()
            else:
                if t == 0:
                    dq.dq_quantize_pack(two.x, b_x, two.absmax_x, False, seed, it, dq.TAG_MODEL, dq.MASTER_ID, two.xq, two.delta_x,
                                        two.status)
                dq.dq_sample_indices(n, M, B, seed, it, 0, idx)
                dq.dq_worker_step(P, idx, M, B, two.xq, two.delta_x, b_x, False, two.x_snap, two.z_snap, False, b, seed, it, 0,
                                  two.packed, two.delta, None, None, two.status, two.ws)
            step = dq.dq_master_step_each if each else dq.dq_master_step
            args = (two.packed, two.delta, M, b) + (() if each else (float(np.float32(1) / np.float32(M)),))
            step(*args, two.g_snap, two.x, two.y if acc else None, two.x_snap, two.xsum if acc else None, two.eta, two.theta,
                 P.l1, b_x, seed, it + 1, two.xq, two.delta_x, two.absmax_x[t & 1:], two.status)
        torch.cuda.synchronize()
        for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status") + (("y", "xsum") if acc else ()):
            assert torch.equal(getattr(one, name), getattr(two, name)), (e, name)
        one.epoch_epilogue(); two.epoch_epilogue()
    assert host(one.x).any() and host(one.status)[0] == 0


@pytest.mark.parametrize("B", [1, 5, 16])
def test_small_dense_rounds_with_an_infinite_feature(dq, B):
    """The scale of a gradient with an infinite coordinate is infinite, as in the separate worker step, not NaN: a row that is
    requested twice to fill up a batch is not added a second time."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    d = 100
    X = np.ones((1, d), dtype=np.float32)
    X[0, 7] = np.inf
    P = dq.DeviceProblem(n=1, d=d, y=-torch.ones(1, device="cuda"), l2=0.0, l1=0.0, dense=dev(X))
    one = DoubleQuantTrainer(P, "asylpg", 2, B, 8, 8, 4, 0.5, x0=torch.ones(d, device="cuda"))
    two = DoubleQuantTrainer(P, "asylpg", 2, B, 8, 8, 4, 0.5, x0=torch.ones(d, device="cuda"))
    for tr in (one, two):
        tr.z_snap.zero_()
        tr.x_snap.copy_(torch.linspace(0.1, 1.0, d))
        tr.delta_x.fill_(1.0 / 64)
        tr.xq.copy_(torch.full_like(tr.xq, 0x20202020))    # (every coordinate of the model: 32/64)
    one.rounds(1, 1)
    idx = torch.zeros(2 * B, dtype=torch.int32, device="cuda")
    dq.dq_worker_step(P, idx, 2, B, two.xq, two.delta_x, 8, False, two.x_snap, two.z_snap, False, 8, 0, 1, 0, two.packed, two.delta,
                      None, None, two.status, two.ws)
    assert host(two.delta).tolist() == [np.inf, np.inf] and host(one.delta).tolist() == [np.inf, np.inf]
    assert torch.equal(one.packed, two.packed) and host(one.status)[0] == 1 and host(two.status)[0] == 1


@pytest.mark.parametrize("d,b_x", [(4096, 8), (4097, 2), (8194, 4), (20959, 8), (32768, 2), (32771, 8)])
@pytest.mark.parametrize("algo,b,B", [("asylpg", 8, 1), ("acc", 4, 33), ("asylpg", 2, 150)])
def test_csr_rounds_of_one_call_equal_single_rounds(dq, d, b_x, algo, b, B):
    """CSR features: between the rounds of a call the model is quantized by the next round's worker kernel, from
    mini-batches prepared a round ahead (150 rows of 30 entries: more than a block keeps in its registers); in calls of a
    single round by the master, from rows read in the round.  Everything must be identical, ragged last quads and slices
    of up to 4096 columns included."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    P = dq.DeviceProblem.from_host(synth.sparse_text_logistic(500, d, mean_nnz=30.0, seed=4))
    one, many = (DoubleQuantTrainer(P, algo, 6, B, b_x, b, 5, 0.5, seed=3) for _ in range(2))
    one.epoch_prologue(); many.epoch_prologue()
    one.rounds(0, 5)
    for t in range(5):
        many.rounds(t, 1)
    torch.cuda.synchronize()
    for name in ("packed", "delta", "x", "xq", "delta_x", "status") + (("y", "xsum") if algo == "acc" else ()):
        assert torch.equal(getattr(one, name), getattr(many, name)), name
    assert host(one.x).any() and host(one.packed).any() and host(one.status)[0] == 0


def _many_rounds_and_few(dq, d, M, B, algo, b, b_x, each, nnz, entries, m=19):
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    P = dq.DeviceProblem.from_host(synth.sparse_text_logistic(500, d, mean_nnz=nnz, seed=4))
    if entries:
        P._s.lda = entries                                 # (what the problem says of its entries changes no result)
    return tuple(DoubleQuantTrainer(P, algo, M, B, b_x, b, m, 0.5, seed=3, each=each) for _ in range(2))


ONE_DIE = [
    (5, 1, 1, "asylpg", 8, 8, False, 2.0, 0), (257, 1, 9, "acc", 2, 2, True, 9.0, 0), (4097, 28, 24, "asylpg", 4, 3, True, 30.0, 0),
    (7170, 14, 70, "acc", 8, 16, False, 30.0, 0), (20959, 8, 33, "acc", 4, 12, True, 30.0, 0), (20958, 8, 128, "asylpg", 8, 8, False, 30.0, 0),
    (28415, 4, 25, "asylpg", 8, 4, False, 30.0, 0), (20958, 8, 64, "asylpg", 8, 8, False, 30.0, 500), (9001, 5, 128, "acc", 4, 8, False, 90.0, 500)]


def _joined(tr):
    """How many blocks the trainer's last one-launch rounds found on their die."""
    words = tr.M * ((tr.prob.d + 3) // 4 * 4) + tr.M * 16
    return int(tr.ws.view(torch.int32)[words + 1])


def _shared_rounds(dq, tr, t0, count, members):
    """The rounds of a call that takes one launch, as if no more than `members` of its blocks had found room on a die."""
    import ctypes as C
    from paper_1805_10111_amd import api
    f = api._lib.dq_test_run_rounds_shared
    f.argtypes = [C.c_void_p] * 3 + [C.c_int64] * 3 + [C.c_float] * 2 + [C.c_int32, C.c_void_p]
    assert f(tr.prob.ptr, C.byref(tr.cfg), C.byref(tr.state), tr.epoch_index, t0, count, tr.eta, tr.theta, members,
             torch.cuda.current_stream().cuda_stream) == 0


@pytest.mark.parametrize("d,M,B,algo,b,b_x,each,nnz,entries", ONE_DIE)
def test_csr_rounds_in_one_launch_equal_calls_of_a_few(dq, d, M, B, algo, b, b_x, each, nnz, entries):
    """CSR features: a call of eight rounds or more does them in one launch on one die, a shorter one with launches for each.
    Everything must be identical: one member and one slice a worker and several, ragged last quads and chunks, fields that straddle
    words, and, where the problem says rows of one entry, batches that are more than the members hold or a step stages."""
    many, few = _many_rounds_and_few(dq, d, M, B, algo, b, b_x, each, nnz, entries)
    for epoch in range(2):
        many.epoch_prologue(); few.epoch_prologue()
        for t, n in ((0, 11), (11, 8)):
            many.ws.view(torch.int32).fill_(-1)
            many.rounds(t, n)
            assert _joined(many) == {5: 1, 257: 2, 4097: 28, 7170: 29}.get(d, 32), "the route, and every member on it"
        for t, n in ((0, 5), (5, 5), (10, 1), (11, 5), (16, 3)):
            few.rounds(t, n)
        for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status") + (("y", "xsum") if algo == "acc" else ()):
            assert torch.equal(getattr(many, name), getattr(few, name)), (epoch, name)
        many.epoch_epilogue(); few.epoch_epilogue()
    assert host(many.x).any() and host(many.packed).any() and host(many.status)[0] == 0


@pytest.mark.parametrize("members", [1, 2, 7, 27])
@pytest.mark.parametrize("d,M,B,algo,b,b_x,each,nnz,entries", ONE_DIE)
def test_csr_rounds_by_fewer_members_equal_calls_of_a_few(dq, d, M, B, algo, b, b_x, each, nnz, entries, members):
    """The same where fewer blocks find room on a die than there are parts of the work: they share them, from one block that does all to
    a few short.  Everything must be identical again."""
    many, few = _many_rounds_and_few(dq, d, M, B, algo, b, b_x, each, nnz, entries)
    for epoch in range(2):
        many.epoch_prologue(); few.epoch_prologue()
        for t, n in ((0, 11), (11, 8)):
            many.ws.view(torch.int32).fill_(-1)
            _shared_rounds(dq, many, t, n, members)
            assert 1 <= _joined(many) <= members
        for t, n in ((0, 5), (5, 5), (10, 1), (11, 5), (16, 3)):
            few.rounds(t, n)
        for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status") + (("y", "xsum") if algo == "acc" else ()):
            assert torch.equal(getattr(many, name), getattr(few, name)), (epoch, name)
        many.epoch_epilogue(); few.epoch_epilogue()
    assert host(many.x).any() and host(many.packed).any() and host(many.status)[0] == 0


def _problem_of_rows(lens, d, seed=6):
    """CSR features with these numbers of entries in the rows."""
    rng = np.random.default_rng(seed)
    cols = np.concatenate([np.sort(rng.choice(d, k, replace=False)) for k in lens]).astype(np.int32)
    values = (rng.standard_normal(cols.size) / 8).astype(np.float32)
    return synth.Problem(n=len(lens), d=d, y=np.where(rng.random(len(lens)) < 0.5, -1.0, 1.0).astype(np.float32), l2=1e-3, l1=1e-6,
                         indptr=np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), indices=cols, values=values)


@pytest.mark.parametrize("members", [0, 1, 5])
@pytest.mark.parametrize("d,M,B,algo", [(20958, 8, 24, "asylpg"), (20958, 4, 1, "acc"), (9500, 3, 128, "asylpg"), (12000, 14, 9, "acc")])
def test_csr_rounds_of_uneven_rows_in_one_launch_equal_calls_of_a_few(dq, d, M, B, algo, members):
    """Mini-batches of more entries than the blocks hold are read in the round, in pieces of as many as there is room for: empty rows,
    rows around a wavefront's width, rows longer than a piece and than a group of rows, few entries beside very many."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    lens = [0, 9000, 1, 63, 64, 65, 0, 0, 5056, 127, 128, 129, 7680, 3000, 6400, 2, 0, 8192, 700, 9001, 40, 4999, 8200, 0]
    P = dq.DeviceProblem.from_host(_problem_of_rows(lens, d))
    P._s.lda = 30 * len(lens)                              # (the rows are said to be short: else such calls keep their launches)
    many, few = (DoubleQuantTrainer(P, algo, M, B, 8, 8, 12, 0.1, seed=3) for _ in range(2))
    many.epoch_prologue(); few.epoch_prologue()
    many.ws.view(torch.int32).fill_(-1)
    if members:
        _shared_rounds(dq, many, 0, 12, members)
    else:
        many.rounds(0, 12)
    assert 1 <= _joined(many) <= members if members else _joined(many) == 32
    for t, n in ((0, 5), (5, 5), (10, 2)):
        few.rounds(t, n)
    for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status") + (("y", "xsum") if algo == "acc" else ()):
        assert torch.equal(getattr(many, name), getattr(few, name)), name
    assert host(many.x).any() and host(many.packed).any() and host(many.status)[0] == 0


@pytest.mark.parametrize("members", [0, 3])
@pytest.mark.parametrize("algo,each", [("asylpg", False), ("asylpg", True), ("acc", False)])
@pytest.mark.parametrize("what", ["feature inf", "feature nan", "model", "margin", "long rows"])
def test_csr_rounds_in_one_launch_on_what_is_not_finite(dq, what, algo, each, members):
    """An infinity or NaN reaches the gradients (a feature of some rows, a cached margin; among more entries than the blocks hold) or comes
    with the model: status, scales, messages and models are those of the separate rounds, NaNs where theirs are."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    d, M, B = 9500, 6, 8
    long_rows = what == "long rows"
    p = _problem_of_rows([40, 0, 9000, 5000, 700, 64, 9, 8200], d) if long_rows else synth.sparse_text_logistic(400, d, mean_nnz=30.0, seed=4)
    if what.startswith("feature") or long_rows:
        p.values = p.values.copy()
        p.values[p.indptr[-2] if long_rows else slice(p.indptr[200], p.indptr[204])] = np.nan if "nan" in what else np.inf
    P = dq.DeviceProblem.from_host(p)
    if long_rows:
        P._s.lda = 30 * p.n
    many, few = (DoubleQuantTrainer(P, algo, M, B, 8, 8, 16, 0.1, seed=3, each=each) for _ in range(2))
    for tr in (many, few):
        tr.epoch_prologue()
        tr.z_snap.nan_to_num_(0.0, 0.0, 0.0); tr.g_snap.nan_to_num_(0.0, 0.0, 0.0)         # (the rounds' own business only)
        if what == "margin":
            tr.z_snap[200:230] = float("nan")
        tr.rounds(0, 3)
        if what == "model":
            tr.x[d - 1] = float("-inf")
            if algo == "acc":
                tr.y[d - 1] = float("-inf")
    many.ws.view(torch.int32).fill_(-1)
    if members:
        _shared_rounds(dq, many, 3, 11, members)
    else:
        many.rounds(3, 11)
    assert 1 <= _joined(many) <= members if members else _joined(many) == 32
    for t, n in ((3, 5), (8, 5), (13, 1)):
        few.rounds(t, n)
    for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status") + (("y", "xsum") if algo == "acc" else ()):
        a, b = getattr(many, name), getattr(few, name)
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num()), name
    assert host(many.status)[0] == 1


def test_csr_rounds_without_a_status_word_are_not_done_in_one_launch(dq):
    """The status word is how a caller learns that the blocks of such a launch gave up waiting for each other.  Without one each round has
    launches of its own, with the same results."""
    many, few = _many_rounds_and_few(dq, 4097, 8, 24, "asylpg", 8, 8, False, 30.0, 0)
    for tr in (many, few):
        tr.epoch_prologue()
        tr.rounds(0, 11)
    assert launches(lambda: many.rounds(0, 11)) <= 3
    few.state.status = None
    assert launches(lambda: few.rounds(0, 11)) >= 22
    many.rounds(11, 8); few.rounds(11, 8)
    for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x"):
        assert torch.equal(getattr(many, name), getattr(few, name)), name


def test_csr_rounds_on_part_of_the_compute_units_are_not_done_in_one_launch(dq):
    """A stream with a mask of compute units need not have a whole die.  Each round has launches of its own there, with the same results."""
    import ctypes as C
    from paper_1805_10111_amd import api
    many, few = _many_rounds_and_few(dq, 4097, 8, 24, "asylpg", 8, 8, False, 30.0, 0)
    handle, units = C.c_void_p(), torch.cuda.get_device_properties(0).multi_processor_count
    half = (C.c_uint32 * (units // 32))(*[0xFFFFFFFF] * (units // 64))
    assert api._lib.hipExtStreamCreateWithCUMask(C.byref(handle), len(half), half) == 0
    masked = torch.cuda.ExternalStream(handle.value)
    for tr in (many, few):
        tr.epoch_prologue()
        tr.rounds(0, 11)
    torch.cuda.synchronize()
    assert launches(lambda: many.rounds(0, 11)) <= 3
    assert launches(lambda: few.rounds(0, 11), masked) >= 22
    many.rounds(11, 8)
    with torch.cuda.stream(masked):
        few.rounds(11, 8)
    torch.cuda.synchronize()
    for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status"):
        assert torch.equal(getattr(many, name), getattr(few, name)), name
    assert api._lib.hipStreamDestroy(handle) == 0


@pytest.mark.parametrize("stream", [0, 1, 2])
def test_csr_rounds_on_the_default_streams(dq, stream):
    """The null stream, hipStreamLegacy and hipStreamPerThread by their handles: one launch, as on any stream without a mask."""
    import ctypes as C
    from paper_1805_10111_amd import api
    many, few = _many_rounds_and_few(dq, 4097, 8, 24, "asylpg", 8, 8, False, 30.0, 0)
    for tr in (many, few):
        tr.epoch_prologue()
        tr.rounds(0, 1)
    many.ws.view(torch.int32).fill_(-1)
    torch.cuda.synchronize()
    assert api._lib.dq_run_rounds(many.prob.ptr, C.byref(many.cfg), C.byref(many.state), C.c_int64(0), C.c_int64(1), C.c_int64(10),
                                  C.c_float(many.eta), C.c_float(many.theta), None, C.c_void_p(stream)) == 0
    torch.cuda.synchronize()
    assert _joined(many) == 32
    for t in (1, 6):
        few.rounds(t, 5)
    for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status"):
        assert torch.equal(getattr(many, name), getattr(few, name)), name


@pytest.mark.parametrize("members", [0, 3])
def test_csr_rounds_of_a_long_call_equal_calls_of_a_few(dq, members):
    """A call of more rounds than one launch does, the model kept between the launches as between calls; also by fewer members."""
    many, few = _many_rounds_and_few(dq, 700, 2, 6, "acc", 8, 8, False, 9.0, 0, m=1050)
    many.epoch_prologue(); few.epoch_prologue()
    if members:
        _shared_rounds(dq, many, 0, 1050, members)
    else:
        many.rounds(0, 1050)
    for t in range(0, 1050, 5):
        few.rounds(t, 5)
    for name in ("packed", "delta", "x", "xq", "delta_x", "absmax_x", "status", "y", "xsum"):
        assert torch.equal(getattr(many, name), getattr(few, name)), name
    assert host(many.x).any() and host(many.status)[0] == 0


def test_csr_rounds_in_one_launch_on_several_streams_at_once(dq):
    """Three threads, a stream each, call at the same time, beside products that want the whole part: each of their launches finds a
    die, or waits for one, and the results are those of the separate rounds."""
    import ctypes as C
    import threading
    from paper_1805_10111_amd import api
    pairs = [_many_rounds_and_few(dq, d, M, 32, "asylpg", 8, 8, False, 30.0, 0, m=40) for d, M in ((20958, 8), (7000, 14), (4097, 20))]
    streams = [torch.cuda.Stream() for _ in range(len(pairs) + 1)]
    for many, few in pairs:
        many.epoch_prologue(); few.epoch_prologue()
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()

    def call(tr, stream):
        with torch.cuda.stream(stream):
            for _ in range(5):
                tr.rounds(0, 40)

    threads = [threading.Thread(target=call, args=(many, s)) for (many, _), s in zip(pairs, streams)]
    with torch.cuda.stream(streams[-1]):
        for _ in range(10):
            b = a @ a
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    taken = np.full(16, 7, dtype=np.uint32)
    assert api._lib.dq_test_dies_taken(taken.ctypes.data_as(C.c_void_p)) == 0 and not taken.any(), "every launch gives its die back"
    for many, few in pairs:
        for _ in range(5):
            for t in range(0, 40, 5):
                few.rounds(t, 5)
        for name in ("packed", "delta", "x", "xq", "delta_x", "status"):
            assert torch.equal(getattr(many, name), getattr(few, name)), name
    assert bool(torch.isfinite(b).all())


@pytest.mark.parametrize("d,M,B", [(4097, 5, 24), (20958, 16, 33), (30211, 3, 150)])
@pytest.mark.parametrize("l2", [1e-4, 50.0])
def test_csr_sparsified_rounds_of_one_call_equal_single_rounds(dq, d, M, B, l2):
    """Alg. 2 on CSR features: between the rounds of a call a worker finds ||alpha||_inf among the columns that its rows touch
    (l2 = 1e-4), unless the others may exceed them (l2 = 50: the whole vector is looked at); in calls of a single round
    always from the whole vector.  Everything must be identical."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.sparse_text_logistic(500, d, mean_nnz=30.0, seed=5)
    P = dq.DeviceProblem.from_host(p)
    P = dq.DeviceProblem(n=P.n, d=P.d, y=P.y, indptr=P.indptr, indices=P.indices, values=P.values, l2=l2, l1=1e-5)
    one, many = (DoubleQuantTrainer(P, "sparse", M, B, 8, 4, 5, 0.01, seed=3) for _ in range(2))
    one.epoch_prologue(); many.epoch_prologue()
    one.rounds(0, 5)
    for t in range(5):
        many.rounds(t, 1)
    torch.cuda.synchronize()
    for name in ("packed", "delta", "nnz", "x", "xq", "delta_x", "status"):
        assert torch.equal(getattr(one, name), getattr(many, name)), name
    assert host(one.x).any() and host(one.packed).any() and host(one.status)[0] == 0


@pytest.mark.parametrize("algo,cached,d,M,B,nnz,least,most", [
    ("sparse", False, 8192, 8, 100, 30.0, 2049, 4096), ("sparse", False, 8192, 8, 200, 30.0, 4097, 7040),
    ("sparse", False, 20958, 8, 172, 18.0, 2049, 3848), ("sparse", False, 47236, 8, 100, 30.0, 2049, 4096),
    ("sparse", False, 47236, 4, 200, 18.0, 2049, 4244), ("sparse", True, 20958, 16, 80, 30.0, 1025, 4096),
    ("sparse", True, 20958, 3, 147, 30.0, 4097, 5130), ("sparse", True, 4097, 5, 160, 30.0, 4097, 8192),
    ("sparse", True, 4097, 5, 230, 30.0, 4097, 8192), ("asylpg", True, 2000, 6, 230, 30.0, 4097, 8192),
    ("asylpg", True, 20958, 32, 40, 30.0, 1025, 4096), ("acc", True, 3001, 4, 40, 9.0, 1, 1024), ("acc", True, 777, 3, 5, 9.0, 1, 64)])
def test_csr_rounds_from_prepared_batches_equal_single_rounds(dq, algo, cached, d, M, B, nnz, least, most):
    """CSR features, mini-batches prepared a round ahead: of `least` to `most` entries each, which is no more than a block stages at
    that width (up to 1024 entries the reading block forms their maximum, up to 4096 they stay in its registers).  In calls of a
    single round nothing is prepared.  Everything must be identical."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    p = synth.sparse_text_logistic(500, d, mean_nnz=nnz, seed=6)
    lengths = np.diff(p.indptr)
    for t in range(1, 5):
        for w in range(M):
            assert least <= lengths[oracle.sample_indices(500, B, 3, t, w)].sum() <= most
    P = dq.DeviceProblem.from_host(p)
    one, many = (DoubleQuantTrainer(P, algo, M, B, 8, 4, 5, 0.05, seed=3, cache_margins=cached) for _ in range(2))
    one.epoch_prologue(); many.epoch_prologue()
    one.rounds(0, 5)
    for t in range(5):
        many.rounds(t, 1)
    torch.cuda.synchronize()
    for name in ("packed", "delta", "x", "xq", "delta_x", "status") + (("nnz",) if algo == "sparse" else ()):
        assert torch.equal(getattr(one, name), getattr(many, name)), name
    assert host(one.x).any() and host(one.packed).any() and host(one.status)[0] == 0


@pytest.mark.parametrize("cached,d,M,B,read", [(True, 8192, 8, 32, True), (True, 20958, 16, 32, True), (False, 8192, 8, 32, False),
                                               (True, 47236, 8, 32, False), (True, 8192, 33, 32, False), (True, 4000, 8, 32, False),
                                               (True, 8192, 8, 200, False)])
def test_the_distance_from_the_snapshot_is_formed_only_where_the_next_step_reads_it(dq, cached, d, M, B, read):
    """Alg. 2 on CSR features: the master's ||x - x_snap||_inf beside the prepared mini-batches, a word of either set in the
    workspace (which ends with the two sets), is for steps with cached margins whose sparsifier is split over several blocks that
    hold all columns, and light mini-batches.  A step split over the columns, one without cached margins or one of a single block
    per worker has no use for it."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    P = dq.DeviceProblem.from_host(synth.sparse_text_logistic(500, d, mean_nnz=30.0, seed=7))
    tr = DoubleQuantTrainer(P, "sparse", M, B, 8, 4, 6, 0.05, seed=3, cache_margins=cached)
    tr.epoch_prologue()
    tr.ws.zero_()
    tr.rounds(0, 6)
    words, rows = host(tr.ws).view(np.int32), M * ((d + 3) // 4 * 4) + 16 * M
    words = words[:dq.dq_workspace_bytes(dq.OP_VR_GRAD, P, M, B) // 4]
    sets = words[rows + (d + 3) // 4 * 4:].reshape(2, M, -1)
    formed = sets[:, 0, 4 + 256 + 3].view(np.float32)
    assert (formed > 0).all() if read else not formed.any()


@pytest.mark.parametrize("d,M,B,entries", [(4200, 8, 128, None), (20958, 8, 150, None), (32000, 6, 48, None), (20958, 8, 60, 0), (20958, 8, 16, 1 << 40)])
def test_heavy_mini_batches_leave_the_model_to_a_launch_of_its_own(dq, d, M, B, entries):
    """CSR features, step split over the columns: with heavy mini-batches (or such as may be) the model message is the master's, which
    leaves (decoded model) - snapshot behind the rows and maxima in the workspace.  What the problem says of its entries changes no result."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    P = dq.DeviceProblem.from_host(synth.sparse_text_logistic(500, d, mean_nnz=60.0, seed=8))
    if entries is not None:
        P._s.lda = entries
    one, two, light = (DoubleQuantTrainer(P, "asylpg", M, B, 8, 8, 4, 0.5, seed=3) for _ in range(3))
    for tr in (one, two, light):
        tr.epoch_prologue()
    one.rounds(0, 2)
    two.rounds(0, 3)
    rows = M * ((d + 3) // 4 * 4) + 16 * M
    q = one.xq.view(torch.int8)[:d].float() * one.delta_x[:1] - one.x_snap
    assert torch.equal(two.ws[rows:rows + d], q) and bool(q.any())
    two.rounds(3, 1)
    P._s.lda = 500                                         # (rows of one entry: the worker kernel quantizes)
    light.rounds(0, 4)
    for name in ("packed", "delta", "x", "xq", "delta_x", "status"):
        assert torch.equal(getattr(two, name), getattr(light, name)), name


def test_csr_sparsified_rounds_with_a_model_whose_message_overflows(dq):
    """Alg. 2 on CSR features: a coordinate at the largest float32 comes back from its 8-bit message as infinity (127 times the rounded
    scale), although the model is as close to its snapshot as ever; it is in no row, so no touched column shows it.  The rounds of
    one call still equal single ones."""
    from paper_1805_10111_amd.driver import DoubleQuantTrainer
    d, top = 8192, np.finfo(np.float32).max
    p = synth.sparse_text_logistic(500, d - 1, mean_nnz=30.0, seed=9)
    P = dq.DeviceProblem.from_host(p)
    P = dq.DeviceProblem(n=P.n, d=d, y=P.y, indptr=P.indptr, indices=P.indices, values=P.values, l2=0.0, l1=0.0)
    x0 = torch.linspace(-0.5, 0.5, d, device="cuda")       # (all but the last coordinate come back as zero)
    x0[d - 1] = float(top)
    one, many = (DoubleQuantTrainer(P, "sparse", 8, 32, 8, 4, 4, 0.01, seed=3, x0=x0.clone()) for _ in range(2))
    one.epoch_prologue(); many.epoch_prologue()
    one.rounds(0, 4)
    for t in range(4):
        many.rounds(t, 1)
    torch.cuda.synchronize()
    for name in ("packed", "nnz", "xq", "status"):
        assert torch.equal(getattr(one, name), getattr(many, name)), name
    assert host(one.xq.view(torch.int8))[d - 1] == 127 and host(one.x)[d - 1] == top
    for name in ("delta", "x", "delta_x"):
        assert np.array_equal(host(getattr(one, name)), host(getattr(many, name)), equal_nan=True), name
