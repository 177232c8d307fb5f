"""GPU parity: the HIP library (through the C ABI) against the CPU oracle.

Graphs, weights and schedules on the oracle side come from the oracle's own
builders; the library's are only compared with them (bit for bit).  Both
sides start from the same seeded inputs and run independently (nothing the
GPU computes is fed to the oracle); models are compared after every round
within 1e-5 relative (floor: the row's rms) and the loss F(w_bar) reported by
the library's metrics within 1e-4 of the oracle's.
"""
import numpy as np
import pytest

from conftest import assert_models_close
from paper_1612_08608_amd import asap, synth
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    asap.lib()  # fail loudly if the HIP library is missing
    return _t


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu] {request.node.nodeid}", flush=True)
    yield


def graph(kind, n, d=0, seed=0):
    """Oracle graph + weights; asserts the library builds the same bytes."""
    if kind == "ring":
        p, i = oracle.graphs.ring(n)
        lp, li = asap.asap_graph_ring(n)
    elif kind == "complete":
        p, i = oracle.graphs.complete(n)
        lp, li = asap.asap_graph_complete(n)
    elif kind == "root":
        p, i = oracle.graphs.root_expander(n)
        lp, li = asap.asap_graph_root_expander(n)
    elif kind == "chain":
        p, i = oracle.graphs.chain(n)
        lp, li = asap.asap_graph_chain(n)
    else:
        p, i = oracle.graphs.random_regular(n, d, seed)
        lp, li = asap.asap_graph_random_regular(n, d, seed)
    w = oracle.graphs.metropolis_weights(p, i)
    assert np.array_equal(lp, p) and np.array_equal(li, i)
    assert np.array_equal(asap.asap_metropolis_weights(lp, li).view(np.uint32), w.view(np.uint32))
    return p, i, w


def f32(x):
    return float(np.float32(x))


def params(wl, local_steps=0):
    return asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, wl.batch, wl.seed, local_steps)


def oracle_kw(wl):
    return dict(batch=wl.batch, loss=wl.loss, lr_kind=wl.lr_kind, lr0=f32(wl.lr0), l2=f32(wl.l2))


def csr_shards(wl, rp, col, val, y):
    S = wl.samples
    out = []
    for k in range(wl.n_workers):
        lo = rp[k * S]
        out.append(("csr", rp[k * S:(k + 1) * S + 1] - lo, col[lo:rp[(k + 1) * S]],
                    val[lo:rp[(k + 1) * S]], y[k * S:(k + 1) * S]))
    return out


def mean_loss(W, shards, loss, l2):
    return oracle.metrics.mean_objective(oracle.metrics.mean_model(W), shards, loss, l2)


def ambiguity_mask(amb, shards, p, i, shape):
    """Entries an fp32 hinge decision within rounding of the kink may change:
    the columns of each such row (worker k, row q) in every worker that reads
    k's half-step in the reduce."""
    mask = np.zeros(shape, bool)
    for k, q in amb:
        _, rpk, ck, _, _ = shards[k]
        readers = [j for j in range(shape[0]) if k in i[p[j]:p[j + 1]]]
        mask[np.ix_(readers, ck[rpk[q]:rpk[q + 1]])] = True
    return mask


# ----------------------------------------------------------------------------
# schedule
# ----------------------------------------------------------------------------
@pytest.mark.parametrize("n,S,rnd", [(64, 20480, 3), (4, 1, 0), (4, 2, 5), (8, 1000, 17), (32, 65536, 29)])
def test_schedule_device_matches_oracle(torch, n, S, rnd):
    p, i, w = graph("ring", max(n, 3))
    n = max(n, 3)
    sess = asap.Session(n, 64, p, i, w)
    rp = np.arange(n * S + 1, dtype=np.int64)
    sess.bind_csr(rp, np.zeros(n * S, np.int32), np.ones(n * S, np.float32), np.ones(n * S, np.float32), S)
    sess.ready()
    out = torch.empty(n * S, dtype=torch.int32, device="cuda")
    asap.asap_schedule_device(sess.ctx, 0, rnd, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(n, S)
    for k in range(n):
        assert np.array_equal(got[k], oracle.prng.schedule(S, 0, k, rnd)), k
    sess.close()


# ----------------------------------------------------------------------------
# free-running rounds: both sides start from the same seeded models and run
# independently; models are compared after every round
# ----------------------------------------------------------------------------
def _free_run(torch, wl, kind, d, rounds, W0=None, loss_curve=False, local_steps=0, data=None, gr=None, members=0):
    """`rounds` rounds on the GPU and in the oracle from the same seeded start,
    compared after every round.  `data` (CSR arrays) and `gr` (graph) replace
    the workload's own; `members` sets the workgroups per worker of the
    planned CSR pass (0: the library's choice).  A round in which the oracle finds hinge decisions
    within rounding of the kink is compared outside the entries they can
    change (`ambiguity_mask`), and the comparison ends there: from then on
    the two runs may legitimately differ.  Round 0 is always compared."""
    p, i, w = graph(kind, wl.n_workers, d) if gr is None else gr
    if wl.features == "dense":
        X, y = synth.dense_data(wl)
        shards = [("dense", X[k], y[k]) for k in range(wl.n_workers)]
    else:
        rp, col, val, yy = synth.csr_data(wl) if data is None else data
        shards = csr_shards(wl, rp, col, val, yy)
    sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
    W = np.zeros((wl.n_workers, wl.dim)) if W0 is None else W0.astype(np.float64)
    if W0 is not None:
        sess.set_models(W0)
    if wl.features == "dense":
        sess.bind_dense(X, y)
    else:
        sess.bind_csr(rp, col, val, yy, wl.samples)
        if members:
            sess.set_csr_members(members)
    prm = params(wl, local_steps)
    K = oracle.sgd.n_steps(wl.samples, wl.batch)
    for r in range(rounds):
        if r % 2:
            sess.prepare_sgd(prm)  # optional; asap_local_sgd prepares by itself on even rounds
        sess.round(prm)
        got = sess.models().cpu().numpy()
        amb = []
        halves = []
        q, k0, k1 = oracle.sgd.round_steps(r, local_steps, K)
        for k in range(wl.n_workers):
            sched = oracle.prng.schedule(wl.samples, wl.seed, k, q)
            if shards[k][0] == "dense":
                halves.append(oracle.sgd.sgd_pass_dense(W[k], shards[k][1], shards[k][2], sched, rnd=q,
                                                        steps=(k0, k1), **oracle_kw(wl)))
            else:
                a = []
                _, rpk, ck, vk, yk = shards[k]
                halves.append(oracle.sgd.sgd_pass_csr(W[k], rpk, ck, vk, yk, sched, rnd=q, ambiguous=a,
                                                      steps=(k0, k1), **oracle_kw(wl)))
                amb += [(k, qq) for qq in a]
        W = oracle.mix.stochastic_reduce(np.stack(halves), p, i, w)
        if amb:
            mask = ambiguity_mask(amb, shards, p, i, W.shape)
            assert mask.mean() < 0.5, "too few entries left to compare"
            assert_models_close(got, W, what=f"round {r}", mask=mask)
            print(f"round {r}: {len(amb)} ambiguous hinge rows, comparison stops", flush=True)
            break
        assert_models_close(got, W, what=f"round {r}")
        if loss_curve:
            m = sess.metrics(wl.loss, f32(wl.l2))
            assert abs(m[1] - mean_loss(W, shards, wl.loss, f32(wl.l2))) <= 1e-4, r
    assert sess.check()[0] == asap.OK
    sess.close()
    return W, shards


def test_ring8_dense_full_workload_every_round_and_loss_curve(torch):
    wl = synth.RING8_DENSE_LR
    W, shards = _free_run(torch, wl, "ring", 2, wl.rounds, loss_curve=True)
    assert mean_loss(W, shards, wl.loss, wl.l2) < 0.6 * np.log(2)   # it learns


@pytest.mark.parametrize("n,dim,S,B,l2", [(4, 100, 50, 7, 0.0), (3, 1000, 64, 64, 0.01), (5, 4096, 300, 256, 0.0),
                                         (3, 16384, 20, 3, 0.0), (4, 5, 9, 2, 0.1),
                                         (1, 1, 3, 1, 0.0), (2, 3, 1, 1, 0.05)])  # one worker, one feature; one sample
def test_dense_shapes(torch, n, dim, S, B, l2):
    wl = synth.DENSE_LR_32W.with_(n_workers=n, dim=dim, samples=S, batch=B, l2=l2, lr_kind="inv_sqrt", lr0=0.3)
    W0 = synth.initial_models(wl.with_(seed=3)) * np.float32(0.01)
    _free_run(torch, wl, "complete", 0, 3, W0=W0)


# wide dense models: a worker's workgroups own columns and exchange the
# minibatch's partial margins
@pytest.mark.parametrize("n,dim,S,B,l2,loss", [
    (3, 1025, 40, 5, 0.0, "logistic"),    # five units, the last of one column
    (2, 2048, 33, 8, 0.05, "logistic"),   # ragged last minibatch, L2
    (6, 3001, 100, 16, 0.0, "hinge"),     # twelve units, ragged, hinge
    (2, 8192, 24, 3, 0.0, "logistic"),    # 32 units, fewer rows a step than row waves
    (300, 1500, 16, 4, 0.0, "logistic"),  # more workers than compute units: one workgroup each
])
def test_dense_wide_kernel_shapes(torch, n, dim, S, B, l2, loss):
    wl = synth.DENSE_LR_32W.with_(n_workers=n, dim=dim, samples=S, batch=B, l2=l2, loss=loss,
                                  lr_kind="inv_sqrt", lr0=0.3)
    W0 = synth.initial_models(wl.with_(seed=5)) * np.float32(0.01)
    _free_run(torch, wl, "complete" if n > 8 else "ring" if n >= 3 else "complete", 2, 3, W0=W0)


def test_dense_wide_run_twice_is_bitwise_identical(torch):
    wl = synth.DENSE_LR_32W.with_(n_workers=4, samples=96, batch=32)
    p, i, w = graph("ring", 4)
    X, y = synth.dense_data(wl)
    out = []
    for _ in range(2):
        sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
        sess.bind_dense(X, y)
        for _ in range(2):
            sess.round(params(wl))
        out.append(sess.models().cpu().numpy().copy())
        sess.close()
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))


def test_dense_32w_launch_shape_reduced_samples(torch):
    # the 32-worker dense workload's launch shape (D = 4096, B = 256, 6-regular)
    # with 2048 samples per worker instead of 65536
    wl = synth.DENSE_LR_32W.with_(samples=2048)
    _free_run(torch, wl, "random", wl.degree, 2, loss_curve=True)


def test_csr_logistic_ragged_batches(torch):
    # S = 1000 = 15 * 64 + 40: a ragged last minibatch every round
    wl = synth.SPARSE_LR_64W.with_(n_workers=16, dim=1 << 14, samples=1000)
    _free_run(torch, wl, "random", 4, 4, loss_curve=True)


def test_csr_hinge_l2_scale_form(torch):
    wl = synth.SPARSE_SVM_256W.with_(n_workers=32, dim=1 << 12, samples=700, l2=1e-3)
    _free_run(torch, wl, "random", 8, 4, loss_curve=True)


# The planned CSR pass with 1, 2 and 4 workgroups per worker: member m owns
# the columns c mod members == m, and the members exchange their partial
# margins once per step (Appendix A, update (A.2), first line).
@pytest.mark.parametrize("members", [1, 2, 4])
@pytest.mark.parametrize("case", ["logistic_ragged", "hinge_l2"])
def test_csr_members_against_the_oracle(torch, case, members):
    if case == "logistic_ragged":
        wl = synth.SPARSE_LR_64W.with_(n_workers=16, dim=1 << 14, samples=1000)  # 15 steps of 64 + one of 40
        _free_run(torch, wl, "random", 4, 3, loss_curve=True, members=members)
    else:
        wl = synth.SPARSE_SVM_256W.with_(n_workers=16, dim=1 << 12, samples=700, l2=1e-3)
        _free_run(torch, wl, "random", 8, 3, loss_curve=True, members=members)


def test_csr_long_steps_with_many_cold_columns(torch):
    # one workgroup per worker over 64-row steps of Poisson(80) rows on 2^20
    # columns: up to 64 x 114 nonzeros and about 1400 distinct cold columns
    # per step, so planning takes 512-thread blocks and tables of 2^12
    # positions, and links hold whole lists
    wl = synth.SPARSE_LR_64W.with_(n_workers=8, samples=2048)
    _free_run(torch, wl, "random", 4, 3, loss_curve=True, members=1)


def test_csr_small_batch_pass_on_a_full_device(torch):
    # 160 workers with minibatches of 32 rows fill the device: the planned
    # pass runs 512-thread workgroups (32 rows of 16 lanes), so that the next
    # round's planning fits beside them
    wl = synth.SPARSE_SVM_256W.with_(n_workers=160, dim=1 << 12, samples=200, l2=1e-3)
    _free_run(torch, wl, "random", 8, 3, loss_curve=True)


def test_csr_members_on_several_xcds(torch):
    # 12 workers (not a multiple of the 8 XCDs): a worker's members are
    # consecutive workgroups, which land on different XCDs, so they exchange
    # their partial margins with device-scope stores
    wl = synth.SPARSE_LR_64W.with_(n_workers=12, dim=1 << 13, samples=640)
    _free_run(torch, wl, "random", 4, 3, loss_curve=True, members=2)


@pytest.mark.parametrize("members", [1, 4])
def test_csr_l2_scale_fold(torch, members):
    # strong L2 with a constant step: the pass's scale s = prod (1 - eta l2)
    # drops below 1e-6 after 48 steps of a pass and is folded back into the model (each
    # member folds its own columns)
    wl = synth.SPARSE_SVM_256W.with_(n_workers=8, dim=1 << 12, samples=704, batch=8, l2=0.5, lr_kind="const",
                                   lr0=0.5)  # 88 steps per pass
    W0 = synth.initial_models(wl.with_(seed=5))
    _free_run(torch, wl, "random", 4, 3, W0=W0, members=members)


def test_csr_hinge_complete_graph(torch):
    wl = synth.SPARSE_SVM_256W.with_(n_workers=16, dim=1 << 12, samples=512)
    _free_run(torch, wl, "complete", 0, 3, loss_curve=True)


def test_csr_many_distinct_cold_columns_fall_back(torch):
    # 64 rows of ~110 nearly uniform columns of 2^20: a step holds more
    # distinct rarely used columns than the planned pass keeps on chip, so
    # the round runs on the general kernel
    wl = synth.SPARSE_LR_64W.with_(n_workers=4, samples=256, nnz_mean=110.0, zipf_s=0.3)
    _free_run(torch, wl, "ring", 2, 2, loss_curve=True)


def test_csr_long_rows_and_large_batch_general_path(torch):
    # rows of ~200 nonzeros (> 128) and minibatches of 100 and 300 rows (> 64):
    # every step goes through the chunked general path
    for B in (100, 300):
        wl = synth.SPARSE_LR_64W.with_(n_workers=4, dim=1 << 13, samples=650, batch=B, nnz_mean=200.0,
                                       zipf_s=0.9)
        W0 = synth.initial_models(wl.with_(seed=9)) * np.float32(0.01)
        _free_run(torch, wl, "complete", 0, 2, W0=W0)


@pytest.mark.parametrize("kind", ["root", "chain"])
def test_csr_logistic_on_directed_graphs(torch, kind):
    wl = synth.SPARSE_LR_64W.with_(n_workers=16, dim=1 << 13, samples=200)
    _free_run(torch, wl, kind, 0, 4)


# (A.2) as printed is one gradient step per mix (local_steps = 1); blocks of
# L steps walk through the passes one after the other
@pytest.mark.parametrize("case,L", [("dense", 1), ("dense", 4), ("wide", 1), ("wide", 3), ("csr", 1), ("csr", 4),
                                    ("csr_general", 2), ("svm", 2)])
def test_local_steps(torch, case, L):
    if case == "dense":
        wl = synth.RING8_DENSE_LR.with_(samples=128, batch=16)          # K = 8
        kind, d = "ring", 2
    elif case == "wide":
        wl = synth.DENSE_LR_32W.with_(n_workers=3, dim=2048, samples=72, batch=8, lr_kind="inv_sqrt", lr0=0.2)  # K = 9
        kind, d = "complete", 0
    elif case == "csr":
        wl = synth.SPARSE_LR_64W.with_(n_workers=8, dim=1 << 13, samples=256, batch=32)  # K = 8, planned pass
        kind, d = "random", 4
    elif case == "csr_general":
        wl = synth.SPARSE_LR_64W.with_(n_workers=4, dim=1 << 12, samples=96, batch=96 // 4, nnz_mean=200.0)  # long rows
        kind, d = "ring", 2
    else:
        wl = synth.SPARSE_SVM_256W.with_(n_workers=8, dim=1 << 12, samples=128, batch=16)  # K = 8, hinge + L2
        kind, d = "random", 4
    K = -(-wl.samples // wl.batch)
    _free_run(torch, wl, kind, d, 2 * K // L + 1, local_steps=L)


def test_local_steps_must_divide_the_pass(torch):
    wl = synth.RING8_DENSE_LR.with_(samples=128, batch=16)  # K = 8
    p, i, w = graph("ring", wl.n_workers, 2)
    X, y = synth.dense_data(wl)
    sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
    sess.bind_dense(X, y)
    for L in (3, -1, 16):
        with pytest.raises(asap.AsapError) as e:
            sess.local_sgd(params(wl, L))
        assert e.value.status == asap.E_INVALID_ARG
    sess.local_sgd(params(wl, 8))  # a whole pass in one round is allowed
    sess.close()


def test_csr_single_sample_and_full_batch(torch):
    for S, B in ((1, 1), (37, 37), (37, 1)):
        wl = synth.SPARSE_LR_64W.with_(n_workers=3, dim=300, samples=S, batch=B, nnz_mean=10.0)
        _free_run(torch, wl, "ring", 2, 2)


@pytest.mark.parametrize("features", ["csr", "dense"])
def test_checkpoint_resume_is_bitwise_identical(torch, tmp_path, features):
    if features == "csr":
        wl = synth.SPARSE_LR_64W.with_(n_workers=8, dim=1 << 13, samples=256)
        data = synth.csr_data(wl)
    else:
        wl = synth.DENSE_LR_32W.with_(n_workers=4, dim=2048, samples=64, batch=16)
        data = synth.dense_data(wl)
    p, i, w = graph("random", wl.n_workers, 2 if wl.n_workers == 4 else 4)

    def session():
        sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
        if features == "csr":
            sess.bind_csr(*data, wl.samples)
        else:
            sess.bind_dense(*data)
        return sess

    prm = params(wl)
    a = session()
    for _ in range(3):
        a.round(prm)
    ck = tmp_path / "ck.npz"
    a.save(ck)
    for _ in range(2):
        a.round(prm)
    want = a.models().cpu().numpy().copy()
    assert a.current()[1] == 5
    a.close()
    b = session()
    b.load(ck)
    assert b.current() == (0, 3, 0)
    for _ in range(2):
        b.round(prm)
    assert b.current()[1] == 5
    assert np.array_equal(b.models().cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert b.check()[0] == asap.OK
    b.close()


def test_csr_run_twice_is_bitwise_identical(torch):
    wl = synth.SPARSE_LR_64W.with_(n_workers=8, dim=1 << 14, samples=640)
    outs = []
    for _ in range(2):
        p, i, w = graph("random", 8, 4)
        rp, col, val, y = synth.csr_data(wl)
        sess = asap.Session(8, wl.dim, p, i, w)
        sess.bind_csr(rp, col, val, y, wl.samples)
        for r in range(3):
            sess.round(params(wl))
        outs.append(sess.models().cpu().numpy().copy())
        sess.close()
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))


def test_csr_plan_ahead_follows_changing_params(torch):
    """The next round is planned while one runs; a call whose batch or seed
    differs from the planned one must not use that plan."""
    wl = synth.SPARSE_LR_64W.with_(n_workers=8, dim=1 << 14, samples=300)
    p, i, w = graph("random", 8, 4)
    rp, col, val, yy = synth.csr_data(wl)
    shards = csr_shards(wl, rp, col, val, yy)
    sess = asap.Session(8, wl.dim, p, i, w)
    sess.bind_csr(rp, col, val, yy, wl.samples)
    W = np.zeros((8, wl.dim))
    # (batch, seed, what asap_prepare_sgd is called with first) per round:
    # look-ahead hit, batch change, seed change, prepared with the same
    # parameters, prepared with other ones (ignored), hit
    plan = [(64, 0, None), (64, 0, None), (37, 0, None), (37, 5, (37, 5)), (37, 5, (64, 1)), (37, 5, None)]
    for r, (B, seed, prep) in enumerate(plan):
        prm = asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, B, seed)
        if prep is not None:
            sess.prepare_sgd(asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, prep[0], prep[1]))
        sess.round(prm)
        got = sess.models().cpu().numpy()
        kw = dict(oracle_kw(wl), batch=B)
        halves = []
        for k in range(8):
            _, rpk, ck, vk, yk = shards[k]
            sched = oracle.prng.schedule(wl.samples, seed, k, r)
            halves.append(oracle.sgd.sgd_pass_csr(W[k], rpk, ck, vk, yk, sched, rnd=r, **kw))
        W = oracle.mix.stochastic_reduce(np.stack(halves), p, i, w)
        assert_models_close(got, W, what=f"round {r} (batch {B}, seed {seed})")
    assert sess.check()[0] == asap.OK
    sess.close()


def _cone_round0(wl, shards, p, i, w, rows):
    """Oracle round 0 from zero models for the listed output rows only.

    Returns (expected rows, mask) where mask marks the columns of hinge rows
    whose fp64 decision sits within rounding of the kink (both sides decide
    in fp64, but their models differ by fp32 rounding).
    """
    need = sorted({int(j) for r in rows for j in i[p[r]:p[r + 1]]})
    half = {}
    amb = []
    for k in need:
        _, rpk, ck, vk, yk = shards[k]
        a = []
        half[k] = oracle.sgd.sgd_pass_csr(np.zeros(wl.dim), rpk, ck, vk, yk,
                                          oracle.prng.schedule(wl.samples, wl.seed, k, 0), rnd=0,
                                          ambiguous=a, **oracle_kw(wl))
        amb += [(k, q) for q in a]
    mask = np.zeros((len(rows), wl.dim), bool)
    for k, q in amb:
        _, rpk, ck, _, _ = shards[k]
        for n_, r in enumerate(rows):
            if k in i[p[r]:p[r + 1]]:
                mask[n_, ck[rpk[q]:rpk[q + 1]]] = True
    if amb:
        print(f"{len(amb)} ambiguous hinge rows masked ({int(mask.sum())} entries)", flush=True)
    return oracle.mix.stochastic_reduce_rows(lambda j: half[j], p, i, w, rows), mask


def test_csr_full_size_sparse_lr_sampled_rows(torch):
    # 64 workers, D = 2^20, 20480 samples each, minibatch 64, 4-regular:
    # round 0 on the GPU; the oracle computes the sampled rows' dependency cone
    wl = synth.SPARSE_LR_64W
    p, i, w = graph("random", wl.n_workers, wl.degree)
    rp, col, val, y = synth.csr_data(wl)
    shards = csr_shards(wl, rp, col, val, y)
    sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
    sess.bind_csr(rp, col, val, y, wl.samples)
    sess.round(params(wl))
    rows = [0, 37, 63]
    got = sess.models()[rows].cpu().numpy()
    assert sess.check()[0] == asap.OK
    sess.close()
    ref, mask = _cone_round0(wl, shards, p, i, w, rows)
    assert mask.sum() < 0.01 * mask.size
    assert_models_close(got, ref, what="round 0 sampled rows", mask=mask)


def test_csr_full_size_svm_sampled_rows(torch):
    wl = synth.SPARSE_SVM_256W
    p, i, w = graph("random", wl.n_workers, wl.degree)
    rp, col, val, y = synth.csr_data(wl)
    shards = csr_shards(wl, rp, col, val, y)
    sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
    sess.bind_csr(rp, col, val, y, wl.samples)
    sess.round(params(wl))
    rows = [0, 200]
    got = sess.models()[rows].cpu().numpy()
    assert sess.check()[0] == asap.OK
    sess.close()
    ref, mask = _cone_round0(wl, shards, p, i, w, rows)
    assert mask.sum() < 0.01 * mask.size
    assert_models_close(got, ref, what="round 0 sampled rows", mask=mask)


def test_csr_full_size_svm_complete_graph_half_steps(torch):
    # complete graph at full size: half-steps of sampled workers (scale form
    # folded by a reduce over the identity would be needed to read them, so
    # check the reduce separately: every reduced row is the same vector)
    wl = synth.SPARSE_SVM_256W
    p, i, w = graph("complete", wl.n_workers)
    rp, col, val, y = synth.csr_data(wl)
    sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
    sess.bind_csr(rp, col, val, y, wl.samples)
    sess.round(params(wl))
    got = sess.models().cpu().numpy()
    assert np.array_equal(got[0].view(np.uint32), got[-1].view(np.uint32))
    assert np.all(got.view(np.uint32) == got[0].view(np.uint32)[None, :])
    assert sess.check()[0] == asap.OK
    sess.close()


# ----------------------------------------------------------------------------
# stochastic reduce
# ----------------------------------------------------------------------------
@pytest.mark.parametrize("d", [2, 4, 8, 16])
def test_reduce_matches_oracle_ragged_dim(torch, d):
    wl = synth.MIX_STRESS_1024W.with_(dim=1001)
    p, i, w = graph("random", wl.n_workers, d)
    W = synth.initial_models(wl)
    sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
    sess.set_models(W)
    ref = W.astype(np.float64)
    for r in range(3):
        sess.stochastic_reduce()
        ref = oracle.mix.stochastic_reduce(ref, p, i, w)
        assert_models_close(sess.models().cpu().numpy(), ref, what=f"reduce {r}")
    assert sess.current() == (1, 3, 0)
    assert sess.check()[0] == asap.OK
    sess.close()


def irregular_graph(kind, n):
    """A graph with unequal degrees, built here; weights from both builders."""
    if kind == "path":      # the chain of Figure 2: end points have degree 1
        adj = [{j for j in (i - 1, i + 1) if 0 <= j < n} for i in range(n)]
    elif kind == "star":    # parameter-server shape: the hub has degree n-1
        adj = [set(range(1, n))] + [{0} for _ in range(1, n)]
    else:                   # ring plus chords from every third node
        adj = [{(i - 1) % n, (i + 1) % n} for i in range(n)]
        for i in range(0, n, 3):
            j = (i + n // 2 + 1) % n
            adj[i].add(j)
            adj[j].add(i)
    ptr = np.zeros(n + 1, np.int32)
    idx = []
    for i in range(n):
        row = sorted(adj[i] | {i})
        idx.extend(row)
        ptr[i + 1] = ptr[i] + len(row)
    idx = np.asarray(idx, np.int32)
    w = oracle.graphs.metropolis_weights(ptr, idx)
    assert np.array_equal(asap.asap_metropolis_weights(ptr, idx).view(np.uint32), w.view(np.uint32))
    return ptr, idx, w


# (workers, graph, degree, dim): powers of two up to 1024 with rows of at most
# 17 entries take the LDS-slab kernel (chunks of 2^15 or 2^14 floats split
# over the rows), the rest the tile kernel; dims cover one partial float4,
# exact chunk multiples, ragged tails and fewer chunks than compute units.
REDUCE_SHAPES = [
    (8, "ring", 2, 1), (8, "ring", 2, 4097), (8, "ring", 2, 3 * 4096),
    (16, "random", 6, 64), (32, "ring", 2, 33), (64, "random", 4, 3 * 512),
    (64, "random", 4, 515), (256, "random", 8, 130), (1024, "random", 16, 130),
    (1024, "random", 2, 67), (16, "path", 0, 1003), (128, "chords", 0, 999),
    (100, "random", 4, 777), (64, "random", 20, 1001), (64, "star", 0, 300),
    (3, "ring", 2, 5),
    # Figure 2's directed topologies (P not symmetric): root expander and chain
    (64, "root", 0, 1029), (25, "root", 0, 517), (1024, "root", 0, 70), (6, "chain", 0, 301),
    (1024, "chain", 0, 66),
]


@pytest.mark.parametrize("n,kind,d,dim", REDUCE_SHAPES)
def test_reduce_kernel_shapes(torch, n, kind, d, dim):
    if kind in ("path", "star", "chords"):
        p, i, w = irregular_graph(kind, n)
    else:
        p, i, w = graph(kind, n, d)
    W = synth.initial_models(synth.MIX_STRESS_1024W.with_(n_workers=n, dim=dim))
    sess = asap.Session(n, dim, p, i, w)
    sess.set_models(W)
    ref = W.astype(np.float64)
    for r in range(2):
        sess.stochastic_reduce()
        ref = oracle.mix.stochastic_reduce(ref, p, i, w)
        assert_models_close(sess.models().cpu().numpy(), ref, what=f"{kind} n={n} dim={dim} reduce {r}")
    assert sess.check()[0] == asap.OK
    sess.close()


def test_complete_graph_reduce_is_column_mean(torch):
    n, dim = 256, 3000
    p, i, w = graph("complete", n)
    W = synth.initial_models(synth.MIX_STRESS_1024W.with_(n_workers=n, dim=dim))
    sess = asap.Session(n, dim, p, i, w)
    sess.set_models(W)
    sess.stochastic_reduce()
    got = sess.models().cpu().numpy()
    assert_models_close(got, oracle.mix.stochastic_reduce(W, p, i, w), what="complete")
    assert np.allclose(got, W.astype(np.float64).mean(axis=0), rtol=0, atol=1e-6)
    sess.close()


def test_reduce_stress_full_size_sampled_columns(torch):
    # 1024 workers x 2^20 floats, 100 rounds per degree d in {2, 4, 8, 16}.
    # Columns mix independently, so the oracle runs the same 100 rounds on a
    # column sample of the seeded start; the GPU's sample must follow it, keep
    # the column means, and lose its deviation from consensus at least as fast
    # as sigma_2(P)^t.
    wl = synth.MIX_STRESS_1024W
    W0 = synth.initial_models(wl)
    rng = np.random.default_rng(0)
    cols = np.unique(np.concatenate([rng.choice(wl.dim, 2048, replace=False), [0, wl.dim - 1]]))
    cols_t = torch.as_tensor(cols, device="cuda")
    S0 = W0[:, cols].astype(np.float64)
    mean0 = S0.mean(axis=0)
    dev0 = float(np.linalg.norm(S0 - mean0))
    for d in (2, 4, 8, 16):
        p, i, w = graph("random", wl.n_workers, d)
        s2 = oracle.graphs.sigma2(oracle.graphs.dense_matrix(p, i, w))
        sess = asap.Session(wl.n_workers, wl.dim, p, i, w)
        sess.set_models(W0)
        ref = S0
        for t in range(1, wl.rounds + 1):
            sess.stochastic_reduce()
            ref = oracle.mix.stochastic_reduce(ref, p, i, w)
            if t in (1, 10, 50, 100):
                St = sess.models()[:, cols_t].cpu().numpy().astype(np.float64)
                assert_models_close(St, ref, what=f"d={d} round {t}")
                drift = np.abs(St.mean(axis=0) - mean0).max()
                assert drift <= t * (d + 2) * 2.0 ** -24 * np.abs(S0).max(), (d, t, drift)
                dev = float(np.linalg.norm(St - St.mean(axis=0)))
                assert dev <= max(dev0 * s2 ** t * (1 + 1e-4), 1e-5 * dev0), (d, t, dev)
                print(f"d={d} t={t} deviation {dev / dev0:.3e} (bound {s2 ** t:.3e})", flush=True)
        assert sess.check()[0] == asap.OK
        sess.close()
        torch.cuda.empty_cache()


# ----------------------------------------------------------------------------
# NOTIFY-ACK epochs and state machine
# ----------------------------------------------------------------------------
def test_stale_neighbour_tag_is_reported(torch):
    n = 8
    p, i, w = graph("ring", n)
    sess = asap.Session(n, 256, p, i, w)
    sess.ready()
    sess.stochastic_reduce()
    assert sess.check() == (asap.OK, -1)
    # worker 3 has not published round 1: its readers 2, 3, 4 must not reduce
    b, r, _ = sess.current()
    asap.asap_debug_set_tag(sess.ctx, b, 3, 2 * r - 2)
    sess.stochastic_reduce()
    st, bad = sess.check()
    assert st == asap.E_EPOCH and bad == 2
    assert sess.check() == (asap.OK, -1)   # cleared
    sess.close()
    # complete graph: everyone reads everyone
    p, i, w = graph("complete", 16)
    sess = asap.Session(16, 300, p, i, w)
    sess.ready()
    asap.asap_debug_set_tag(sess.ctx, 0, 9, 77)
    sess.stochastic_reduce()
    assert sess.check()[0] == asap.E_EPOCH
    sess.close()


def test_state_machine_on_device(torch):
    wl = synth.SPARSE_LR_64W.with_(n_workers=4, dim=512, samples=64)
    p, i, w = graph("ring", 4)
    rp, col, val, y = synth.csr_data(wl)
    sess = asap.Session(4, wl.dim, p, i, w)
    sess.bind_csr(rp, col, val, y, wl.samples)
    prm = params(wl)
    sess.local_sgd(prm)
    assert sess.current() == (0, 0, 1)
    with pytest.raises(asap.AsapError) as e:
        sess.local_sgd(prm)
    assert e.value.status == asap.E_STATE
    sess.stochastic_reduce()
    assert sess.current() == (1, 1, 0)
    for bad in (asap.sgd_params(batch=0), asap.sgd_params(batch=513), asap.sgd_params(batch=4, lr0=-1.0),
                asap.sgd_params(batch=4, l2=-1.0), asap.sgd_params(loss=7, batch=4)):
        with pytest.raises(asap.AsapError) as e:
            sess.local_sgd(bad)
        assert e.value.status == asap.E_INVALID_ARG
    # resume: buffer 1 declared as round 5 -> schedule and step counter continue from 5
    asap.asap_set_round(sess.ctx, 5, 1)
    assert sess.current() == (1, 5, 0)
    sess.round(prm)
    assert sess.current() == (0, 6, 0)
    assert sess.check()[0] == asap.OK
    sess.close()


def test_bad_csr_rejected_at_workspace_bind(torch):
    wl = synth.SPARSE_LR_64W.with_(n_workers=3, dim=100, samples=10, nnz_mean=5.0)
    p, i, w = graph("ring", 3)
    rp, col, val, y = synth.csr_data(wl)
    for mutate, what in ((lambda c, v, yy: (np.where(c == c.max(), 100, c), v, yy), "outside"),
                         (lambda c, v, yy: (c, v, np.where(np.arange(yy.size) == 4, 0.5, yy)), "labels")):
        c2, v2, y2 = mutate(col.copy(), val.copy(), y.copy())
        sess = asap.Session(3, 100, p, i, w)
        sess.bind_csr(rp, c2, v2, y2, wl.samples)
        with pytest.raises(asap.AsapError) as e:
            sess.ready()
        assert e.value.status == asap.E_INVALID_ARG and what in str(e.value)
        sess.close()


def test_metrics_match_oracle(torch):
    wl = synth.SPARSE_SVM_256W.with_(n_workers=8, dim=1 << 12, samples=300, l2=1e-3)
    p, i, w = graph("random", 8, 4)
    rp, col, val, y = synth.csr_data(wl)
    shards = csr_shards(wl, rp, col, val, y)
    W = synth.initial_models(wl.with_(seed=5)) * np.float32(0.05)
    sess = asap.Session(8, wl.dim, p, i, w)
    sess.set_models(W)
    sess.bind_csr(rp, col, val, y, wl.samples)
    l2 = f32(wl.l2)
    m = sess.metrics(wl.loss, l2)
    W = W.astype(np.float64)
    own = np.mean([oracle.sgd.objective_csr(W[k], *shards[k][1:], wl.loss, l2) for k in range(8)])
    wbar = oracle.metrics.mean_model(W)
    bar = np.mean([oracle.sgd.objective_csr(wbar, *shards[k][1:], wl.loss, l2) for k in range(8)])
    assert m[0] == pytest.approx(own, rel=1e-9)
    assert m[1] == pytest.approx(bar, rel=1e-9)
    assert m[2] == pytest.approx(oracle.metrics.consensus_distance(W), rel=1e-9)
    assert m[3] == pytest.approx(W.mean(), rel=1e-9, abs=1e-15)
    sess.close()


@pytest.mark.parametrize("features", ["dense", "csr"])
def test_drop_workers_continues_on_the_new_graph(torch, features):
    """Reconfiguration after a failure: two of eight workers leave after round
    2; the six survivors, renumbered in order, continue on a ring built for
    six from the models they hold.  The oracle runs the same trajectory on
    its own state (its models of the survivors, the same new graph)."""
    if features == "dense":
        wl = synth.RING8_DENSE_LR.with_(samples=160)
    else:
        wl = synth.SPARSE_LR_64W.with_(n_workers=8, dim=1 << 13, samples=200)
    p, i, w = graph("ring", 8, 2)
    if features == "dense":
        X, y = synth.dense_data(wl)
        shards = [("dense", X[k], y[k]) for k in range(8)]
    else:
        rp, col, val, yy = synth.csr_data(wl)
        shards = csr_shards(wl, rp, col, val, yy)
    sess = asap.Session(8, wl.dim, p, i, w)
    if features == "dense":
        sess.bind_dense(X, y)
    else:
        sess.bind_csr(rp, col, val, yy, wl.samples)
    prm = params(wl)
    W = np.zeros((8, wl.dim))

    def oracle_round(W, shards, p, i, w, r):
        halves = []
        for k, sh in enumerate(shards):
            sched = oracle.prng.schedule(wl.samples, wl.seed, k, r)
            if sh[0] == "dense":
                halves.append(oracle.sgd.sgd_pass_dense(W[k], sh[1], sh[2], sched, rnd=r, **oracle_kw(wl)))
            else:
                halves.append(oracle.sgd.sgd_pass_csr(W[k], sh[1], sh[2], sh[3], sh[4], sched, rnd=r,
                                                      **oracle_kw(wl)))
        return oracle.mix.stochastic_reduce(np.stack(halves), p, i, w)

    for r in range(2):
        sess.round(prm)
        W = oracle_round(W, shards, p, i, w, r)
        assert_models_close(sess.models().cpu().numpy(), W, what=f"round {r}")
    dropped, keep = [2, 5], [0, 1, 3, 4, 6, 7]
    p6, i6, w6 = graph("ring", 6, 2)
    before = sess.models().cpu().numpy().copy()
    sess.drop_workers(dropped, p6, i6, w6)
    assert sess.current()[1] == 2
    # the survivors keep their models bit for bit, in order
    assert np.array_equal(sess.models().cpu().numpy().view(np.uint32), before[keep].view(np.uint32))
    gp, gi, gw = asap.asap_get_graph(sess.ctx)  # the graph the reduce now applies
    assert np.array_equal(gp, p6) and np.array_equal(gi, i6) and np.array_equal(gw, np.asarray(w6, np.float32))
    W = W[keep]
    shards = [shards[k] for k in keep]
    for r in range(2, 4):
        sess.round(prm)
        W = oracle_round(W, shards, p6, i6, w6, r)
        assert_models_close(sess.models().cpu().numpy(), W, what=f"round {r} after the drop")
    assert sess.check()[0] == asap.OK
    sess.close()


def _csr_run_against_oracle(wl, rp, col, val, yy, p, i, w, rounds):
    """Stream-ordered rounds on the given shards and graph, free-running
    against the oracle from zero models."""
    _free_run(None, wl, None, 0, rounds, data=(rp, col, val, yy), gr=(p, i, w))


@pytest.mark.parametrize("batch", [32, 100])  # planned pass, general kernel
def test_csr_empty_rows_and_an_empty_shard(torch, batch):
    # rows without nonzeros (margin 0: only their label and the batch size
    # count) in every worker, and one worker whose whole shard is empty
    wl = synth.SPARSE_LR_64W.with_(n_workers=6, dim=1 << 12, samples=300, batch=batch, nnz_mean=20.0)
    rp, col, val, yy = synth.csr_data(wl)
    S = wl.samples
    keep_row = np.ones(wl.n_workers * S, bool)
    keep_row[::7] = False              # every 7th row empty
    keep_row[2 * S:3 * S] = False      # worker 2: no nonzeros at all
    lens = np.diff(rp) * keep_row
    rp2 = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    keep_nz = np.repeat(keep_row, np.diff(rp))
    col2, val2 = col[keep_nz], val[keep_nz]
    assert rp2[3 * S] == rp2[2 * S] and rp2[-1] == col2.size
    p, i, w = graph("ring", wl.n_workers, 2)
    _csr_run_against_oracle(wl, rp2, col2, val2, yy, p, i, w, 3)


def test_single_worker_context(torch):
    # n = 1: the graph is the worker itself (P = [1]), the reduce a copy
    wl = synth.SPARSE_SVM_256W.with_(n_workers=1, dim=1 << 11, samples=200, l2=1e-3)
    rp, col, val, yy = synth.csr_data(wl)
    p, i, w = np.array([0, 1], np.int32), np.array([0], np.int32), np.array([1.0], np.float32)
    _csr_run_against_oracle(wl, rp, col, val, yy, p, i, w, 3)
