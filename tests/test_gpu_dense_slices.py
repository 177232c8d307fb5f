"""The dense pass at the edges of its layout: widths around a lane group, a
unit and a workgroup's units, worker counts that change how many workgroups a
worker gets, batches that leave row waves idle, against the oracle and, for
the multi-round launch, against the stream-ordered rounds bit for bit."""
import numpy as np
import pytest

from conftest import assert_models_close
from paper_1612_08608_amd import asap, synth
import oracle

pytestmark = pytest.mark.gpu

# workers, dim, samples, batch, local steps (0: whole passes)
SHAPES = [
    (3, 63, 37, 16, 0), (3, 64, 33, 40, 0), (5, 65, 70, 33, 0),          # 16 lanes a row slice, then a whole wave
    (9, 256, 40, 7, 0), (9, 257, 40, 8, 0), (8, 513, 66, 33, 0),         # one unit, two, three
    (20, 1000, 101, 50, 0), (40, 1000, 24, 3, 0), (72, 700, 20, 20, 0),  # 8, 6 and 3 workgroups a worker at most
    (130, 500, 18, 5, 0), (130, 1023, 18, 5, 0),                         # one: two and four float4 a lane
    (300, 40, 30, 10, 0), (600, 300, 8, 8, 0), (1500, 70, 6, 4, 0),      # several workers a compute unit
    (3072, 33, 5, 3, 0), (3073, 64, 4, 3, 0), (4096, 64, 5, 2, 0),       # ... 12 and 16: all resident in a launch
    (33, 4097, 20, 8, 0), (72, 9001, 9, 4, 0), (130, 1500, 16, 6, 0),    # several units a workgroup
    (130, 8190, 9, 4, 0), (66, 16384, 6, 3, 0),                          # ... of four float4 a lane
    (130, 8200, 6, 2, 0),                                                # wider than a workgroup's waves hold
    (1, 8193, 12, 5, 0), (2, 16381, 10, 64, 0),                          # few workers, wide models, batch > samples
    (4, 600, 48, 8, 2), (12, 2000, 40, 10, 1),                           # several rounds a pass
    # groups of eight rows (more than 32 rows a step): five to eight units, several groups a step
    (8, 2048, 150, 128, 0), (12, 1300, 70, 40, 0), (5, 700, 200, 130, 0), (16, 2000, 300, 256, 0), (3, 1793, 90, 66, 1),
]


@pytest.mark.parametrize("n,dim,S,B,L", SHAPES)
def test_dense_pass_shapes(n, dim, S, B, L):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] dense pass n={n} dim={dim} S={S} B={B} L={L}", flush=True)
    loss = "hinge" if (dim + n) % 2 else "logistic"
    # Features N(0, 1), without columns scaled tenfold: the model is held in
    # fp32 between steps, and with scaled columns that rounding alone moves
    # entries by up to 1.83e-5 (130 x 8190, an fp64 pass rounded to fp32 after
    # every step, to the digit what the device gives) against 4.0e-7 without.
    wl = synth.DENSE_LR_32W.with_(n_workers=n, dim=dim, samples=S, batch=B, l2=0.01 if n % 2 else 0.0, loss=loss,
                                  lr_kind="inv_sqrt", lr0=0.1, seed=n, scaled_frac=0.0)
    p, i = oracle.graphs.ring(n) if n >= 3 else oracle.graphs.complete(n)
    w = oracle.graphs.metropolis_weights(p, i)
    X, y = synth.dense_data(wl)
    # entries past dim are never used: NaN there must not reach a result
    ldx = (dim + 3) // 4 * 4
    Xp = np.full((n, S, ldx), np.nan, np.float32)
    Xp[:, :, :dim] = X
    W0 = synth.initial_models(wl) * np.float32(0.01)
    prm = asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, wl.batch, wl.seed, L)
    rounds = 3
    got = []
    for launch in (False, True):
        sess = asap.Session(n, dim, p, i, w)
        sess.set_models(W0)
        Xd, yd = torch.as_tensor(Xp).cuda(), torch.as_tensor(y).cuda()
        asap.asap_bind_dense(sess.ctx, Xd, yd, S, ldx)
        if launch:
            sess.run_rounds(prm, rounds, wait_ms=3000)
        else:
            for _ in range(rounds):
                sess.round(prm)
        assert sess.check()[0] == asap.OK
        got.append(sess.models().cpu().numpy().copy())
        sess.close()
    K = oracle.sgd.n_steps(S, B)
    ref = W0.astype(np.float64)
    for r in range(rounds):
        q, k0, k1 = oracle.sgd.round_steps(r, L, K)
        half = [oracle.sgd.sgd_pass_dense(ref[k], X[k], y[k], oracle.prng.schedule(S, wl.seed, k, q), batch=B, loss=loss,
                                          lr_kind=wl.lr_kind, lr0=float(np.float32(wl.lr0)),
                                          l2=float(np.float32(wl.l2)), rnd=q, steps=(k0, k1)) for k in range(n)]
        ref = oracle.mix.stochastic_reduce(np.stack(half), p, i, w)
    assert_models_close(got[0], ref, what="stream-ordered rounds")
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))


@pytest.mark.parametrize("n,dim,fits", [(4096, 3, True), (4097, 64, False), (2048, 256, True), (1024, 512, True),
                                         (1100, 300, False), (512, 1024, True), (520, 1000, False), (256, 2000, True),
                                         (300, 1500, False), (256, 16384, True), (257, 9000, False)])
def test_launch_fits_or_is_refused(n, dim, fits):
    """The most workers a multi-round launch takes; one that does not fit is
    refused with ASAP_E_STATE and leaves the state as it was."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] launch limit n={n} dim={dim}", flush=True)
    wl = synth.DENSE_LR_32W.with_(n_workers=n, dim=dim, samples=2, batch=1, scaled_frac=0.0)
    p, i = oracle.graphs.ring(n)
    w = oracle.graphs.metropolis_weights(p, i)
    gen = torch.Generator("cuda").manual_seed(n)
    X = torch.randn((n, 2, (dim + 3) // 4 * 4), generator=gen, device="cuda")
    y = torch.where(torch.rand((n, 2), generator=gen, device="cuda") < 0.5, -1.0, 1.0)
    prm = asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, wl.batch, wl.seed)
    stream, launch = asap.Session(n, dim, p, i, w), asap.Session(n, dim, p, i, w)
    for s in (stream, launch):
        asap.asap_bind_dense(s.ctx, X, y, 2, X.shape[2])
        s.ready()
    if fits:
        launch.run_rounds(prm, 2, wait_ms=3000)
    else:
        with pytest.raises(asap.AsapError) as refused:
            launch.run_rounds(prm, 2, wait_ms=3000)
        assert refused.value.status == asap.E_STATE
    for k in range(2):
        stream.round(prm)
        if not fits:
            launch.round(prm)
    assert stream.check()[0] == launch.check()[0] == asap.OK
    assert torch.equal(stream.models(), launch.models())
    stream.close()
    launch.close()


@pytest.mark.parametrize("n,dim,S,B", [(4, 600, 24, 64), (8, 2000, 64, 8)])  # one group a launch, eight
def test_captured_pass_replays(n, dim, S, B):
    """A captured half-step replayed: every replay takes new exchange tags, so
    it gives the bits of the same half-step run eagerly."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] captured dense pass n={n} dim={dim} S={S} B={B}", flush=True)
    wl = synth.DENSE_LR_32W.with_(n_workers=n, dim=dim, samples=S, batch=B, scaled_frac=0.0)
    p, i = oracle.graphs.ring(n)
    w = oracle.graphs.metropolis_weights(p, i)
    X, y = synth.dense_data(wl)
    prm = asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, wl.batch, wl.seed)
    eager, captured = asap.Session(n, dim, p, i, w), asap.Session(n, dim, p, i, w)
    for s in (eager, captured):
        s.bind_dense(X, y)
        s.ready()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        captured.local_sgd(prm)
    for _ in range(4):
        eager.local_sgd(prm)
        asap.asap_set_round(eager.ctx, 0, 0)  # the same half-step again
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured.models(), eager.models())
    eager.close()
    captured.close()


# one shape for each variant of the pass, with a last group that its rows do not fill
@pytest.mark.parametrize("n,dim,S", [(3, 60, 5), (5, 200, 5), (130, 500, 5), (130, 1000, 3), (4, 600, 5), (4, 600, 37),
                                     (33, 4097, 5), (130, 1500, 5), (130, 8190, 3), (130, 8200, 3)])
@pytest.mark.parametrize("loss", ["logistic", "hinge"])
def test_infinite_entry_stays_in_its_column(n, dim, S, loss):
    """A step (B > S) from models with one infinite entry: its rows' margins are
    infinite, which both losses have a derivative for, so the other columns stay
    finite.  Rows that fill up a group but do not exist must not turn the
    infinity into NaN (0 * inf) and add that to every column."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] infinite entry n={n} dim={dim} S={S} {loss}", flush=True)
    wl = synth.DENSE_LR_32W.with_(n_workers=n, dim=dim, samples=S, batch=64, l2=0.0, loss=loss, lr_kind="const", lr0=0.1,
                                  seed=n, scaled_frac=0.0)
    p, i = oracle.graphs.ring(n)
    X, y = synth.dense_data(wl)
    W0 = synth.initial_models(wl) * np.float32(0.01)
    hot = dim // 3
    W0[:, hot] = np.where(np.arange(n) % 2, np.inf, -np.inf)
    sess = asap.Session(n, dim, p, i, oracle.graphs.metropolis_weights(p, i))
    sess.set_models(W0)
    sess.bind_dense(X, y)
    sess.local_sgd(asap.sgd_params(wl.loss, wl.lr_kind, wl.lr0, wl.l2, wl.batch, wl.seed))
    assert sess.check()[0] == asap.OK
    got = sess.models().cpu().numpy().copy()
    sess.close()
    with np.errstate(invalid="ignore"):  # the infinite column itself: inf - 0 * inf
        ref = np.stack([oracle.sgd.sgd_pass_dense(W0[k].astype(np.float64), X[k], y[k],
                                                  oracle.prng.schedule(S, wl.seed, k, 0), batch=wl.batch, loss=loss,
                                                  lr_kind=wl.lr_kind, lr0=float(np.float32(wl.lr0)), l2=0.0, rnd=0)
                        for k in range(n)])
    rest = np.arange(dim) != hot
    assert np.isfinite(ref[:, rest]).all()
    assert_models_close(got[:, rest], ref[:, rest], what="finite columns")


@pytest.mark.parametrize("dim,checked", [(1024, False), (1025, True), (8192, True), (8193, False)])
def test_shards_checked_when_bound(dim, checked):
    """Widths at which labels and finiteness are checked; padding columns are
    not."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] bind check dim={dim}", flush=True)
    p, i = oracle.graphs.ring(3)
    ldx = (dim + 3) // 4 * 4 + 4

    def bind(edit):
        X, y = torch.ones((3, 20, ldx), device="cuda"), torch.ones((3, 20), device="cuda")
        X[:, :, dim:] = float("nan")
        edit(X, y)
        sess = asap.Session(3, dim, p, i, oracle.graphs.metropolis_weights(p, i))
        asap.asap_bind_dense(sess.ctx, X, y, 20, ldx)
        sess.ready()
        sess.close()

    def label(X, y):
        y[2, 19] = 0.5

    def value(X, y):
        X[2, 19, dim - 1] = float("inf")

    bind(lambda X, y: None)
    for edit in (label, value):
        if checked:
            with pytest.raises(asap.AsapError) as refused:
                bind(edit)
            assert refused.value.status == asap.E_INVALID_ARG
        else:
            bind(edit)


def _two_sessions(torch, shapes):
    """Dense sessions on random shards, with their parameters."""
    out = []
    for k, (n, dim, S, B) in enumerate(shapes):
        p, i = oracle.graphs.ring(n)
        gen = torch.Generator("cuda").manual_seed(k)
        X = torch.randn((n, S, (dim + 3) // 4 * 4), generator=gen, device="cuda")
        y = torch.where(torch.rand((n, S), generator=gen, device="cuda") < 0.5, -1.0, 1.0)
        sess = asap.Session(n, dim, p, i, oracle.graphs.metropolis_weights(p, i))
        asap.asap_bind_dense(sess.ctx, X, y, S, X.shape[2])
        sess.ready()
        out.append((sess, asap.sgd_params("logistic", "inv_sqrt", 0.1, 0.0, B, k), X, y))
    torch.cuda.synchronize()
    return out


STREAM_PAIRS = [((25, 1000, 400, 50), (33, 1000, 300, 20)), ((20, 600, 300, 16), (12, 12000, 64, 16)),
                ((32, 4096, 128, 32), (64, 1000, 256, 32))]


@pytest.mark.parametrize("pair", STREAM_PAIRS)
def test_two_contexts_on_two_streams(pair):
    """Passes whose workgroups wait for each other, of two contexts at once:
    each context's bits are those it has alone."""
    import threading

    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] two contexts {pair}", flush=True)
    rounds = 20
    want = []
    for sess, prm, *_ in _two_sessions(torch, pair):
        for _ in range(rounds):
            sess.round(prm)
        assert sess.check()[0] == asap.OK
        want.append(sess.models().clone())
        sess.close()
    both = _two_sessions(torch, pair)

    def work(sess, prm):
        stream = torch.cuda.Stream()
        for _ in range(rounds // 2):
            sess.round(prm, stream=stream)
        sess.run_rounds(prm, rounds // 2, wait_ms=3000, stream=stream)
        stream.synchronize()

    threads = [threading.Thread(target=work, args=both[k][:2]) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert both[k][0].check()[0] == asap.OK
        assert torch.equal(both[k][0].models(), want[k])
        both[k][0].close()


@pytest.mark.parametrize("pair", STREAM_PAIRS)
def test_two_captured_passes_on_two_streams(pair):
    """The same for captured half-steps, replayed side by side: together they
    have more workgroups than fit, and each launch has to get all of its own."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] two captured passes {pair}", flush=True)
    replays = 10
    want = []
    for sess, prm, *_ in _two_sessions(torch, pair):
        for _ in range(replays):
            sess.local_sgd(prm)
            asap.asap_set_round(sess.ctx, 0, 0)
        assert sess.check()[0] == asap.OK
        want.append(sess.models().clone())
        sess.close()
    both = _two_sessions(torch, pair)
    graphs, streams = [], []
    for sess, prm, *_ in both:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            sess.local_sgd(prm)
        graphs.append(g)
        streams.append(torch.cuda.Stream())
    torch.cuda.synchronize()
    for _ in range(replays):
        for g, stream in zip(graphs, streams):
            with torch.cuda.stream(stream):
                g.replay()
    torch.cuda.synchronize()
    for k in range(2):
        assert both[k][0].check()[0] == asap.OK
        assert torch.equal(both[k][0].models(), want[k])
        both[k][0].close()
