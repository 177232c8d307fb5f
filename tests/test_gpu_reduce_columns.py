"""The reduce's column kernel at the edges of its layouts: worker counts and
widths around a change of lanes per row, graphs whose lists just fit or do not
fit beside the chunk, ragged columns, rows with a stale neighbour."""
import numpy as np
import pytest

from paper_1612_08608_amd import asap
import oracle

pytestmark = pytest.mark.gpu


def _rows_in_order(W, ptr, idx, w):
    """fp64 sums in row order, rounded once: a product of two fp32 values is
    exact in fp64, so this is bit for bit a chain of fused multiply-adds."""
    out = np.zeros(W.shape)
    for i in range(W.shape[0]):
        for p in range(ptr[i], ptr[i + 1]):
            out[i] += float(w[p]) * W[idx[p]].astype(np.float64)
    return out.astype(np.float32)


def _circulant(n, d):
    """Every worker with its d nearest and itself."""
    rows = [sorted({(i + s) % n for s in range(-(d // 2), d // 2 + 1)}) for i in range(n)]
    return np.arange(n + 1, dtype=np.int32) * (d + 1), np.concatenate(rows).astype(np.int32)


SHAPES = [
    (1, 0, 5), (3, 2, 1), (5, 2, 255), (7, 4, 256), (9, 2, 257), (25, 4, 1023), (66, 6, 515), (127, 4, 1030),
    (128, 20, 260), (129, 4, 131), (254, 18, 127), (255, 4, 128), (257, 4, 65), (511, 6, 64), (513, 4, 33),
    (1000, 4, 70), (1000, 16, 67), (1023, 4, 31), (1026, 2, 40),
    # a chunk for every compute unit, with each number of lanes; narrower ones;
    # lists that do not fit beside a narrower one
    (66, 4, 65281), (128, 20, 65537), (254, 6, 32641), (400, 4, 16321), (544, 4, 8100), (545, 4, 8100), (1000, 4, 8161),
    (100, 6, 40003), (255, 4, 20000), (300, 20, 9001), (127, 124, 40001), (128, 126, 20003),
    # rows of three entries, models within the memory-side cache and below
    (66, 2, 198900), (66, 2, 198800), (129, 2, 46600), (129, 2, 46400),
]


@pytest.mark.parametrize("n,d,dim", SHAPES)
def test_reduce_is_the_rows_sum_in_order(n, d, dim):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] reduce n={n} d={d} dim={dim}", flush=True)
    if n == 1:
        p, i = np.array([0, 1], np.int32), np.zeros(1, np.int32)
    else:
        p, i = oracle.graphs.random_regular(n, d, 3) if d <= 20 else _circulant(n, d)
    w = oracle.graphs.metropolis_weights(p, i)
    W = np.random.default_rng([n, dim]).standard_normal((n, dim), dtype=np.float32)
    sess = asap.Session(n, dim, p, i, w)
    sess.set_models(W)
    sess.bufs[1].fill_(7.0)
    sess.stochastic_reduce()
    got = sess.models().cpu().numpy()
    assert sess.check()[0] == asap.OK
    assert np.array_equal(got.view(np.uint32), _rows_in_order(W, p, i, w).view(np.uint32))
    assert bool((sess.bufs[1][:, dim:] == 7.0).all())  # entries past dim are never written
    # a stale tag: the rows that read that worker stay, the others are reduced
    asap.asap_set_round(sess.ctx, 5, 0)
    sess.bufs[1].fill_(7.0)
    stale = n // 2
    asap.asap_debug_set_tag(sess.ctx, 0, stale, 3)
    sess.stochastic_reduce()
    want = _rows_in_order(W, p, i, w)
    readers = [r for r in range(n) if stale in i[p[r]:p[r + 1]]]
    want[readers] = 7.0
    st, bad = sess.check()
    assert (st, bad) == (asap.E_EPOCH, min(readers))
    assert np.array_equal(sess.models().cpu().numpy().view(np.uint32), want.view(np.uint32))
    sess.close()


@pytest.mark.parametrize("n,d,dim", [(100, 4, 70001), (300, 6, 20001), (1000, 4, 9001), (1000, 4, 300), (64, 0, 5003),
                                     (64, 8, 9000), (64, 16, 9000), (1030, 4, 500)])
def test_captured_reduce_replays(n, d, dim):
    """Every kernel of the reduce captured and replayed on other models, with
    eager work between the replays (d = 0: the complete graph)."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] captured reduce n={n} d={d} dim={dim}", flush=True)
    p, i = oracle.graphs.random_regular(n, d, 5) if d else oracle.graphs.complete(n)
    w = oracle.graphs.metropolis_weights(p, i)
    gen = torch.Generator("cuda").manual_seed(n)
    eager, captured = asap.Session(n, dim, p, i, w), asap.Session(n, dim, p, i, w)
    for s in (eager, captured):
        s.ready()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        captured.stochastic_reduce()
    for _ in range(4):
        W = torch.randn((n, dim), generator=gen, device="cuda")
        for s in (eager, captured):
            asap.asap_set_round(s.ctx, 0, 0)
            s.bufs[0][:, :dim].copy_(W)
            s.bufs[1].zero_()
        eager.stochastic_reduce()
        g.replay()
        torch.cuda.synchronize()
        assert eager.check()[0] == captured.check()[0] == asap.OK
        assert bool(eager.bufs[1].any()) and torch.equal(eager.bufs[1], captured.bufs[1])
    eager.close()
    captured.close()
