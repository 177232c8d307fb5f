"""The general CSR step at its edges: minibatches that are one row more or less
than a pass over the lane groups, rows that fill the cold table by themselves,
chunks cut inside a minibatch, rows with the longest length accepted."""
import numpy as np
import pytest

from conftest import assert_models_close
from paper_1612_08608_amd import asap
import oracle

pytestmark = pytest.mark.gpu

# workers, dim, samples, batch, shortest and longest row, l2
SHAPES = [
    (3, 3000, 70, 65, 1, 40, 0.0),            # one row more than the lane groups; every column on chip
    (2, 200000, 130, 128, 30, 60, 0.0),       # cold columns, several chunks
    (2, 200000, 40, 20, 100, 700, 1e-3),      # long rows in small minibatches
    (1, 150000, 9, 4, 4000, 4096, 0.0),       # rows that fill the table
    (2, 150000, 513, 512, 0, 12, 1e-3),       # the largest minibatch, a last one of one row, empty rows
    # 64, 32 and 16 lanes a row: 16 rows and one more, 32 and one more
    (2, 30000, 48, 16, 120, 400, 1e-3), (2, 30000, 50, 17, 0, 500, 0.0), (2, 2000, 64, 32, 129, 300, 0.0),
    (3, 30000, 66, 33, 1, 200, 0.0), (2, 100000, 22, 10, 1000, 4096, 0.0),
]


@pytest.mark.parametrize("n,D,S,B,lo,hi,l2", SHAPES)
@pytest.mark.parametrize("loss", ["logistic", "hinge"])
def test_general_step_shapes(n, D, S, B, lo, hi, l2, loss):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[gpu] csr general n={n} D={D} S={S} B={B} rows {lo}..{hi} {loss}", flush=True)
    rng = np.random.default_rng([n, D, S, B])
    lens = rng.integers(lo, hi + 1, n * S)
    lens[0] = hi
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(D, k, replace=False)) for k in lens]).astype(np.int32)
    val = (rng.standard_normal(col.size) / np.sqrt(max(hi, 1))).astype(np.float32)
    y = np.where(rng.random(n * S) < 0.5, -1.0, 1.0).astype(np.float32)
    p, i = oracle.graphs.ring(n) if n >= 3 else oracle.graphs.complete(n)
    w = oracle.graphs.metropolis_weights(p, i)
    prm = asap.sgd_params(loss, "inv_sqrt", 0.3, l2, B, 5)
    got = []
    for launch in (False, True):
        sess = asap.Session(n, D, p, i, w)
        sess.bind_csr(rp, col, val, y, S)
        sess.set_csr_members(1)
        if launch:
            sess.run_rounds(prm, 2, wait_ms=3000)
        else:
            sess.round(prm)
            sess.round(prm)
        assert sess.check()[0] == asap.OK
        got.append(sess.models().cpu().numpy().copy())
        sess.close()
    ref = np.zeros((n, D))
    for r in range(2):
        half = []
        for k in range(n):
            a, b = rp[k * S], rp[(k + 1) * S]
            half.append(oracle.sgd.sgd_pass_csr(ref[k], rp[k * S:(k + 1) * S + 1] - a, col[a:b], val[a:b],
                                                y[k * S:(k + 1) * S], oracle.prng.schedule(S, 5, k, r), batch=B,
                                                loss=loss, lr_kind="inv_sqrt", lr0=float(np.float32(0.3)),
                                                l2=float(np.float32(l2)), rnd=r))
        ref = oracle.mix.stochastic_reduce(np.stack(half), p, i, w)
    assert_models_close(got[0], ref, what="stream-ordered rounds")
    if B > 64:  # below, the stream path may take the planned pass, the launch without a ring the general one
        assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
    else:
        assert_models_close(got[1], ref, what="multi-round launch")
