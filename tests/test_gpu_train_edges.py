"""GPU training step at the edges of its tiles: batches around 16 rows (a
workgroup), 32 rows (a block of the weight gradients' sums) and 256 rows (the
blocks loaded ahead), with indices outside the rows among them.

Bars as for the step's test at one batch: gradients 1e-3 of their norm
against the BF16 oracle (BF16 activations, FP32 sums on both sides), the
loss 1e-3.  The oracle takes a row of an invalid index as one of zero features
and zero targets.
"""
import numpy as np
import pytest

import oracle
from paper_2007_12273_amd import synth

from gpu_util import dev, torch
from test_gpu_warm import _oracle_feature_bits, _params, _rel, _subset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,bad", [(1, 0), (15, 0), (17, 2), (32, 0), (33, 1), (256, 3), (257, 0), (512, 0), (545, 5)])
def test_train_step_at_the_edges_of_its_tiles(B, bad):
    from paper_2007_12273_amd import api
    n = 600
    d = _subset(synth.make("weibel_3v"), n)
    f, X, _ = _oracle_feature_bits(d)
    rng = np.random.default_rng(B)
    T = np.zeros((n, 160))
    for r in range(n):
        k = rng.integers(1, 6)
        w = np.sort(rng.dirichlet(np.ones(k)))[::-1]
        for j in range(k):
            T[r, 10 * j] = w[j]
            T[r, 10 * j + 1:10 * j + 10] = rng.normal(size=9) * 0.5
    idx = rng.permutation(n)[:B].astype(np.int32)
    wrong = rng.permutation(B)[:bad]
    idx[wrong] = np.where(np.arange(bad) % 2, -1, n)
    Xb, Tb = X[idx % n], T[idx % n]
    Xb[wrong] = Tb[wrong] = 0.0
    P = _params(12)
    m = api.WarmStart(16, batch=B, seed=1)
    m.set_params(api.params_to_flat(P))
    rows = torch.full((B,), 7.0, dtype=torch.float32, device=dev())
    m.train_step(f, torch.from_numpy(T.astype(np.float32)).to(dev()), torch.from_numpy(idx).to(dev()), lr=1e-3, lam=1.0,
                 loss_rows=rows)
    rows = rows.cpu().numpy()
    assert (rows[wrong] == 0).all()
    Lo, go = oracle.mlp_loss_backward(Xb, P, Tb.astype(np.float32), lam=1.0, bf16=True)
    assert abs(float(rows.sum()) / B - Lo) <= 1e-3 * abs(Lo)
    grads = api.flat_to_params(m.gradients())
    for name in ("W1", "b1", "W2", "b2", "W3", "b3"):
        gg = grads[name][:105] if name == "W1" else grads[name]
        err = _rel(gg, go[name])
        print("batch %d, grad %s: relative error %.2e" % (B, name, err))
        assert err < 1e-3, name
    assert (grads["W1"][105:] == 0).all()
    m.close()
