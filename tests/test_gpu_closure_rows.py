"""Closure batches of many rows.

* Above 4096 rows the forward layers take other tiles (64 columns, the contraction in panels of 64); every sum keeps its order, so
  the outputs are those of the same rows in calls of at most 4096, bit for bit.
* Above 4608 rows a split of a weight gradient has more than one panel of 288 rows (here 320 and 288 + 288 + 32 a split): loss and
  gradients against the oracle's network with the same bfloat16 rounding points, 1e-3 normwise as for small batches.
"""
import numpy as np
import pytest

from helpers import rel
from oracle import closure as oc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _closure(max_batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_18026_amd as m
    plan = m.Plan(12, 8, 6, 1.2, 4.0)
    return m.Closure(plan, max_batch=max_batch, beta=1.0)


def _problem(seed, nb):
    rng = np.random.default_rng(seed)
    w = [rng.standard_normal(n) * s for n, s in ((256 * 258, 0.06), (256, 0.1), (256 * 256, 0.06), (256, 0.1),
                                                 (256 * 256, 0.06), (256, 0.1))]
    return (np.concatenate(w).astype(np.float32), rng.standard_normal((nb, 258)).astype(np.float32),
            rng.standard_normal((nb, 256)).astype(np.float32))


@pytest.mark.parametrize("nb", [4097, 4160, 9000])
def test_many_rows_keep_the_bits(nb):
    print("closure forward rows", nb, flush=True)
    cl = _closure(nb)
    params, X, _ = _problem(1, nb)
    cl.set_params(params)
    x = torch.from_numpy(X).cuda()
    whole, parts = torch.full((nb, 256), float("nan"), device="cuda"), torch.empty((nb, 256), device="cuda")
    cl.forward(x, whole)
    for r in range(0, nb, 4096):
        n = min(4096, nb - r)
        y = torch.empty((n, 256), device="cuda")
        cl.forward(x[r:r + n].contiguous(), y)
        parts[r:r + n] = y
    assert torch.equal(whole, parts)


@pytest.mark.parametrize("nb", [4700, 9700])
def test_gradients_of_many_rows(nb):
    print("closure gradients rows", nb, flush=True)
    cl = _closure(nb)
    params, X, Y = _problem(2, nb)
    cl.set_params(params)
    loss = cl.train_step(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), None, nb, 0.0, want_loss=True)
    ref_loss, ref = oc.loss_and_grads(X.astype(np.float64), Y.astype(np.float64), *oc.network_params(params))
    assert abs(loss - ref_loss) < 1e-5 * ref_loss
    err = rel(cl.get_grads(), oc.flatten_grads(ref))
    print("  gradient", err, flush=True)
    assert err < 1e-3
