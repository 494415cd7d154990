"""The trainer's loop, two launches a step (the gradient kernel draws its own
minibatch; the Adam kernel also stores the new parameters in the packed
operands), against the same steps made one by one: the rows from the oracle's
Philox draw, hca_mlp_gradient on them (which packs the parameters anew) and
hca_mlp_apply_gradient.  Both sum the same partials in the same order, so the
losses and parameters agree bit for bit, at one workgroup, at batches that are
not a multiple of the Adam kernel's 64 partials, and at several of them."""
import numpy as np
import pytest
import torch

from oracle import philox
from paper_2105_00448_amd import hca

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [64, 192, 4096, 64 * 65, 64 * 130])
def test_train_equals_single_steps(batch):
    print(f"\n[train step] batch {batch}", flush=True)
    n, seed, steps, lr = 5003, 11, 3, 1e-3
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X = torch.rand((n, 6), generator=g, device="cuda")
    Y = torch.stack([X[:, 0] * X[:, 3], torch.sin(3 * X[:, 1]), X[:, 5] - X[:, 2]], 1).contiguous()
    loop, single = hca.Trainer(X, Y, seed=seed), hca.Trainer(X, Y, seed=seed)
    losses = loop.train(steps, batch=batch, lr=lr)
    grad = torch.empty(hca.MLP_NPARAM, device="cuda")
    for t in range(1, steps + 1):
        o0, _, _, _ = philox.block_vec(np.arange(batch, dtype=np.uint64), t, 3, 0, (seed, 0))
        idx = torch.from_numpy((o0 % np.uint64(n)).astype(np.int32)).cuda()
        loss = single.gradient(idx, grad)
        assert np.float32(loss) == losses[t - 1]
        single.apply_gradient(grad, lr)
    assert np.array_equal(single.params(), loop.params())
