"""The training kernels at the batch sizes where their work split changes: a
single sample, the most that have a workgroup each, fewer than a workgroup's
four waves leave over, one more round than the persistent grid, against the fp64 oracle.

Tolerances: a logit is three chained sums of at most 64 products, so its
rounding error is a few tens of fp32 epsilons (6e-8) of its terms; gradients
chain five such sums.  Relative to the 2-norm: 64 eps per sum, worst case,
3 * 64 * 6e-8 = 1.2e-5 and 5 * 64 * 6e-8 = 2e-5.  The Adam step divides the
gradient by its own magnitude, so only its entries well above that rounding
are compared, at 1e-3 of the step (lr)."""
import numpy as np
import pytest

from oracle import mlp
from workloads.mlp_init import he_uniform

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 3, 5, 31, 257, 512, 513, 1025, 4099])
def test_mlp_batch_sizes(B):
    import torch
    from paper_2509_01425_amd import hicr as H
    print("mlp batch", B, flush=True)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    g = np.random.default_rng(B)
    theta = he_uniform(B)
    x = np.log2(1.0 + g.integers(0, 300, size=(B, 32)) * (g.random((B, 32)) < 0.4)).astype(np.float32)
    y = g.integers(0, 12, size=B).astype(np.int32)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    z = torch.zeros(B, 12, device="cuda")
    grad = torch.zeros(mlp.N_PARAMS, device="cuda")
    loss = torch.zeros(2, device="cuda")
    torch.cuda.synchronize()
    assert H.hicr_mlp_set_params(ctx, theta) == H.OK
    assert H.hicr_mlp_forward(ctx, xd.data_ptr(), B, z.data_ptr()) == H.OK
    assert H.hicr_mlp_grad(ctx, xd.data_ptr(), yd.data_ptr(), B, grad.data_ptr(),
                           loss.data_ptr()) == H.OK
    assert H.hicr_mlp_train_step(ctx, xd.data_ptr(), yd.data_ptr(), B, 1e-3,
                                 loss.data_ptr() + 4) == H.OK
    rc, stepped = H.hicr_mlp_get_params(ctx)
    assert rc == H.OK
    th64, x64 = theta.astype(np.float64), x.astype(np.float64)
    z_ref, _ = mlp.forward(th64, x64)
    g_ref, L_ref = mlp.grad(th64, x64, y), mlp.loss(th64, x64, y)

    def off(a, ref):
        return np.linalg.norm(a.astype(np.float64) - ref) / np.linalg.norm(ref)

    assert off(z.cpu().numpy(), z_ref) <= 1.2e-5
    assert off(grad.cpu().numpy(), g_ref) <= 2e-5
    assert abs(float(loss[0]) - L_ref) <= 1.2e-5 * max(abs(L_ref), np.abs(z_ref).max())
    assert float(loss[1]) == float(loss[0])
    ref = mlp.Adam(mlp.N_PARAMS).step(th64, g_ref)
    big = np.abs(g_ref) > 1e-2 * np.abs(g_ref).max()
    assert big.any()
    assert np.abs(stepped - ref)[big].max() <= 1e-6
    assert (stepped[g_ref == 0] == theta[g_ref == 0]).all()
    # logits written over their own inputs are the logits
    assert H.hicr_mlp_set_params(ctx, theta) == H.OK
    assert H.hicr_mlp_forward(ctx, xd.data_ptr(), B, xd.data_ptr()) == H.OK
    assert torch.equal(xd.view(-1)[:12 * B], z.view(-1))
    assert H.hicr_ctx_destroy(ctx) == H.OK
