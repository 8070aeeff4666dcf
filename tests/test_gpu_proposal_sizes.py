"""The proposal network's kernels at the edges of their work splits: runs of
tiles that hold less than one per workgroup, cross clouds or end in half a
pair, and particle counts on either side of the set loss's parts and passes."""
import numpy as np
import pytest
import torch

import test_gpu_proposal as T
from oracle import proposal_oracle as PO
from paper_2106_03287_amd import proposal as PR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,B", [(64, 3), (64, 64), (128, 3), (192, 50), (1088, 60), (4096, 5)])
def test_per_point_kernel_over_runs_of_tiles(P, B):
    """Every pair of a batch gives the bits it gives alone: batches of up to 64
    pairs take the same products in the head (one row tile), so only the runs
    of point tiles differ, from one cloud in a workgroup to several."""
    K = 16
    clouds = T._cuda(T._clouds(B, P, 41))
    m = T._model(K, P, B, T._params(K, 42))
    together = m.forward(clouds)[0].clone()
    for b in sorted({0, 1, B // 2, B - 1}):
        alone = m.forward(clouds[b:b + 1].contiguous())[0]
        assert torch.equal(alone[0], together[b]), f"P={P} pair {b} of {B}"
    m.close()


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 255, 256, 257, 300])
def test_set_loss_and_its_gradient_at_the_edges_of_the_parts(K):
    """Loss (FP64 sums of FP64 terms: 1e-12 of the largest sum) and the
    gradient of the last bias, the sum over the batch of the loss's gradients
    rounded to FP32 (2^-24 of each, and of their sum)."""
    B, P = 2, 8
    rng = np.random.default_rng(K)
    params = T._params(K, 31)
    clouds = T._cuda(T._clouds(B, P, 32))
    targets = rng.standard_normal((B, K, 6)) * 0.3
    sigma = np.array([[0.1] * 3 + [0.2] * 3, [0.4] * 3 + [0.8] * 3])
    cfg = PR.stein_icp_proposal_default_config(num_particles=K, points=P, max_batch=B, loss_sigma=sigma)
    m = PR.Proposal(cfg, params)
    y = m.forward(clouds)[0].cpu().numpy()
    loss, grad = m.loss(clouds, T._cuda(targets, torch.float64), grad=True)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy().astype(np.float64)
    m.close()
    want = np.array([PO.mmd2(y[b], targets[b], sigma) for b in range(B)])
    np.testing.assert_allclose(loss, want, rtol=0, atol=1e-12 * 2 * len(sigma))
    each = np.stack([PO.mmd2_grad(y[b], targets[b], sigma) for b in range(B)]).reshape(B, -1) / B
    o, s = PO.layout(K)["b5"]
    got = grad[o:o + int(np.prod(s))]
    bound = 2.0 ** -24 * (np.abs(each).sum(0) + np.abs(each.sum(0))) + 1e-12 * np.abs(each).max()
    assert (np.abs(got - each.sum(0)) <= bound).all()


@pytest.mark.parametrize("K", [1, 255, 256, 257, 1000])
def test_stand_alone_set_distance_in_passes(K):
    rng = np.random.default_rng(K)
    X, Y = rng.standard_normal((2, 2, K, 6)) * 0.2
    sigma = np.array([[0.2] * 3 + [0.4] * 3])
    got = PR.stein_icp_proposal_mmd(T._cuda(X, torch.float64), T._cuda(Y, torch.float64), sigma).cpu().numpy()
    want = np.array([PO.mmd2(X[b], Y[b], sigma) for b in range(2)])
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-12)


def euler_gaps(params, grad, K):
    """A layer y = x W + b below a ReLU gate passes sum(y dy) = <W, gW> + <b, gb> down as sum(x dx) = <W, gW>: for
    each pair of layers the difference of both forms, and the summed magnitudes of its terms."""
    out = {}
    dot = {n: params[o:o + int(np.prod(s))] * grad[o:o + int(np.prod(s))] for n, (o, s) in PO.layout(K).items()}
    for lower, upper in ((1, 2), (2, 3), (3, 4), (4, 5)):
        terms = [dot[f"W{lower}"], dot[f"b{lower}"], -dot[f"W{upper}"]]
        out[f"{lower}-{upper}"] = (abs(sum(t.sum() for t in terms)), sum(np.abs(t).sum() for t in terms))
    return out


@pytest.mark.parametrize("P,B", [(1, 1), (8, 3), (64, 2), (300, 5), (1088, 33)])
def test_gradients_agree_between_layers(P, B):
    """Winner rows from one to all shares of a cloud, gates inside the products, bias sums of all layers at once.
    Four BF16 operands stand between the two forms, 2^-8 relative each: 2^-6 of the summed magnitudes. A row, a gate
    or a sum out of place changes a form by an amount of its own size."""
    K = 8
    params = T._params(K, 51)
    targets = np.random.default_rng(52).standard_normal((B, K, 6)) * 0.3
    sigma = np.array([[0.1] * 3 + [0.2] * 3, [0.4] * 3 + [0.8] * 3])
    cfg = PR.stein_icp_proposal_default_config(num_particles=K, points=P, max_batch=B + 2, loss_sigma=sigma)
    m = PR.Proposal(cfg, params)
    _, grad = m.loss(T._cuda(T._clouds(B, P, 53)), T._cuda(targets, torch.float64), grad=True)
    grad = grad.cpu().numpy().astype(np.float64)
    m.close()
    assert np.isfinite(grad).all()
    for layers, (gap, size) in euler_gaps(np.asarray(params, np.float64), grad, K).items():
        assert gap <= 2.0 ** -6 * size, layers


@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,splits", [(33, 600, 512, 7), (64, 130, 288, 8), (64, 130, 288, 9), (448, 65, 640, 20),
                                          (449, 65, 640, 20), (128, 256, 4096, 64), (130, 1, 320, 10)])
def test_products_over_every_map_of_tiles_and_slices(ta, tb, M, N, K, splits):
    """Seven and eight row tiles, seven to nine slices and counts off eight: integers, so exact."""
    rng = np.random.default_rng(M + N + K + splits + ta)
    A, B, bias, C0 = T._gemm_case(ta, tb, M, N, K, rng, integer=True)
    got = T._run_gemm(A, B, bias, C0, ta, tb, 1, 1, splits)
    assert np.array_equal(got, T._oracle_gemm(A, B, bias, C0, ta, tb, 1, 1))
