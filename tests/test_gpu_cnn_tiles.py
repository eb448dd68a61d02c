"""The restoration network at the edges of its kernels' tiles: the forward
pass's 14 x 26 output tile and the backward pass's 16 x 32 block (one pixel,
exactly one tile, one pixel more and less in each direction, several tiles),
against the float64 oracle; the activations it keeps are checked through the
gradients.

Tolerances: as in test_gpu_cnn, what differs is a bfloat16 rounding that flips
(2^-8 relative) next to a boundary.  One flipped activation reaches up to 7 x 7
pixels, which is any fraction of an image this small, so every output is held
to the bound for single values (2e-3 of the output range); a gradient sums
32 signals of every pixel, of which four may be off by 2^-8 (relative L2
4 2^-8 / sqrt(32 pixels)) where that is more than test_gpu_cnn's 2e-4."""
import numpy as np
import pytest
import torch

from oracle import cnn as ocnn
from test_gpu_cnn import _case, _dev_t, _dev_x

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 14, 26), (2, 13, 25), (1, 15, 27), (3, 28, 53), (1, 5, 80),
                                   (1, 60, 3), (1, 16, 32), (2, 17, 33), (1, 31, 63)])
def test_forward_and_gradients_at_tile_edges(shape):
    from paper_2208_10859_amd import cnn
    x, t, params = _case(70 + shape[1], shape)
    net = cnn.Net(int(np.prod(shape)))
    net.set_params(cnn.flatten(params))
    z = torch.full(shape + (4,), 9.0, dtype=torch.float32, device="cuda")
    z2 = torch.full(shape + (4,), 5.0, dtype=torch.float32, device="cuda")
    xd = _dev_x(x)
    net.infer(xd, z2)
    net.forward(xd, z)
    loss = net.loss_grad(_dev_t(t))
    grads = torch.full((cnn.param_count(),), 3.0, dtype=torch.float32, device="cuda")
    net.backward(grads)
    torch.cuda.synchronize()
    assert torch.equal(z, z2)
    got = z.cpu().numpy()
    _, want, _ = ocnn.forward(x, params, round_acts=True)
    assert np.all(got[..., 3] == 0)
    err = np.abs(got[..., :3] - want)
    scale = max(1.0, float(np.abs(want).max()))
    assert err.max() <= 2e-3 * scale
    want_loss, wg = ocnn.loss_and_grads(x, t, params, round_acts=True)
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    for k, (g, w) in enumerate(zip(cnn.unflatten(grads.cpu().numpy()), wg)):
        rel = np.linalg.norm(g - w) / max(np.linalg.norm(w), 1e-12)
        assert rel <= max(2e-4, 4 * 2.0 ** -8 / np.sqrt(32 * np.prod(shape))), (k, rel)


def test_training_steps_leave_the_matrices_of_their_parameters():
    """Adam rounds each parameter into the convolutions' matrices: after a few
    steps the forward pass and the gradients are those of a new network given
    the same parameters, bit for bit."""
    from paper_2208_10859_amd import cnn
    shape = (1, 20, 40)
    x, t, params = _case(91, shape)
    xd, td = _dev_x(x), _dev_t(t)
    net, fresh = cnn.Net(800), cnn.Net(800)
    net.set_params(cnn.flatten(params))
    for s in range(1, 4):
        net.train_step(xd, td, 1e-2, s)
    got = net.get_params()
    assert np.abs(got - cnn.flatten(params)).max() > 5e-3
    fresh.set_params(got)
    out = []
    for k in (net, fresh):
        z = torch.zeros(shape + (4,), dtype=torch.float32, device="cuda")
        g = torch.zeros(cnn.param_count(), dtype=torch.float32, device="cuda")
        k.forward(xd, z)
        k.loss_grad(td)
        k.backward(g)
        out.append((z.cpu(), g.cpu()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("shape", [(1, 289, 449), (601, 5, 7)])
def test_gradients_of_several_blocks_per_workgroup(shape):
    """More than 256 blocks: a workgroup of the backward kernel takes two (285
    blocks) or three (601) in turn, the last one of them a single block, and hands
    each block's first-layer signals over in LDS once more; the first shape has
    more pixels than the loss kernel takes in one stride.  test_gpu_cnn's
    tolerances."""
    from paper_2208_10859_amd import cnn
    x, t, params = _case(17 + shape[0], shape)
    net = cnn.Net(int(np.prod(shape)))
    net.set_params(cnn.flatten(params))
    net.forward(_dev_x(x))
    loss = net.loss_grad(_dev_t(t))
    grads = torch.full((cnn.param_count(),), 3.0, dtype=torch.float32, device="cuda")
    net.backward(grads)
    want_loss, wg = ocnn.loss_and_grads(x, t, params, round_acts=True)
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    for k, (g, w) in enumerate(zip(cnn.unflatten(grads.cpu().numpy()), wg)):
        rel = np.linalg.norm(g - w) / max(np.linalg.norm(w), 1e-12)
        assert rel <= 2e-4, (k, rel)
