"""Where the fused kernels of the warm-start network (mlp_fused.h) are held to
more than the network's parity bars: SiLU and its derivative where the sigmoid
is below the smallest normal number, and the loss of a large batch."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def _net(n_in, depth, n_out, max_batch, flat):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_14425_amd import rcx
    net = rcx.Mlp(n_in, 128, depth, n_out, max_batch=max_batch)
    net.set_params(flat)
    return net, torch


@pytest.mark.parametrize("z", [-87.0, -88.0, -88.7, 87.0])
def test_silu_where_the_sigmoid_is_tiny(z):
    """One hidden layer at the pre-activation z: silu(-88) = -5e-37, and its
    derivative, are normal numbers though the sigmoid is not; output weights of
    1e35 bring them to order 1 (1e36 takes dL/dh past the FP32 range at -87). Five roundings to BF16 lie between the exact
    gradient and this one: 5 x 2^-9."""
    w_out = 1e35 if z < 0 else 1.0
    flat = np.concatenate([np.zeros(128), np.full(128, z), np.full(128, w_out), [0.0]]).astype(np.float32)
    print(f"[gpu] silu at {z}", flush=True)
    net, torch = _net(1, 1, 1, 1, flat)
    x, yr = np.ones((1, 1), np.float32), np.zeros((1, 1), np.float32)
    xt, yt = torch.from_numpy(x).cuda(), torch.from_numpy(yr).cuda()
    y = net.forward(xt).cpu().numpy()
    _, g = net.gradients(xt, yt)
    g = g.cpu().numpy().astype(np.float64)
    net.close()
    params = omlp.unflatten(flat.astype(np.float64), 1, 128, 1, 1)
    yo, _, _ = omlp.forward(params, x.astype(np.float64))
    _, go = omlp.loss_and_grads(params, x.astype(np.float64), yr.astype(np.float64))
    gb, go = g[128:256], go[0][1].ravel()
    print(y, yo, gb[0], go[0])
    assert np.abs(y - yo).max() <= 2 * 2.0**-9 * np.abs(yo).max()
    assert np.abs(gb - go).max() <= 5 * 2.0**-9 * np.abs(go).max()


@pytest.mark.parametrize("batch", [1000, 1 << 20])
def test_loss_of_equal_errors(batch):
    """A network of zeros against a constant: every squared error is the same
    FP32 number c, so the mean is c, to the rounding of 1 / (batch x outputs)
    and of the result (2^-23) when the sums are exact or in FP64."""
    n_out = 4
    flat = np.zeros(6 * 128 + 128 + 128 * n_out + n_out, np.float32)
    print(f"[gpu] loss of {batch}", flush=True)
    net, torch = _net(6, 1, n_out, batch, flat)
    yr = torch.full((batch, n_out), 1.1, device="cuda", dtype=torch.float32)
    loss, _ = net.gradients(torch.zeros((batch, 6), device="cuda"), yr)
    net.close()
    c = np.float32(1.1) * np.float32(1.1)
    print(loss, c)
    assert abs(float(loss) - float(c)) <= 2.0**-23 * float(c)
