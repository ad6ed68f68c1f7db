"""Surrogate products and inference against the FP64 network oracle at the edges
of the kernels' forms: splits over K with few and many tiles, the 128 x 128
tiles of the output layer, targets that start off a 16-byte boundary, and
whole-network tiles of 128 and 208 voxels with ragged ends. Tolerances are those
of the network's BF16 roundings: 2e-2 for outputs and loss, 3e-2 and cosine
0.999 per gradient block."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I
from test_gpu_mlp import _blocks, _case, _oracle_weights, _params, torch_gpu  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [
    # n_tr, width, depth, batch, first column (ld = batch + column + 3)
    (8, 64, 2, 64, 0),
    (40, 192, 3, 576, 1),
    (16, 320, 2, 1024, 0),
    (136, 128, 1, 832, 5),
    (1120, 64, 2, 1024, 0),
]


@pytest.mark.parametrize("n_tr,width,depth,batch,col", SIZES)
def test_gradients_match_oracle(torch_gpu, n_tr, width, depth, batch, col):  # noqa: F811
    torch = torch_gpu
    from oracle import mlp as M
    from paper_1904_13244_amd.binding import Surrogate
    flat = _params(n_tr, width, depth, seed=3)
    theta, trains, scale = _case(n_tr, width, depth, batch, seed=5)
    wide = np.zeros((4, n_tr, batch + col + 3), dtype=np.float32)
    wide[:, :, col:col + batch] = trains
    wth = np.zeros((3, batch + col + 3), dtype=np.float32)
    wth[:, col:col + batch] = theta[:3]
    net = Surrogate(n_tr, width, depth, batch)
    net.set_scaling(I.SURR_LO, I.SURR_HI, scale)
    net.set_params(torch.from_numpy(flat).cuda())
    loss, g = net.gradients(torch.from_numpy(wth).cuda(), torch.from_numpy(wide).cuda(), col=col)
    g = g.cpu().numpy().astype(np.float64)
    net.close()
    x = M.normalise_inputs(theta.astype(np.float64), I.SURR_LO, I.SURR_HI)
    tgt = M.scaled_targets(trains.astype(np.float64), scale.astype(np.float64))
    loss_o, g_o = M.loss_and_grad(_oracle_weights(flat, n_tr, width, depth), x, tgt, n_tr, width, depth)
    assert abs(loss - loss_o) < 2e-2 * loss_o
    for s, sl in _blocks(n_tr, width, depth):
        a, b = g[sl], g_o[sl]
        e = np.linalg.norm(a - b) / np.linalg.norm(b)
        assert e < 3e-2 and a @ b > 0.999 * np.linalg.norm(a) * np.linalg.norm(b), (s, e)


@pytest.mark.parametrize("n", [16384, 16385, 32771, 33000])
def test_predict_matches_oracle(torch_gpu, n):  # noqa: F811
    torch = torch_gpu
    from oracle import mlp as M
    from paper_1904_13244_amd.binding import Surrogate
    n_tr, width, depth = 24, 256, 3
    flat = _params(n_tr, width, depth, seed=7)
    theta, _, scale = _case(n_tr, width, depth, n, seed=9)
    net = Surrogate(n_tr, width, depth, 64)
    net.set_scaling(I.SURR_LO, I.SURR_HI, scale)
    net.set_params(torch.from_numpy(flat).cuda())
    got = net.predict(torch.from_numpy(theta[:3].copy()).cuda()).cpu().numpy().astype(np.float64)
    net.close()
    x = M.normalise_inputs(theta.astype(np.float64), I.SURR_LO, I.SURR_HI)
    y, _ = M.forward(_oracle_weights(flat, n_tr, width, depth), x, n_tr, width, depth)
    ref = y[4 * n_tr:].reshape(4, n_tr, n) * scale.astype(np.float64)[:, None, None]
    assert np.linalg.norm(got - ref) < 2e-2 * np.linalg.norm(ref)
    assert np.abs(got - ref).max() < 5e-2 * np.abs(ref).max()
