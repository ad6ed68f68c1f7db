"""The automatic tile of the fused inference: the same bits as 64-voxel
workgroups on both sides of each change of the tile."""
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu


def _net(torch, n_tr):
    from paper_1904_13244_amd.binding import Surrogate
    net = Surrogate(n_tr, 256, 4, 64)
    net.set_scaling(I.SURR_LO, I.SURR_HI, (0.12, 0.08, 0.06, 0.05))
    net.set_params(torch.from_numpy(I.mlp_init_params(n_tr, width=256, depth=4, seed=3)).float().cuda())
    return net


@pytest.mark.parametrize("n", [16384, 16385, 32768, 32769, 53248, 53249, 65536, 65537, 98305])
def test_every_tile_gives_the_same_bits(n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    net = _net(torch, 24)
    th = torch.from_numpy(I.surrogate_samples(n, seed=4)).float().cuda()
    got = net.predict(th).clone()
    for tile in (-64, 64, 32):
        net.set_infer_tile(tile)
        assert torch.equal(got, net.predict(th)), tile
    net.close()
