"""The RF rotation's sines: after an ideal inversion one TR records
sin(B1 alpha) E2(TE), here with flip angles around half a turn, where the sine
itself is small and an error of the angle shows whole.

Bound: the angle B1 alpha in FP32 would be off by half a unit of its last place
(2^-23 in [2, 4), 2^-22 in [4, 8)), which moves the sine by as much times
|cos|; sine and cosine of the half angle are good to 2 units each, their
product, its relaxation and the stored value to half a unit each, 8 units of
2^-24 together, of |sin|."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flip", [150.0, 178.0, 200.0, 300.0])
@pytest.mark.parametrize("K,lanes", [(6, 1), (6, 4), (16, 1), (16, 2), (32, 8)])
def test_sines_around_half_a_turn(flip, K, lanes):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    prob = I.make_problem(64, 64, 1, 64, K, flip_deg=np.array([flip]), t_inv=0.0)
    rng = np.random.default_rng(int(flip))
    th = I.iid_maps(prob.nv, seed=3, b1=rng.uniform(0.9, 1.1, prob.nv)).astype(np.float32)
    th[1] = 0.5
    ctx = B.Context(prob)
    ctx.set_epg_lanes(lanes)
    got = ctx.simulate(torch.from_numpy(th).cuda())[0, 0].cpu().numpy().astype(np.float64)
    ctx.close()
    a = th[2].astype(np.float64) * float(np.float32(np.deg2rad(flip)))
    want = np.sin(a) * np.exp(-prob.te * np.exp(-0.5))
    got = got * np.sign((got * want).sum())
    ulp = np.spacing(a.astype(np.float32)).astype(np.float64)
    err = np.abs(got - want) / (0.5 * ulp * np.abs(np.cos(a)) + 8.0 * 2.0 ** -24 * np.abs(np.sin(a)))
    print(f"  worst {err.max():.2f} of the bound, abs {np.abs(got - want).max():.2e}")
    assert err.max() <= 1.0
