"""EPG trains against the oracle at the edges of the kernel's forms: orders per
lane 2 to 16 with and without masked orders, groups of four, two and one TRs
with every remainder, and the automatic split over lanes. Tolerances: 1e-5 relative in FP32,
2^-11 with FP16 trains (rounding to nearest of each value, at most
half a unit of 2^-10, plus the FP32 error and values below 2^-14)."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, T, K
    (5, 3, 1, 3),
    (8, 8, 2, 8),
    (7, 9, 3, 8),
    (4, 6, 5, 9),
    (11, 3, 7, 16),
    (16, 16, 9, 16),
    (3, 3, 6, 17),
    (9, 7, 11, 32),
    (16, 12, 45, 32),
    (5, 5, 10, 33),
    (6, 7, 69, 64),
]


@pytest.mark.parametrize("nx,ny,T,K", CASES)
def test_trains_match_oracle(oracle_lib, nx, ny, T, K):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    rng = np.random.default_rng(T * 100 + K)
    prob = I.make_problem(nx, ny, T, nx, K, flip_deg=60.0 * np.abs(np.sin(0.3 * np.arange(T) + 0.2)) + 5.0)
    th = I.iid_maps(prob.nv, seed=K, b1=rng.uniform(0.8, 1.2, prob.nv)).astype(np.float32)
    ref = oracle_lib.epg(prob, th.astype(np.float64)).imag
    thd = torch.from_numpy(th).cuda()
    ctx = B.Context(prob)
    for prec, tol in ((B.TRAINS_FP32, 1e-5), (B.TRAINS_FP16, 2.0 ** -11)):
        ctx.set_train_precision(prec)
        for lanes in (0, 1, 2, 4, 8):
            ctx.set_epg_lanes(lanes)
            got = ctx.simulate(thd).cpu().numpy().astype(np.float64)
            for p in range(4):
                n = np.linalg.norm(ref[p])
                e = np.linalg.norm(got[p] - ref[p]) / n if n > 0 else np.abs(got[p]).max()
                assert e <= tol, (prec, lanes, p, e)
    ctx.close()
