"""The EPG runs inside a Gauss-Newton step: the objective of the line-search
trial, which comes from the value-only kernels, against the oracle at every
count of orders per lane, and the automatic split over lanes against the
splits a caller can set.

Tolerances: the signal of FP16 trains is within 1e-3 of the oracle's normwise
and that of FP32 trains within 1e-5, so with e of either times ||d|| the
objective r^H r / 2 is within e ||r|| + e^2 / 2. The automatic split may take
up to 1.2 times the fastest one: twice the few per cent by which the rule's
estimates miss, and the runs' spread."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding
    binding.lib()
    return torch


def _problem(nx, ny, T, K):
    prob = I.make_problem(nx, ny, T, nx, K, flip_deg=60.0 * np.abs(np.sin(0.3 * np.arange(T) + 0.2)) + 5.0)
    rng = np.random.default_rng(K)
    th = I.iid_maps(prob.nv, seed=K, b1=rng.uniform(0.8, 1.2, prob.nv))
    th0 = th.copy()
    th0[0] += 0.1 * rng.standard_normal(prob.nv)
    th0[1] += 0.1 * rng.standard_normal(prob.nv)
    return prob, th, th0.astype(np.float32)


@pytest.mark.parametrize("K,lanes", [(6, 2), (13, 1), (16, 1), (16, 0), (24, 2), (32, 2), (32, 4), (50, 4), (64, 4),
                                     (64, 8)])
def test_trial_objective_matches_oracle(torch_gpu, oracle_lib, K, lanes):
    torch = torch_gpu
    from paper_1904_13244_amd import binding as B
    prob, th, th0 = _problem(13, 11, 40, K)
    d = oracle_lib.signal(prob, th, oracle_lib.epg(prob, th, tangents=False)).astype(np.complex64)
    ctx = B.Context(prob)
    ctx.set_epg_lanes(lanes)
    dd = torch.from_numpy(d).cuda()
    for prec, tol in ((B.TRAINS_FP32, 1e-5), (B.TRAINS_FP16, 1e-3)):
        ctx.set_train_precision(prec)
        thd = torch.from_numpy(th0).cuda()
        rep = ctx.gn_step(thd, dd, 6, 0b11011, I.GN_LO, I.GN_HI)
        assert rep.accepted
        f, r = oracle_lib.residual(prob, thd.cpu().numpy().astype(np.float64), d.astype(np.complex128))
        e = tol * np.linalg.norm(d)
        print(f"  prec {prec}: f1 {rep.f1:.6e} oracle {f:.6e} f0 {rep.f0:.3e}")
        assert abs(rep.f1 - f) <= e * np.linalg.norm(r) + 0.5 * e * e
    ctx.close()


@pytest.mark.parametrize("K,n,param_mask", [(8, 320, 0b11111), (16, 181, 0b11111), (32, 224, 0b11011),
                                            (64, 200, 0b11111)])
def test_automatic_lanes_are_near_the_fastest(torch_gpu, K, n, param_mask):
    torch = torch_gpu
    from paper_1904_13244_amd import binding as B
    prob, _, th0 = _problem(n, n, 128, K)
    ctx = B.Context(prob)
    thd = torch.from_numpy(th0).cuda()
    data = torch.zeros(ctx.data_shape, dtype=torch.complex64, device="cuda")
    ctx.profile_select(["epg"])
    times = {}
    for _ in range(6):   # the splits in turn, the fastest run of each
        for lanes in (0, 1, 2, 4, 8):
            ctx.set_epg_lanes(lanes)
            ctx.profile(True)
            ctx.gn_step(thd.clone(), data, 1, param_mask, I.GN_LO, I.GN_HI, n_ls_max=1)
            launches, ms = ctx.profile_read()["epg"]
            ctx.profile(False)
            times[lanes] = min(times.get(lanes, 1e9), ms / launches)
    ctx.close()
    print("  " + ", ".join(f"{l}: {1e3 * t:.0f} us" for l, t in times.items()))
    assert times[0] <= 1.2 * min(times[l] for l in (1, 2, 4, 8))
