"""The Cartesian y-stages with receive coils against the oracle at the edges of
their tiles: coil slots 2, 4, 8 and 16 with unused ones, columns in tiles of 64
and of 32 with ragged last ones, several row blocks of the adjoint, several row
slabs of the forward (few TRs) whose parts are summed, more rows than one slab
may hold, and TRs off the multiple of a block's.

Tolerances, those of the one-coil paths: trains and products 1e-5 normwise with
FP32 trains and 1e-3 with FP16 trains; a Gauss-Newton step of three CG
iterations 1e-4 and 1e-3 of the maps."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, coils, TRs, mask
    (64, 17, 2, 33, False),
    (61, 33, 3, 5, True),
    (33, 65, 4, 7, False),
    (70, 130, 4, 9, True),
    (64, 130, 5, 6, True),
    (40, 66, 8, 17, False),
    (128, 33, 8, 3, False),
    (33, 17, 9, 21, True),
    (64, 97, 12, 5, False),
    (70, 65, 16, 4, True),
    (61, 18, 16, 67, False),
    (3, 1030, 2, 4, True),
    (1, 33, 8, 40, False),
]


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("nx,ny,coils,T,masked", CASES)
def test_coil_products_match_oracle(oracle_lib, nx, ny, coils, T, masked, f16):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    dev = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt).contiguous()
    rng = np.random.default_rng(nx * 1000 + ny + coils)
    prob = I.make_problem(nx, ny, T, nx + 5, 6, n_coils=coils, flip_deg=rng.uniform(10.0, 70.0, T),
                          ky_line=rng.integers(0, ny, T))
    th = I.iid_maps(prob.nv, seed=coils, b1=rng.uniform(0.8, 1.2, prob.nv)).astype(np.float32).astype(np.float64)
    th0 = th.copy()
    th0[0] += 0.1 * rng.standard_normal(prob.nv)
    th0[1] += 0.1 * rng.standard_normal(prob.nv)
    th0 = th0.astype(np.float32).astype(np.float64)
    coil = I.coil_maps(nx, ny, coils)
    mask = (rng.uniform(size=prob.nv) > 0.2).astype(np.uint8) if masked else None
    ora = oracle_lib.epg(prob, th0)
    kw = dict(coil=coil, mask=mask)
    d = oracle_lib.signal(prob, th, oracle_lib.epg(prob, th, tangents=False), **kw).astype(np.complex64)
    d64 = d.astype(np.complex128)
    v, w = I.probe_vectors(prob)
    tol, tol_gn = (1e-3, 1e-3) if f16 else (1e-5, 1e-4)

    ctx = B.Context(prob, coil=dev(coil, torch.complex64), mask=None if mask is None else dev(mask, torch.uint8))
    ctx.set_train_precision(B.TRAINS_FP16 if f16 else B.TRAINS_FP32)
    thd, dd = dev(th0, torch.float32), dev(d, torch.complex64)
    ctx.linearise(thd)
    jv = ctx.jv(thd, dev(v, torch.float32), reuse=True).cpu().numpy().astype(np.complex128)
    jhw = ctx.jhw(thd, dev(w, torch.complex64), reuse=True).cpu().numpy().astype(np.float64)
    f, r = ctx.residual(thd, dd)
    f_ref, r_ref = oracle_lib.residual(prob, th0, d64, **kw)
    e = (_rel(jv, oracle_lib.jv(prob, th0, ora, v, **kw)), _rel(jhw, oracle_lib.jhw(prob, th0, ora, w, **kw)),
         float(np.linalg.norm(r.cpu().numpy() - r_ref) / np.linalg.norm(d64)))
    print(f"  jv {e[0]:.2e} jhw {e[1]:.2e} residual {e[2]:.2e}", flush=True)
    assert max(e) <= tol
    for param_mask in (0b11011, 0b11111):
        t_ora, rep_o = oracle_lib.gn_step(prob, th0, d64, n_cg=3, param_mask=param_mask, lo=I.GN_LO, hi=I.GN_HI, **kw)
        t_gpu = thd.clone()
        rep = ctx.gn_step(t_gpu, dd, 3, param_mask, I.GN_LO, I.GN_HI)
        eg = _rel(t_gpu.cpu().numpy().astype(np.float64), t_ora)
        print(f"  gn {param_mask:05b}: maps {eg:.2e}, t {rep.t}/{rep_o.t}", flush=True)
        assert rep.accepted == rep_o.accepted and rep.t == rep_o.t
        assert eg <= tol_gn
    ctx.close()
