"""Non-Cartesian products at the edges of their tiles: 128 samples and 32 per
step, 32-column steps and 128-column blocks, row passes of at most 224 rows,
image rows padded to 8 columns, the passes over TRs and coils that the
workspace holds, and a single voxel, sample or TR. Both encodings against the
oracle's direct sums; the bar is the plain path's 1e-5 relative for either
(both run the split products whose error is FP32's)."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, T, nk, coils, f16 trains, encoding
    (1, 1, 1, 1, 1, False, 0),
    (1, 40, 3, 33, 2, False, 1),
    (7, 3, 9, 31, 1, False, 0),
    (33, 33, 17, 129, 3, False, 1),
    (129, 10, 8, 40, 1, False, 0),
    (256, 2, 5, 128, 1, False, 1),
    (9, 225, 12, 65, 2, False, 0),
    (5, 449, 10, 20, 1, False, 0),
    (57, 64, 130, 32, 2, False, 0),
    (130, 97, 20, 257, 1, True, 1),
]


@pytest.mark.parametrize("nx,ny,T,nk,coils,f16,enc", CASES)
def test_products_match_oracle(oracle_lib, nx, ny, T, nk, coils, f16, enc):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    rng = np.random.default_rng(1000 * nx + ny)
    prob = I.make_problem(nx, ny, T, nk, 8, n_coils=coils, flip_deg=rng.uniform(10, 60, T))
    prob.traj = (rng.uniform(-0.5, 0.5, (T, nk)) * nx, rng.uniform(-0.5, 0.5, (T, nk)) * ny)
    th = I.iid_maps(prob.nv, seed=4, b1=rng.uniform(0.8, 1.2, prob.nv)).astype(np.float32).astype(np.float64)
    coil = I.coil_maps(nx, ny, coils).astype(np.complex64) if coils > 1 else None
    mask = (rng.uniform(size=prob.nv) > 0.2).astype(np.uint8)
    mask[0] = 1
    v, w = I.probe_vectors(prob)
    v, w = v.astype(np.float32), w.astype(np.complex64)
    tr = oracle_lib.epg(prob, th)
    co = None if coil is None else coil.astype(np.complex128)
    ref = [oracle_lib.jv(prob, th, tr, v.astype(np.float64), coil=co, mask=mask),
           oracle_lib.jhw(prob, th, tr, w.astype(np.complex128), coil=co, mask=mask),
           oracle_lib.residual(prob, th, w.astype(np.complex128), coil=co, mask=mask)[1]]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = B.Context(prob, coil=None if coil is None else dev(coil), mask=dev(mask))
    ctx.set_encoding(enc)
    if f16:
        ctx.set_train_precision(B.TRAINS_FP16)
    t = dev(th.astype(np.float32))
    ctx.linearise(t)
    got = [ctx.jv(t, dev(v), reuse=True), ctx.jhw(t, dev(w), reuse=True), ctx.residual(t, dev(w), reuse=True)[1]]
    errs = [float(np.linalg.norm(g.cpu().numpy() - r) / np.linalg.norm(r)) for g, r in zip(got, ref)]
    ctx.close()
    print(f"  {nx}x{ny} T {T} nk {nk} C {coils}: jv {errs[0]:.1e} jhw {errs[1]:.1e} residual {errs[2]:.1e}", flush=True)
    assert max(errs) <= (1e-3 if f16 else 1e-5)


@pytest.mark.parametrize("scale", [1e-30, 1e-3, 1e30])
def test_products_scale_with_their_inputs(oracle_lib, scale):
    """Directions and data far from 1 (the split operands are scaled by powers
    of two): the same products times the factor."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    rng = np.random.default_rng(5)
    prob = I.make_problem(40, 36, 16, 50, 8, flip_deg=rng.uniform(10, 60, 16))
    prob.traj = I.radial_golden(16, 50, 40, 36)
    t = torch.from_numpy(I.iid_maps(prob.nv, seed=4).astype(np.float32)).cuda()
    v, w = I.probe_vectors(prob)
    v, w = torch.from_numpy(v.astype(np.float32)).cuda(), torch.from_numpy(w.astype(np.complex64)).cuda()
    ctx = B.Context(prob)
    ctx.linearise(t)
    for f, x in ((ctx.jv, v), (ctx.jhw, w)):
        a, b = f(t, x, reuse=True), f(t, x * scale, reuse=True)
        e = float(torch.linalg.vector_norm(torch.view_as_real(b / scale - a) if a.is_complex() else b / scale - a) /
                  torch.linalg.vector_norm(torch.view_as_real(a) if a.is_complex() else a))
        assert e <= 1e-6
    # One value that is not finite reaches every sample of its TR (and only
    # those): w in the adjoint reaches every voxel.
    bad = w.clone()
    bad[0, 3, 7] = float("inf")
    assert not torch.isfinite(ctx.jhw(t, bad, reuse=True)).any(dim=0).any()
    ctx.close()
