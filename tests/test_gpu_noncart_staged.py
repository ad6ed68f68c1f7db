"""Non-Cartesian products where the forward stages FP32 voxel values (up to 128
columns, and with coils): one, two and four sample waves per block with every
number of row tiles, row passes, ragged columns, rows and samples, launches
split because the row exponents fill their space, partial sums of f past the
reduction buffer. Against the oracle's direct sums at the plain path's 1e-5
relative (1e-3 with FP16 trains)."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, T, nk, coils, f16 trains, encoding
    (1, 3, 300, 5, 1, False, 0),       # three launches (127 TRs of exponents each)
    (2, 5, 600, 9, 3, True, 1),
    (24, 24, 9, 48, 4, False, 1),      # one sample wave, two sample tiles
    (64, 32, 40, 500, 2, False, 0),    # sixteen sample tiles: partials in the other buffer
    (2, 20, 6, 130, 1, False, 0),      # samples past 32 per column: four waves
    (33, 47, 11, 66, 1, False, 0),     # two waves, two tiles
    (31, 128, 5, 33, 1, False, 1),     # two waves, four tiles
    (40, 96, 5, 50, 2, True, 1),       # coils: two row passes of two waves
    (61, 130, 5, 122, 1, False, 0),    # four waves, five tiles
    (61, 130, 5, 122, 4, False, 1),    # coils: four waves, two passes
    (128, 224, 3, 128, 1, False, 1),   # four waves, seven tiles
    (100, 65, 4, 101, 5, False, 0),
    (128, 129, 3, 40, 9, False, 1),
    (160, 40, 5, 40, 2, False, 0),     # wide, too few TRs to split per coil
    (24, 60, 4, 20, 1, False, 1),      # one wave, two tiles
]


def _setup(torch, oracle_lib, nx, ny, T, nk, coils, masked=True):
    rng = np.random.default_rng(7 * nx + ny)
    prob = I.make_problem(nx, ny, T, nk, 8, n_coils=coils, flip_deg=rng.uniform(10, 60, T))
    prob.traj = (rng.uniform(-0.5, 0.5, (T, nk)) * nx, rng.uniform(-0.5, 0.5, (T, nk)) * ny)
    th = I.iid_maps(prob.nv, seed=4, b1=rng.uniform(0.8, 1.2, prob.nv)).astype(np.float32).astype(np.float64)
    th[3:] *= np.exp2(rng.integers(-12, 1, (1, prob.nv)))   # rows with a range of magnitudes
    th = th.astype(np.float32).astype(np.float64)
    coil = I.coil_maps(nx, ny, coils).astype(np.complex64) if coils > 1 else None
    mask = (rng.uniform(size=prob.nv) > 0.2).astype(np.uint8)
    mask[0] = 1
    return prob, th, coil, mask


@pytest.mark.parametrize("nx,ny,T,nk,coils,f16,enc", CASES)
def test_products_match_oracle(oracle_lib, nx, ny, T, nk, coils, f16, enc):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    prob, th, coil, mask = _setup(torch, oracle_lib, nx, ny, T, nk, coils)
    v, w = I.probe_vectors(prob)
    v, w = v.astype(np.float32), w.astype(np.complex64)
    tr = oracle_lib.epg(prob, th)
    co = None if coil is None else coil.astype(np.complex128)
    f_ref, r_ref = oracle_lib.residual(prob, th, w.astype(np.complex128), coil=co, mask=mask)
    jv_ref = oracle_lib.jv(prob, th, tr, v.astype(np.float64), coil=co, mask=mask)
    jhw_ref = oracle_lib.jhw(prob, th, tr, w.astype(np.complex128), coil=co, mask=mask)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rel = lambda a, b: float(np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b))  # noqa: E731
    ctx = B.Context(prob, coil=None if coil is None else dev(coil), mask=dev(mask))
    ctx.set_encoding(enc)
    if f16:
        ctx.set_train_precision(B.TRAINS_FP16)
    t = dev(th.astype(np.float32))
    ctx.linearise(t)
    f, r = ctx.residual(t, dev(w), reuse=True)
    errs = [rel(ctx.jv(t, dev(v), reuse=True), jv_ref), rel(r, r_ref), abs(f - f_ref) / f_ref,
            rel(ctx.jhw(t, dev(w), reuse=True), jhw_ref)]
    ctx.close()
    print(f"  {nx}x{ny} T {T} nk {nk} C {coils}: " + " ".join(f"{e:.1e}" for e in errs), flush=True)
    assert max(errs) <= (1e-3 if f16 else 1e-5)


def test_values_that_are_not_finite(oracle_lib):
    """A direction that is infinite in one voxel reaches every sample; in a masked voxel, none."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    prob, th, coil, mask = _setup(torch, oracle_lib, 40, 36, 6, 50, 2)
    mask[77] = 0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = B.Context(prob, coil=dev(coil), mask=dev(mask))
    t = dev(th.astype(np.float32))
    ctx.linearise(t)
    v = dev(I.probe_vectors(prob)[0].astype(np.float32))
    ref = ctx.jv(t, v, reuse=True)
    v[0, 77] = float("inf")
    assert torch.equal(torch.view_as_real(ctx.jv(t, v, reuse=True)), torch.view_as_real(ref))
    v[0, 0] = float("inf")
    assert not torch.isfinite(torch.view_as_real(ctx.jv(t, v, reuse=True))).any()
    ctx.close()


@pytest.mark.parametrize("nx,ny,T", [(32, 32, 560), (24, 200, 250)])
def test_coils_share_the_voxel_values(nx, ny, T):
    """J v with eight coils costs clearly less than eight calls with one: the voxel
    values are made once and in one launch (2.5 and 3.1 times one coil's call; with
    values per coil, a group of TRs per launch, 7 and 9 times)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    took = {}
    for coils in (1, 8):
        prob = I.make_problem(nx, ny, T, nx, 8, n_coils=coils, flip_deg=np.full(T, 30.0))
        prob.traj = I.radial_golden(T, nx, nx, ny)
        coil = torch.from_numpy(I.coil_maps(nx, ny, coils).astype(np.complex64)).cuda() if coils > 1 else None
        ctx = B.Context(prob, coil=coil)
        t = torch.from_numpy(I.iid_maps(prob.nv, seed=4).astype(np.float32)).cuda()
        ctx.linearise(t)
        v, out = torch.randn_like(t), ctx.jv(t, t, reuse=True)
        best = float("inf")
        for _ in range(30):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(5):
                ctx.jv(t, v, reuse=True, out=out)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 5)
        took[coils] = best
        ctx.close()
    print(f"  {nx}x{ny} T {T}: 1 coil {1e3 * took[1]:.1f} us, 8 coils {1e3 * took[8]:.1f} us", flush=True)
    assert took[8] <= 5.0 * took[1]
