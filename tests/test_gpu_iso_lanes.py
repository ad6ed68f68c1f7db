"""Isochromat trains against the oracle for each split over lanes (16, 8 and 4
per voxel, chosen by voxels and isochromats), slots partly filled, two and
three tangents; 1e-5 relative, the plain path's tolerance."""
import numpy as np
import pytest

from test_gpu_iso import _balanced, _dev, _rel, torch_gpu  # noqa: F401

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n_iso", [(5, 3, 5), (7, 9, 17), (128, 130, 16), (96, 97, 9), (200, 180, 16), (31, 33, 4)])
def test_trains_match_oracle(torch_gpu, oracle_lib, nx, ny, n_iso):  # noqa: F811
    torch = torch_gpu
    from paper_1904_13244_amd.binding import Context
    prob, th = _balanced(nx=nx, ny=ny, n_tr=9, n_read=nx, n_iso=n_iso)
    ora = oracle_lib.epg(prob, th)
    ctx = Context(prob)
    got = ctx.simulate(_dev(torch, th, torch.float32)).cpu().numpy().astype(np.float64)
    assert max(_rel(got[p], ora[p].imag) for p in range(4)) <= 1e-5
    data = oracle_lib.signal(prob, th, ora)
    th0 = th.copy()
    th0[0] += 0.02
    ref, rep_o = oracle_lib.gn_step(prob, th0, data, n_cg=2, param_mask=0b11011, lo=I.GN_LO, hi=I.GN_HI)
    thd = _dev(torch, th0, torch.float32)
    rep = ctx.gn_step(thd, _dev(torch, data, torch.complex64), 2, 0b11011, I.GN_LO, I.GN_HI)
    ctx.close()
    assert rep.t == rep_o.t and _rel(thd.cpu().numpy().astype(np.float64), ref) <= 1e-5
