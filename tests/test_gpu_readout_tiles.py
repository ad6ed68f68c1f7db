"""Readout products against the oracle where the forward's lanes cross columns
and TR pairs and the adjoint's TR chunks are chosen by workgroups: one and 256
columns, an odd TR count, fewer TRs than chunks, tall and wide images. The
plain path's tolerance, 1e-5 relative."""
import dataclasses

import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I
from test_gpu_readout import _dev, _maps, _rel, torch_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,T", [(1, 7, 3), (256, 64, 21), (3, 200, 33), (65, 1, 5), (200, 100, 12)])
def test_products_match_oracle(torch_gpu, oracle_lib, nx, ny, T):  # noqa: F811
    torch = torch_gpu
    from paper_1904_13244_amd.binding import Context
    rng = np.random.default_rng(nx * 7 + T)
    prob = I.make_problem(nx, ny, T, max(nx, 16), 8, tr=0.008, te=0.004, flip_deg=rng.uniform(5, 60, T),
                          ky_line=rng.integers(0, ny, T))
    prob = dataclasses.replace(prob, dwell=1 / 85.6e3, db0=rng.uniform(-150.0, 150.0, prob.nv))
    th = _maps(prob, rng, 3)
    mask = (rng.uniform(size=prob.nv) > 0.2).astype(np.uint8)
    mask[0] = 1
    ctx = Context(prob, mask=_dev(torch, mask, torch.uint8))
    ora = oracle_lib.epg(prob, th)
    v, w = I.probe_vectors(prob)
    thd = _dev(torch, th, torch.float32)
    jv = ctx.jv(thd, _dev(torch, v, torch.float32)).cpu().numpy()
    g = ctx.jhw(thd, _dev(torch, w, torch.complex64)).cpu().numpy()
    ctx.close()
    assert _rel(jv, oracle_lib.jv(prob, th, ora, v, mask=mask)) <= 1e-5
    ref = oracle_lib.jhw(prob, th, ora, w, mask=mask)
    for p in range(5):
        assert _rel(g[p], ref[p]) <= 1e-5, p
