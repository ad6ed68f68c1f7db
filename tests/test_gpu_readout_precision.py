"""J^H w of a readout-dynamics context does not lose accuracy with the length of
its TR chunks: the call is linear in w, so its result is compared with the FP64
sum of calls on 16 TRs at a time, whose sums over TRs are short. The bound is the
difference that chunks of 125 TRs in one sum showed (chunks of 224: 2.8e-7)."""
import numpy as np
import pytest

from paper_1904_13244_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_long_chunks_keep_their_accuracy():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_13244_amd import binding as B
    nx = ny = 224
    T, nk = 1120, 448
    prob = I.make_problem(nx, ny, T, nk, 8, flip_deg=40.0 * np.abs(np.sin(0.02 * np.arange(T))) + 5.0)
    prob.dwell = 1.0 / 85.6e3
    prob.db0 = np.linspace(-100.0, 100.0, prob.nv).astype(np.float32)
    ctx = B.Context(prob)
    t = torch.from_numpy(I.iid_maps(prob.nv, seed=4).astype(np.float32)).cuda()
    ctx.linearise(t)
    g = torch.Generator("cuda").manual_seed(3)
    w = torch.randn(ctx.data_shape, dtype=torch.complex64, device="cuda", generator=g)
    whole = ctx.jhw(t, w, reuse=True).double()
    parts, part = torch.zeros_like(whole), torch.zeros_like(w)
    for n in range(0, T, 16):
        part.zero_()
        part[:, n:n + 16] = w[:, n:n + 16]
        parts += ctx.jhw(t, part, reuse=True).double()
    ctx.close()
    e = float(torch.linalg.vector_norm(whole - parts) / torch.linalg.vector_norm(parts))
    print(f"  {e:.3e}", flush=True)
    assert e <= 2.197e-7
