"""Timing cases of the library's public calls, over the sizes and options it is used with.

A case is a dict of plain values; ``listed`` gives the fixed ones, ``draw`` one more of the same
ranges. ``prepare`` makes what a program holds before the call (inputs on the GPU, a bound context
or network), ``run`` is one pass through the public entry points, ``exact`` the same outputs from
FP64 torch code that shares nothing with the library, and ``work`` the bytes and operations a pass
cannot do without.

Kinds of pass:
  gn        one inexact Gauss-Newton step from a start near the truth on noisy data: the unit of
            every reconstruction (linearisation, gradient, CG, line search);
  gradient  residual, objective and gradient at a new theta: what a caller's own optimiser asks for;
  products  J v and Re(J^H w) on a cached linearisation: a caller's own Krylov solver;
  network   the surrogate's trains for an image's voxels;
  training  loss gradient of one mini-batch of the surrogate.
"""
import math

import numpy as np
import torch

from paper_1904_13244_amd import binding as B
from paper_1904_13244_amd import inputs as I

DEV = "cuda"
ENC = {"fp32": B.ENC_FP32, "split_bf16": B.ENC_SPLIT_BF16}
SURR_SCALE = (0.12, 0.08, 0.06, 0.05)   # head scales of the order of the trains' RMS values
SNR = 50.0


def _case(name, kind, nx, ny, n_tr, n_read, n_states, **kw):
    c = {"name": name, "kind": kind, "nx": nx, "ny": ny, "n_tr": n_tr, "n_read": n_read, "n_states": n_states,
         "coils": 1, "enc": "fp32", "f16": False, "radial": False, "readout": False, "n_iso": 0, "n_cg": 0,
         "fit_b1": True, "masked": False}
    c.update(kw)
    return c


def listed():
    return [
        # The small workload of the tests and of a first try: launches and latency count.
        _case("gn_32", "gn", 32, 32, 128, 32, 16, n_cg=10, fit_b1=False),
        # One objective and gradient on a small ragged grid, the balanced sequence's isochromat model.
        _case("gradient_67x53_iso", "gradient", 67, 53, 210, 97, 16, n_iso=16),
        # The 128 x 128 phantom reconstruction (B1 known, head mask).
        _case("gn_128", "gn", 128, 128, 1024, 256, 32, n_cg=20, fit_b1=False, masked=True),
        # The 1 mm in-plane benchmark reconstruction, plain FP32 form, all parameters fitted.
        _case("gn_224", "gn", 224, 224, 1120, 448, 32, n_cg=20),
        # The same with the reduced-precision options: FP16 trains and the split-BF16 contraction.
        _case("gn_224_reduced", "gn", 224, 224, 1120, 448, 32, n_cg=20, f16=True, enc="split_bf16"),
        # The eight-coil reconstruction in its reduced form.
        _case("gn_256_coils", "gn", 256, 256, 1280, 512, 32, n_cg=30, coils=8, f16=True, enc="split_bf16", masked=True),
        # A caller's own solver on the benchmark workload: both products, trains cached.
        _case("products_224", "products", 224, 224, 1120, 448, 32),
        # Golden-angle radial sampling at the same size.
        _case("products_224_radial", "products", 224, 224, 1120, 448, 32, radial=True),
        # A smaller ragged radial scan with four coils, split-BF16.
        _case("products_101x90_radial_coils", "products", 101, 90, 377, 203, 24, radial=True, coils=4, enc="split_bf16"),
        # T2 decay and off-resonance during each readout.
        _case("products_224_readout", "products", 224, 224, 1120, 448, 32, readout=True, enc="split_bf16"),
        # The learned surrogate: trains of the benchmark image, and one training batch of it.
        _case("network_224", "network", 224, 224, 1120, 224, 1),
        _case("training_4096", "training", 4096, 1, 1120, 4096, 32),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["gn", "gn", "gn_coils", "gradient", "products", "radial", "radial", "readout", "network",
                       "training"])
    if kind == "training":
        c = _case("", kind, 64 * _log_int(rng, 8, 64), 1, 8 * _log_int(rng, 16, 140), 0, rng.choice([16, 24, 32]))
        c["n_read"] = c["nx"]
    elif kind == "network":
        c = _case("", kind, _log_int(rng, 32, 224), _log_int(rng, 32, 224), 8 * _log_int(rng, 16, 140), 0, 1)
        c["n_read"] = c["nx"]
    else:
        coils = rng.choice([2, 4, 8]) if kind == "gn_coils" else 1
        if kind == "radial":
            coils = rng.choice([1, 1, 4])
        top = 128 if coils > 1 and kind == "radial" else 224
        nx, ny = _log_int(rng, 24, top), _log_int(rng, 24, top)
        c = _case("", kind, nx, ny, _log_int(rng, 64, 1120 if coils == 1 else 560),
                  rng.randint(nx, 2 * nx), rng.choice([12, 16, 24, 32]), coils=coils,
                  enc=rng.choice(["fp32", "split_bf16"]), f16=rng.random() < 0.4, fit_b1=rng.random() < 0.6,
                  masked=rng.random() < 0.5)
        if kind in ("gn", "gn_coils"):
            c.update(kind="gn", n_cg=rng.randint(5, 20))
        elif kind == "gradient":
            c.update(n_iso=rng.choice([0, 8, 16]))
        elif kind == "radial":
            c.update(kind="products", radial=True)
        elif kind == "readout":
            c.update(kind="products", readout=True)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
class _Inputs:
    """Problem and arrays of a case, from the seed alone."""

    def __init__(self, case, seed):
        nx, ny, nt = case["nx"], case["ny"], case["n_tr"]
        rng = np.random.default_rng(seed)
        self.case = case
        small = min(nx, ny) < 48
        flips = I.flips_config1(nt) if small else I.flips_sin2_sweeps(nt, ny, seed=seed)
        pr = I.make_problem(nx, ny, nt, case["n_read"], case["n_states"], n_coils=case["coils"], flip_deg=flips)
        if case["n_iso"]:
            pr.iso = I.slice_profile_gaussian(case["n_iso"])
            pr.rf_phase = I.balanced_phases(nt)
        if case["radial"]:
            pr.traj = I.radial_golden(nt, case["n_read"], nx, ny)
        self.pr = pr
        if case["kind"] in ("training", "network"):
            self.theta = torch.from_numpy(I.surrogate_samples(pr.nv, seed=seed).astype(np.float32)).to(DEV)
            self.params = torch.from_numpy(I.mlp_init_params(nt, seed=seed).astype(np.float32)).to(DEV)
            if case["kind"] == "training":
                self.trains = epg_trains(pr, self.theta.double(), True).float().contiguous()
            return
        if small:
            th, head = I.iid_maps(pr.nv, seed=seed, b1=rng.uniform(0.8, 1.2, pr.nv)), np.ones(pr.nv, dtype=bool)
        else:
            th, head = I.brain_phantom(nx, ny, seed=seed, b1_range=(0.8, 1.2))
        if case["kind"] == "gn" and not case["fit_b1"]:
            th[2] = 1.0
        if case["readout"]:
            pr.dwell = 1.0 / 85.6e3
            y, x = np.meshgrid(np.linspace(-1, 1, ny), np.linspace(-1, 1, nx), indexing="ij")
            pr.db0 = (150.0 * (0.6 * x + 0.3 * y * y - 0.1 * x * y)).reshape(-1).astype(np.float32)
            self.db0 = torch.from_numpy(pr.db0).to(DEV)
        self.theta = torch.from_numpy(th.astype(np.float32)).to(DEV)
        self.mask = torch.from_numpy(head.astype(np.uint8)).to(DEV) if case["masked"] else None
        self.coil = None
        if case["coils"] > 1:
            self.coil = torch.from_numpy(I.coil_maps(nx, ny, case["coils"], seed=seed).astype(np.complex64)).to(DEV)
        if case["kind"] == "products":
            v, w = I.probe_vectors(pr, seed=seed)
            self.v = torch.from_numpy(v.astype(np.float32)).to(DEV)
            self.w = torch.from_numpy(w.astype(np.complex64)).to(DEV)
            return
        s = Model(self, self.theta.double(), tangents=False).signal()
        n = torch.from_numpy(I.unit_noise(pr, seed=seed)).to(DEV)
        n *= torch.linalg.vector_norm(s) / (SNR * torch.linalg.vector_norm(n))
        self.data = (s + n).to(torch.complex64).contiguous()
        start = th.copy()
        start[:2] += 0.1 * rng.standard_normal((2, pr.nv))
        if case["fit_b1"]:
            start[2] += 0.02 * rng.standard_normal(pr.nv)
        start[3:] *= 1.0 + 0.05 * rng.standard_normal(pr.nv)
        self.start = torch.from_numpy(start.astype(np.float32)).to(DEV)

    @property
    def param_mask(self):
        return 0b11111 if self.case["fit_b1"] else 0b11011


def prepare(case, seed):
    q = _Inputs(case, seed)
    if case["kind"] in ("training", "network"):
        q.net = B.Surrogate(case["n_tr"], batch=case["nx"] if case["kind"] == "training" else 4096)
        q.net.set_scaling(I.SURR_LO, I.SURR_HI, SURR_SCALE)
        q.net.set_params(q.params)
        return q
    q.ctx = B.Context(q.pr, coil=q.coil, mask=q.mask)
    q.ctx.set_encoding(ENC[case["enc"]])
    q.ctx.set_train_precision(B.TRAINS_FP16 if case["f16"] else B.TRAINS_FP32)
    if case["kind"] == "products":
        q.ctx.linearise(q.theta)
    return q


def run(q):
    kind = q.case["kind"]
    if kind == "gn":
        theta = q.start.clone()   # the step updates theta in place
        rep = q.ctx.gn_step(theta, q.data, q.case["n_cg"], q.param_mask, I.GN_LO, I.GN_HI)
        return {"theta": theta, "f0": rep.f0, "f1": rep.f1, "gnorm": rep.gnorm}
    if kind == "gradient":
        f, r = q.ctx.residual(q.start, q.data)
        return {"f": f, "r": r, "g": q.ctx.jhw(q.start, r, reuse=True)}
    if kind == "products":
        return {"jv": q.ctx.jv(q.theta, q.v, reuse=True), "jhw": q.ctx.jhw(q.theta, q.w, reuse=True)}
    if kind == "network":
        return q.net.predict(q.theta)
    loss, grad = q.net.gradients(q.theta, q.trains)
    return {"loss": loss, "grad": grad}


def work(case):
    nv, nt, nk, c = case["nx"] * case["ny"], case["n_tr"], case["n_read"], case["coils"]
    kind = case["kind"]
    if kind in ("training", "network"):
        mac = nv * (3 * 256 + 3 * 256 * 256 + (8 if kind == "training" else 4) * nt * 256)
        par = 4 * (3 * 256 + 256 + 3 * (256 * 256 + 256) + 8 * nt * 257)
        return {"bytes": 12 * nv + 16 * nt * nv + (2 * par if kind == "training" else par // 2),
                "flops": (6 if kind == "training" else 2) * mac}
    ntr = 4 if case["fit_b1"] or kind != "gn" else 3
    item = 2 if case["f16"] else 4
    trains = item * ntr * nt * nv
    data = 8 * c * nt * nk
    maps = 20 * nv + (8 * c * nv if c > 1 else 0)
    x_stage = 8 * c * nt * nk * (nv if case["radial"] else case["nx"])
    if case["readout"]:
        x_stage *= 16
    y_stage = (2 * ntr + 4 + 8 * c) * nt * nv
    if case["n_iso"]:
        sim = 60 * case["n_iso"] * nt * nv
    else:
        sim = (67 if ntr == 4 else 45) * case["n_states"] * nt * nv
    if kind == "products":
        return {"bytes": 2 * trains + 2 * data + 3 * maps, "flops": 2 * (x_stage + y_stage)}
    if kind == "gradient":
        return {"bytes": trains + 2 * data + 2 * maps, "flops": sim + 2 * (x_stage + y_stage)}
    # A step: the trains written once and read once per CG iteration (they exceed every cache at the
    # larger sizes), a value-only simulation and residual for the line search.
    n = case["n_cg"]
    return {"bytes": (n + 2) * trains + 2 * data + 3 * maps,
            "flops": sim + 13 * case["n_states"] * nt * nv + 3 * (x_stage + y_stage) + n * 2 * y_stage}


# ------------------------------------------------------------------ FP64 reference
def epg_trains(pr, theta, tangents):
    """Gradient-spoiled EPG: imaginary parts of m and its derivatives in ln T1, ln T2, B1, [1 or 4][T][Nv].
    States per order k: F+ = i f, F- = i g, Z = z."""
    nv, kk, nq = theta.shape[1], pr.n_states, 4 if tangents else 1
    t1, t2, b1 = torch.exp(theta[0]), torch.exp(theta[1]), theta[2]
    x = torch.zeros(nq, 3, kk, nv, dtype=torch.float64, device=theta.device)
    x[0, 2, 0] = -1.0

    def relax(tau):
        if tau <= 0.0:
            return
        e1, e2 = torch.exp(-tau / t1), torch.exp(-tau / t2)
        x[:, :2] *= e2
        x[:, 2] *= e1
        if tangents:
            x[1, 2] += (tau / t1) * x[0, 2]
            x[1, 2, 0] -= (tau / t1) * e1
            x[2, :2] += (tau / t2) * x[0, :2]
        x[0, 2, 0] -= torch.expm1(-tau / t1)

    out = torch.empty(nq, pr.n_tr, nv, dtype=torch.float64, device=theta.device)
    relax(pr.t_inv)
    for n in range(pr.n_tr):
        sign = 1.0 if math.cos(float(pr.rf_phase[n])) > 0 else -1.0
        da = sign * math.radians(float(pr.flip_deg[n]))
        ca, sa = torch.cos(b1 * da), torch.sin(b1 * da)
        c2, s2 = 0.5 * (1.0 + ca), 0.5 * (1.0 - ca)
        f, g, z = x[:, 0], x[:, 1], x[:, 2]
        if tangents:
            diff = 0.5 * (f[0] - g[0])
            df = -sa * diff - ca * z[0]
            dz = ca * diff - sa * z[0]
        nf = c2 * f + s2 * g - sa * z
        ng = s2 * f + c2 * g + sa * z
        nz = 0.5 * sa * (f - g) + ca * z
        if tangents:
            nf[3] += da * df
            ng[3] -= da * df
            nz[3] += da * dz
        x[:, 0], x[:, 1], x[:, 2] = nf, ng, nz
        relax(pr.te)
        out[:, n] = sign * x[:, 0, 0]
        relax(pr.tr - pr.te)
        nf = torch.cat([torch.zeros_like(f[:, :1]), x[:, 0, :-1]], 1)
        ng = torch.cat([x[:, 1, 1:], torch.zeros_like(f[:, :1])], 1)
        nf[:, 0] = -ng[:, 0]
        x[:, 0], x[:, 1] = nf, ng
    return out


def isochromat_trains(pr, theta, tangents):
    """Balanced isochromats with a slice profile, the same outputs. States (my, mz); mx stays 0 for RF phases 0, pi."""
    nq = 4 if tangents else 1
    scale = torch.as_tensor(pr.iso[0], dtype=torch.float64, device=theta.device)[:, None]
    weight = torch.as_tensor(pr.iso[1], dtype=torch.float64, device=theta.device)[:, None]
    t1, t2, b1 = torch.exp(theta[0]), torch.exp(theta[1]), theta[2]
    x = torch.zeros(nq, 2, scale.shape[0], theta.shape[1], dtype=torch.float64, device=theta.device)
    x[0, 1] = -1.0

    def relax(tau):
        e1, e2 = torch.exp(-tau / t1), torch.exp(-tau / t2)
        x[:, 0] *= e2
        x[:, 1] *= e1
        if tangents:
            x[1, 1] += (tau / t1) * (x[0, 1] - e1)
            x[2, 0] += (tau / t2) * x[0, 0]
        x[0, 1] += 1.0 - e1

    out = torch.empty(nq, pr.n_tr, theta.shape[1], dtype=torch.float64, device=theta.device)
    relax(pr.t_inv)
    for n in range(pr.n_tr):
        sign = 1.0 if math.cos(float(pr.rf_phase[n])) > 0 else -1.0
        da = sign * math.radians(float(pr.flip_deg[n])) * scale
        c, s = torch.cos(b1 * da), torch.sin(b1 * da)
        y, z = c * x[:, 0] - s * x[:, 1], s * x[:, 0] + c * x[:, 1]
        if tangents:
            y[3], z[3] = y[3] - da * z[0], z[3] + da * y[0]
        x[:, 0], x[:, 1] = y, z
        relax(pr.te)
        out[:, n] = sign * (weight * x[:, 0]).sum(1)
        relax(pr.tr - pr.te)
    return out


class Model:
    """Signal, J v and Re(J^H w) in FP64 at theta (float64 [5][Nv])."""

    def __init__(self, q, theta, tangents=True):
        self.pr, self.theta = q.pr, theta
        self.coil = None if q.coil is None else q.coil.to(torch.complex128)
        self.on = None if q.mask is None else (q.mask != 0).double()
        self.db0 = q.db0.double() if q.case["readout"] else None
        sim = isochromat_trains if q.pr.iso is not None else epg_trains
        self.mu = sim(q.pr, theta, tangents)
        pr = q.pr
        self.x = torch.arange(pr.nx, device=DEV, dtype=torch.float64) - pr.nx // 2
        self.y = torch.arange(pr.ny, device=DEV, dtype=torch.float64) - pr.ny // 2
        ks = torch.arange(pr.n_read, device=DEV, dtype=torch.float64) - pr.n_read // 2
        line = torch.as_tensor(pr.ky_line.astype(np.float64), device=DEV) - pr.ny // 2
        self.ex = self._cis(torch.outer(ks / pr.n_read, self.x))
        self.ey = self._cis(torch.outer(line / pr.ny, self.y))
        if pr.traj is not None:
            self.kx = torch.as_tensor(pr.traj[0], device=DEV) / pr.nx
            self.ky = torch.as_tensor(pr.traj[1], device=DEV) / pr.ny
        self.rho = torch.complex(theta[3], theta[4])
        if self.on is not None:
            self.rho = self.rho * self.on
        if self.db0 is not None:
            self.tau = ks * pr.dwell
            self.lam = torch.complex(-torch.exp(-theta[1]), -2.0 * math.pi * self.db0).view(pr.ny, pr.nx)
            self.te_phase = self._cis(self.db0 * pr.te)

    @staticmethod
    def _cis(cycles):
        return torch.polar(torch.ones_like(cycles), -2.0 * math.pi * (cycles - torch.round(cycles)))

    def _coils(self):
        return [None] if self.coil is None else list(self.coil)

    def _encode(self, x0, x1=None):
        """Voxel values [T][Nv] to samples [C][T][Nk]; x1 is the part weighted by the sample time."""
        pr, out = self.pr, []
        for c in self._coils():
            z = x0 if c is None else x0 * c
            z = z.view(pr.n_tr, pr.ny, pr.nx)
            if pr.traj is not None:
                s = torch.empty(pr.n_tr, pr.n_read, dtype=torch.complex128, device=DEV)
                for n in range(pr.n_tr):
                    p = self._cis(torch.outer(self.kx[n], self.x)) @ z[n].T.contiguous()
                    s[n] = (p * self._cis(torch.outer(self.ky[n], self.y))).sum(1)
            elif self.db0 is not None:
                s = 0.0
                zy = z * self.ey[:, :, None]
                for ix in range(pr.nx):
                    e = torch.exp(torch.outer(self.lam[:, ix], self.tau)) * self.ex[:, ix]
                    s = s + zy[:, :, ix].contiguous() @ e
                    if x1 is not None:
                        s = s + (x1.view_as(z)[:, :, ix] * self.ey).contiguous() @ (e * self.tau)
            else:
                u = torch.cat([(a * b[:, :, None]).sum(1) for a, b in zip(z.split(64), self.ey.split(64))])
                s = u @ self.ex.T.contiguous()
            out.append(s)
        return torch.stack(out)

    def _decode(self, w):
        """Adjoint of _encode: samples [C][T][Nk] to ([T][Nv], the same weighted by the sample time or None)."""
        pr = self.pr
        v = torch.zeros(pr.n_tr, pr.ny, pr.nx, dtype=torch.complex128, device=DEV)
        vt = torch.zeros_like(v) if self.db0 is not None else None
        for c, wc in zip(self._coils(), w):
            if pr.traj is not None:
                u = torch.empty_like(v)
                for n in range(pr.n_tr):
                    e = self._cis(torch.outer(self.ky[n], self.y)).conj() * wc[n][:, None]
                    u[n] = e.T.contiguous() @ self._cis(torch.outer(self.kx[n], self.x)).conj().resolve_conj()
            elif self.db0 is not None:
                u = torch.empty_like(v)
                for ix in range(pr.nx):
                    e = (torch.exp(torch.outer(self.lam[:, ix], self.tau)) * self.ex[:, ix]).conj().T.contiguous()
                    u[:, :, ix] = self.ey.conj() * (wc @ e)
                    vt[:, :, ix] += self.ey.conj() * ((wc * self.tau) @ e)
            else:
                u = self.ey.conj()[:, :, None] * (wc @ self.ex.conj().resolve_conj())[:, None, :]
            if c is not None:
                u = u * c.conj().view(pr.ny, pr.nx)
            v += u
        return v.view(pr.n_tr, -1), None if vt is None else vt.view(pr.n_tr, -1)

    def _phased(self, x):
        return x if self.db0 is None else x * self.te_phase

    def signal(self):
        return self._encode(self._phased(1j * self.rho * self.mu[0]))

    def jv(self, v):
        if self.on is not None:
            v = v * self.on
        nu = torch.complex(v[3], v[4])
        a = v[0] * self.mu[1] + v[1] * self.mu[2] + v[2] * self.mu[3]
        x0 = self._phased(1j * (self.rho * a + nu * self.mu[0]))
        x1 = None
        if self.db0 is not None:
            x1 = self._phased(1j * self.rho * self.mu[0] * torch.exp(-self.theta[1]) * v[1])
        return -self._encode(x0, x1)

    def jhw(self, w):
        v, vt = self._decode(w)
        if self.db0 is not None:
            v, vt = v * self.te_phase.conj(), vt * self.te_phase.conj()
        a = [(m * v).sum(0) for m in self.mu]   # sum_n mu_p V
        rc = self.rho.conj()
        g = [(1j * rc * a[q + 1]).real for q in range(3)]
        if self.db0 is not None:
            g[1] = g[1] + (1j * rc * (self.mu[0] * vt).sum(0)).real * torch.exp(-self.theta[1])
        g += [-(-1j * a[0]).real, a[0].real]
        g = torch.stack(g)
        return g if self.on is None else g * self.on


def _gn_exact(q):
    case, opt = q.case, q.param_mask
    theta, data = q.start.double(), q.data.to(torch.complex128)
    act = torch.tensor([(opt >> p) & 1 for p in range(5)], dtype=torch.float64, device=DEV)[:, None]
    m = Model(q, theta)
    r = data - m.signal()
    f0 = 0.5 * float(torch.linalg.vector_norm(r)) ** 2
    g = act * m.jhw(r)
    step, res = torch.zeros_like(g), -g
    d, rr = res.clone(), float((g * g).sum())
    for _ in range(case["n_cg"]):
        y = act * m.jhw(m.jv(d))
        kappa = float((d * y).sum())
        if rr == 0.0 or kappa <= 0.0:
            break
        step += rr / kappa * d
        res -= rr / kappa * y
        new = float((res * res).sum())
        d, rr = res + new / rr * d, new
    lo, hi = torch.tensor(I.GN_LO, device=DEV).double(), torch.tensor(I.GN_HI, device=DEV).double()
    move = act[:3] * (1.0 if m.on is None else m.on) > 0
    del m
    t, f1 = 1.0, f0
    for _ in range(8):
        trial = theta + t * step
        box = torch.minimum(torch.maximum(trial[:3], lo[:, None]), hi[:, None])
        trial[:3] = torch.where(move, box, trial[:3])
        ft = 0.5 * float(torch.linalg.vector_norm(data - Model(q, trial, False).signal())) ** 2
        if ft <= f0 + 1e-4 * float((g * (trial - theta)).sum()):
            theta, f1 = trial, ft
            break
        t *= 0.5
    return {"theta": theta, "f0": f0, "f1": f1, "gnorm": float(torch.linalg.vector_norm(g))}


def _network_exact(q):
    nt, kind = q.case["n_tr"], q.case["kind"]
    lo = torch.tensor(I.SURR_LO, dtype=torch.float32, device=DEV).double()[:, None]
    hi = torch.tensor(I.SURR_HI, dtype=torch.float32, device=DEV).double()[:, None]
    scale = torch.tensor(SURR_SCALE, dtype=torch.float32, device=DEV).double()
    sizes = [(256, 3), (256,)] + 3 * [(256, 256), (256,)] + [(8 * nt, 256), (8 * nt,)]
    flat, par = q.params.double(), []
    for s in sizes:
        n = math.prod(s)
        par.append(flat[:n].view(s))
        flat = flat[n:]
    h = 2.0 * (q.theta.double() - lo) / (hi - lo) - 1.0
    kept = []
    for k in range(4):
        z = par[2 * k] @ h + par[2 * k + 1][:, None]
        kept.append((h, z))
        h = 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))
    if kind == "network":
        y = par[8][4 * nt:] @ h + par[9][4 * nt:, None]
        return y.view(4, nt, -1) * scale[:, None, None]
    y = par[8] @ h + par[9][:, None]
    y[4 * nt:] -= (q.trains.double() / scale[:, None, None]).view(4 * nt, -1)
    grads = [None] * 10
    dy = 2.0 * y / y.numel()
    grads[8], grads[9] = dy @ h.T.contiguous(), dy.sum(1)
    dh = par[8].T.contiguous() @ dy
    for k in range(3, -1, -1):
        h, z = kept[k]
        dz = dh * (0.5 * (1.0 + torch.erf(z / math.sqrt(2.0))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi))
        grads[2 * k], grads[2 * k + 1] = dz @ h.T.contiguous(), dz.sum(1)
        dh = par[2 * k].T.contiguous() @ dz
    return {"loss": float((y * y).mean()), "grad": torch.cat([t.reshape(-1) for t in grads])}


def exact(case, seed):
    q = _Inputs(case, seed)
    kind = case["kind"]
    if kind in ("network", "training"):
        return _network_exact(q)
    if kind == "gn":
        return _gn_exact(q)
    if kind == "gradient":
        m = Model(q, q.start.double())
        r = q.data.to(torch.complex128) - m.signal()
        return {"f": 0.5 * float(torch.linalg.vector_norm(r)) ** 2, "r": r, "g": m.jhw(r)}
    m = Model(q, q.theta.double())
    return {"jv": m.jv(q.v.double()), "jhw": m.jhw(q.w.to(torch.complex128))}
