"""The forms that sizes above the lanes' line (65,536 particles) take, against the
oracle: the kernel table, mixed precision (candidates and sums in order), the stage
calls, and the reverse passes, at ragged sizes.  Forward fields on sampled targets,
at 1e-12 in FP64 and 1e-5 in mixed precision (C relative to the condition of tau,
h at 1e-12 in both).  Reverse passes on sets made of slabs too far apart to
interact, so that the dense differentiable oracle of one slab is the reference for
its particles, at 1e-12 as for small sets."""
import numpy as np
import pytest
import torch

import oracle
from oracle import torch_adjoint as TA
from paper_2005_02656_amd import inputs, sph
from gpu_support import Run, configs, rel_err

pytestmark = pytest.mark.gpu
TOL, TOL_MIXED = 1e-12, 1e-5
N = 65613
CS = ("c11", "c12", "c13", "c22", "c23", "c33")


def _random(uniform):
    rng = np.random.default_rng(7 + uniform)
    pos = rng.random((3, N))
    h = 0.5 * (60.0 / N / (4.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
    v = rng.normal(0.0, 0.1, size=(3, N))
    arr = dict(x=pos[0], y=pos[1], z=pos[2], vx=v[0], vy=v[1], vz=v[2],
               m=np.full(N, 1.0 / N) if uniform else rng.uniform(0.5, 1.5, N) / N,
               u=np.ones(N) if uniform else rng.uniform(0.5, 1.5, N),
               h=h * rng.uniform(0.97, 1.0, N), id=np.arange(N, dtype=np.int64))
    return inputs.Workload("large", arr, inputs.base_params())


def _condition(Cm):
    M = np.empty((Cm.shape[1], 3, 3))
    for k, (i, j) in enumerate(((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))):
        M[:, i, j] = M[:, j, i] = Cm[k]
    ev = np.linalg.eigvalsh(M)
    return np.abs(ev[:, 2]) / np.abs(ev[:, 0])


@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("precision", [sph.FP64, sph.MIXED])
@pytest.mark.parametrize("path,table", [("step", 0), ("step", 20000), ("stages", 0),
                                        ("stages", 20000)])
def test_forward_fields(path, table, precision, uniform):
    w = _random(uniform)
    cfg, ocfg = configs(w, ng_max=200, n_target=60.0, newton_iters=2, kernel_table=table,
                        precision=precision)
    a = w.arrays
    tol = TOL if precision == sph.FP64 else TOL_MIXED
    r = Run(w, cfg)
    if path == "step":
        sph.step(cfg, r.parts, r.g, r.ws)
    else:
        for f in (sph.build_cells, sph.update_h, sph.find_neighbors, sph.density, sph.iad,
                  sph.momentum_energy):
            f(cfg, r.parts, r.ws)
    assert r.status() == (0, 0)
    tgt = np.random.default_rng(1).choice(N, 24, replace=False)
    h = r.by_id("h")
    h_o = oracle.update_h(ocfg, a["x"], a["y"], a["z"], a["h"], targets=tgt)
    assert rel_err(h[tgt], h_o[tgt]) < TOL
    rho, om, p, c = oracle.density(ocfg, a["x"], a["y"], a["z"], h, a["m"], a["u"], targets=tgt)
    for f, o in (("rho", rho), ("omega", om), ("p", p), ("c", c)):
        assert rel_err(r.by_id(f)[tgt], o[tgt]) < tol, f
    rho_g = r.by_id("rho")
    Cm, _ = oracle.iad(ocfg, a["x"], a["y"], a["z"], h, a["m"], rho_g, targets=tgt)
    Ct = Cm[:, tgt]
    kap = _condition(Ct) if precision == sph.MIXED else 1.0
    for k, f in enumerate(CS):
        den = max(np.max(np.abs(Ct[k])), np.max(np.abs(Ct[[0, 3, 5]])))
        assert np.max(np.abs(r.by_id(f)[tgt] - Ct[k]) / kap) / den < tol, f
    me = oracle.momentum_energy(ocfg, a["x"], a["y"], a["z"], a["vx"], a["vy"], a["vz"], h,
                                a["m"], rho_g, r.by_id("omega"), r.by_id("p"), r.by_id("c"),
                                np.stack([r.by_id(f) for f in CS]), targets=tgt)
    for f in ("ax", "ay", "az"):
        assert rel_err(r.by_id(f)[tgt], me[f][tgt], me["scale_a"][tgt]) < tol, f
    assert rel_err(r.by_id("du")[tgt], me["du"][tgt], me["scale_du"][tgt]) < tol


# ---------------------------------------------------------------- reverse passes
SIDE, LAYERS, GAP = 8, 7, 4
PER = SIDE * SIDE * LAYERS
SLABS = 148                                    # the last one short of 141 particles


def _slabs():
    """SLABS jittered lattice slabs along x, periodic in y and z, spacing 1."""
    rng = np.random.default_rng(12)
    n = SLABS * PER - 141
    i = np.arange(n)
    s, q = i // PER, i % PER
    X = np.stack([s * (LAYERS + GAP) + q // (SIDE * SIDE), q // SIDE % SIDE, q % SIDE]) + 0.5
    X = X + rng.uniform(-0.08, 0.08, size=(3, n))
    v = rng.normal(0.0, 0.05, size=(3, n))
    arr = dict(x=X[0], y=X[1], z=X[2], vx=v[0], vy=v[1], vz=v[2], m=rng.uniform(0.9, 1.1, n),
               u=rng.uniform(0.9, 1.1, n), h=np.full(n, 1.2), id=np.arange(n, dtype=np.int64))
    for k in "xyz":
        arr["vh" + k] = arr["v" + k] + rng.normal(0.0, 0.01, n)
    arr["du_m1"] = rng.normal(0.0, 0.1, n)
    par = inputs.base_params(periodic=(0, 1, 1), box_lo=(0.0, 0.0, 0.0),
                             box_hi=(1.0, float(SIDE), float(SIDE)))
    return inputs.Workload("slabs", arr, par)


def _slab(w, k):
    return slice(k * PER, min((k + 1) * PER, w.n))


def test_step_backward_of_slabs_matches_oracle():
    w = _slabs()
    a, n, dt_m1 = w.arrays, w.n, 0.02
    assert n > 65536 and n % 64 != 0
    cfg, ocfg = configs(w, ng_max=160, n_target=60.0, newton_iters=2)
    rng = np.random.default_rng(5)
    W = {k: rng.normal(size=n) for k in sph.GRAD_FIELDS}
    probe = Run(w, cfg)
    probe.g.t[1] = dt_m1
    sph.step(cfg, probe.parts, probe.g, probe.ws)
    assert probe.status() == (0, 0)
    r = Run(w, cfg)
    r.g.t[1] = dt_m1
    gout, gin = sph.Grads(n), sph.Grads(n)
    for k in sph.GRAD_FIELDS:
        gout[k].copy_(torch.from_numpy(W[k][probe.ids()]))
    sph.step_backward(cfg, r.parts, r.g, r.ws, sph.AdjointWorkspace(cfg), gout, gin)
    assert r.status() == (0, 0)
    G = {k: gin[k].cpu().numpy() for k in sph.GRAD_FIELDS}
    # the oracle's step of every slab: the smallest of their time steps is the set's
    dts, hs = [], []
    for k in range(SLABS):
        st = {f: v[_slab(w, k)].copy() for f, v in a.items()}
        _, gl, f = oracle.step(ocfg, st, {"dt_m1": dt_m1, "t": 0.0})
        dts.append(gl["dt"])
        hs.append(f["h"])
    dt = min(dts)
    for k in (0, 71, SLABS - 1):
        sl = _slab(w, k)
        t = lambda *f: torch.tensor(np.stack([a[x][sl] for x in f], 1), requires_grad=True)
        ts = dict(x=t("x", "y", "z"), v=t("vx", "vy", "vz"), vh=t("vhx", "vhy", "vhz"),
                  u=torch.tensor(a["u"][sl], requires_grad=True),
                  du_m1=torch.tensor(a["du_m1"][sl], requires_grad=True))
        S = TA.Setup(ocfg, a["m"][sl], hs[k])
        out, _ = TA.step(S, ts, dt, dt_m1)
        L = 0.0
        for c, x in enumerate("xyz"):
            L = L + (torch.tensor(W[x][sl]) * out["x"][:, c]).sum()
            L = L + (torch.tensor(W["v" + x][sl]) * out["v"][:, c]).sum()
            L = L + (torch.tensor(W["vh" + x][sl]) * out["vh"][:, c]).sum()
        for f in ("u", "du_m1"):
            L = L + (torch.tensor(W[f][sl]) * out[f]).sum()
        L.backward()
        ref = {"u": ts["u"].grad, "du_m1": ts["du_m1"].grad}
        for c, x in enumerate("xyz"):
            ref[x], ref["v" + x], ref["vh" + x] = (ts[f].grad[:, c] for f in ("x", "v", "vh"))
        for f in sph.GRAD_FIELDS:
            assert rel_err(G[f][sl], ref[f].numpy()) <= TOL, (k, f)


def test_density_backward_of_slabs_matches_oracle():
    w = _slabs()
    a, n = w.arrays, w.n
    cfg, ocfg = configs(w, ng_max=160, n_target=60.0, newton_iters=2)
    wr = np.random.default_rng(8).normal(size=n)
    r = Run(w, cfg)
    sph.density_eval(cfg, r.parts, r.ws)
    rb = torch.from_numpy(wr[r.ids()]).cuda()
    g = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3)]
    sph.density_backward(cfg, r.parts, r.ws, sph.AdjointWorkspace(cfg), rb, *g)
    assert r.status() == (0, 0)
    for k in (0, 71, SLABS - 1):
        sl = _slab(w, k)
        h = oracle.update_h(ocfg, a["x"][sl], a["y"][sl], a["z"][sl], a["h"][sl])
        x = torch.tensor(np.stack([a[f][sl] for f in "xyz"], 1), requires_grad=True)
        rho, _ = TA.density_omega(TA.Setup(ocfg, a["m"][sl], h), x)
        (rho * torch.tensor(wr[sl])).sum().backward()
        for c in range(3):
            assert rel_err(g[c].cpu().numpy()[sl], x.grad[:, c].numpy()) <= TOL, (k, c)
