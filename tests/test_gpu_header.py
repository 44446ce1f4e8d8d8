"""A workspace whose header was never cleared: the cell build writes every field the
kernels go by, so a step, the stage calls, gravity and the reverse pass give the same
bits as on a cleared one (only the error word, which is sticky, means nothing)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2005_02656_amd import inputs, sph
from gpu_support import Run, configs, rel_err

pytestmark = pytest.mark.gpu
CS = ("c11", "c12", "c13", "c22", "c23", "c33")


def _fields(w, cfg, fill, path):
    parts = sph.Particles.from_arrays(w.arrays, cfg)
    ws, g = sph.Workspace(cfg), sph.Globals()
    ws.buf.fill_(fill)
    out = {}
    if path == "step":
        for _ in range(2):
            sph.step(cfg, parts, g, ws)
        out["g"] = g.t
    elif path == "stages":
        for f in (sph.build_cells, sph.update_h, sph.find_neighbors, sph.density, sph.iad,
                  sph.momentum_energy):
            f(cfg, parts, ws)
        sph.timestep(cfg, g, ws)
        sph.integrate(cfg, parts, g, ws)
        out["g"] = g.t
    elif path == "gravity":
        sph.build_cells(cfg, parts, ws)
        for k, t in enumerate(sph.gravity(cfg, parts, ws, sph.GravityWorkspace(cfg), 1.0, 1e-3,
                                          0.5)):
            out[f"g{k}"] = t
    else:
        gout, gin = sph.Grads(w.n), sph.Grads(w.n)
        for k in sph.GRAD_FIELDS:
            gout[k].fill_(1.0)
        sph.step_backward(cfg, parts, g, ws, sph.AdjointWorkspace(cfg), gout, gin)
        out.update({k: gin[k] for k in sph.GRAD_FIELDS})
    out.update({k: parts[k] for k in ("id", "x", "h", "rho", "ax", "u")})
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("path", ["step", "stages", "gravity", "backward"])
@pytest.mark.parametrize("fill", [0x55, 0xff])
def test_uncleared_header(path, fill):
    n = 5003
    w = inputs.random_periodic(n, seed=4, h_lo=0.05, h_hi=0.06)
    if path == "gravity":
        w = inputs.Workload(w.name, w.arrays, {**w.params, "periodic": (0, 0, 0)})
    cfg, _ = configs(w, ng_max=200)
    a, b = _fields(w, cfg, 0, path), _fields(w, cfg, fill, path)
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("field", ["m", "u", "h", "x"])
@pytest.mark.parametrize("n,slot", [(1060001, 65700), (1060001, 1060000), (4300001, 262100)])
def test_record_of_many_workgroups(n, slot, field):
    """One particle differs, in a slot that a late workgroup of the bounding box reads
    (258 of them and 1,024 of them): its density, its neighbours' and the forces
    between them at 1e-12 of the oracle's."""
    rng = np.random.default_rng(3)
    pos = rng.random((3, n))
    pos[:, slot] = 0.5
    h = 0.5 * (60.0 / n / (4.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
    v = rng.normal(0.0, 0.1, size=(3, n))
    a = dict(x=pos[0], y=pos[1], z=pos[2], vx=v[0], vy=v[1], vz=v[2], m=np.full(n, 1.0 / n),
             u=np.ones(n), h=np.full(n, h), id=np.arange(n, dtype=np.int64))
    if field == "x":
        a["x"][slot] = 1.0 + 1.2 * h
        a["h"][slot] = 1.9 * h
    else:
        a[field][slot] *= {"m": 3.0, "u": 0.25, "h": 1.9}[field]
    w = inputs.Workload("one", a, {**inputs.base_params(), "periodic": (0, 0, 0)})
    cfg, ocfg = configs(w, ng_max=600, n_target=60.0)
    r = Run(w, cfg)
    for f in (sph.build_cells, sph.find_neighbors, sph.density, sph.iad, sph.momentum_energy):
        f(cfg, r.parts, r.ws)
    d2 = sum((a[k] - a[k][slot]) ** 2 for k in "xyz")
    tgt = np.argsort(d2)[:12]
    hs = a["h"]
    rho, om, p, c = oracle.density(ocfg, a["x"], a["y"], a["z"], hs, a["m"], a["u"], targets=tgt)
    for f, o in (("rho", rho), ("omega", om), ("p", p), ("c", c)):
        assert rel_err(r.by_id(f)[tgt], o[tgt]) < 1e-12, f
    me = oracle.momentum_energy(ocfg, a["x"], a["y"], a["z"], a["vx"], a["vy"], a["vz"], hs,
                                a["m"], r.by_id("rho"), r.by_id("omega"), r.by_id("p"),
                                r.by_id("c"), np.stack([r.by_id(f) for f in CS]), targets=tgt)
    for f in ("ax", "ay", "az"):
        assert rel_err(r.by_id(f)[tgt], me[f][tgt], me["scale_a"][tgt]) < 1e-12, f
    assert rel_err(r.by_id("du")[tgt], me["du"][tgt], me["scale_du"][tgt]) < 1e-12
