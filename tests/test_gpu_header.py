"""A workspace whose header was never cleared: the cell build writes every field the
kernels go by, so a step, the stage calls, gravity and the reverse pass give the same
bits as on a cleared one (only the error word, which is sticky, means nothing)."""
import numpy as np
import pytest
import torch

from paper_2005_02656_amd import inputs, sph
from gpu_support import configs

pytestmark = pytest.mark.gpu


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
