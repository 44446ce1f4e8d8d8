"""Refits of the fused step over several rounds of their bounded grids, in both
precisions and at particle numbers on either side of where 64 or 8 wavefronts
share the flags of 512 slots: a share of the particles starts with h 15% short and
grows past the short reach.  On sampled targets h is the oracle's at 1e-12 and the
neighbour counts are the oracle's at it."""
import numpy as np
import pytest

import oracle
from paper_2005_02656_amd import inputs, sph
from gpu_support import Run, configs

pytestmark = pytest.mark.gpu
TOL = 1e-12
SHARE_N = 1 << 20


@pytest.mark.parametrize("n,share,precision", [
    (50021, 1.0, sph.FP64), (50021, 0.02, sph.MIXED), (70001, 1.0, sph.MIXED),
    (70001, 0.02, sph.FP64), (SHARE_N, 1.0, sph.FP64), (SHARE_N + 1, 1.0, sph.MIXED),
    (SHARE_N + 1, 0.001, sph.FP64)])
def test_refits_of_many_targets(n, share, precision):
    rng = np.random.default_rng(n)
    pos = rng.random((3, n))
    h = np.full(n, 0.5 * (60.0 / n / (4.0 / 3.0 * np.pi)) ** (1.0 / 3.0))
    grown = rng.random(n) < share
    h[grown] *= 0.85
    v = rng.normal(0.0, 0.1, size=(3, n))
    arr = dict(x=pos[0], y=pos[1], z=pos[2], vx=v[0], vy=v[1], vz=v[2], m=np.full(n, 1.0 / n),
               u=np.ones(n), h=h, id=np.arange(n, dtype=np.int64))
    w = inputs.Workload(f"refit{n}", arr, inputs.base_params())
    cfg, ocfg = configs(w, ng_max=200, n_target=60.0, newton_iters=2, precision=precision)
    r = Run(w, cfg)
    sph.step(cfg, r.parts, r.g, r.ws)
    assert r.status() == (0, 0)
    h_g = r.by_id("h")
    tgt = np.concatenate([rng.choice(n, 24, replace=False),
                          rng.choice(np.nonzero(grown)[0], 24, replace=False)])
    h_o = oracle.update_h(ocfg, *pos.copy(), h, targets=tgt)
    assert np.max(np.abs(h_g[tgt] - h_o[tgt]) / h_o[tgt]) < TOL
    nc_v, ns_v, _ = sph.neighbors_view(cfg, r.ws)
    nc, ns = np.empty(n, np.int64), np.empty(n, np.int64)
    nc[r.ids()], ns[r.ids()] = nc_v.cpu().numpy(), ns_v.cpu().numpy()
    nc_o, ns_o, _, _ = oracle.neighbors(ocfg, *pos.copy(), h_g, targets=tgt)
    assert np.array_equal(nc[tgt], nc_o) and np.array_equal(ns[tgt], ns_o)
