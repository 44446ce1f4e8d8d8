"""The group walk's FP32 tests away from ordinary inputs.

Lengths in other units: positions, box and h times a power of two.  Every stage
of the step is then the same arithmetic on shifted exponents, so h, the lists and
every field are those of the unit box, shifted, bit for bit.

Positions and smoothing lengths that are no numbers: such a particle is nobody's
neighbour by position and has no candidates of its own, whatever the sign of its
NaN, and the lists of the others are the brute-force ones."""
import numpy as np
import pytest

from paper_2005_02656_amd import inputs, sph
from gpu_support import Run, configs

pytestmark = pytest.mark.gpu

# exponent of length of each field a step leaves (times the box's exponent)
POWERS = dict(x=1, y=1, z=1, h=1, vx=0, u=0, rho=-3, omega=0, p=-3, c11=-2, c12=-2, c33=-2,
              ax=-1, ay=-1, az=-1, du=-1)


def _random(n, periodic, seed=0):
    rng = np.random.default_rng(n + seed)
    pos = rng.random((3, n))
    pos[:, : n // 3] = 0.5 + 0.5 * (pos[:, : n // 3] - 0.5)   # a denser middle
    v = rng.normal(0.0, 0.1, size=(3, n))
    h = 0.5 * (60.0 / n / (4.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
    arr = dict(x=pos[0], y=pos[1], z=pos[2], vx=v[0], vy=v[1], vz=v[2],
               m=rng.uniform(0.5, 1.5, n) / n, u=rng.uniform(0.5, 1.5, n),
               h=h * rng.uniform(0.8, 1.0, n), id=np.arange(n, dtype=np.int64))
    return inputs.Workload(f"range{n}", arr, inputs.base_params(periodic=periodic))


def _scaled(w, e):
    f = 2.0 ** e
    arr = {k: (v * f if k in ("x", "y", "z", "h") else v) for k, v in w.arrays.items()}
    par = dict(w.params, box_lo=tuple(f * v for v in w.params["box_lo"]),
               box_hi=tuple(f * v for v in w.params["box_hi"]))
    return inputs.Workload(w.name, arr, par)


def _step(w, **kw):
    cfg, _ = configs(w, ng_max=1000, n_target=60.0, newton_iters=2, **kw)
    r = Run(w, cfg)
    sph.step(cfg, r.parts, r.g, r.ws)
    st = r.status()
    return {k: r.by_id(k) for k in POWERS}, r.neighbor_pairs(), st


@pytest.mark.parametrize("n,periodic", [(3001, (1, 1, 1)), (3001, (0, 1, 0)), (26001, (0, 0, 0))])
@pytest.mark.parametrize("e", [-80, -64, 56, 64, 80])
def test_step_in_other_units(n, periodic, e):
    w = _random(n, periodic)
    f0, p0, st0 = _step(w)
    f1, p1, st1 = _step(_scaled(w, e))
    assert st0 == st1 == (0, 0)
    for k, p in POWERS.items():
        assert np.array_equal(f1[k], f0[k] * 2.0 ** (p * e)), k
    assert all(np.array_equal(a, b) for a, b in zip(p0, p1))


@pytest.mark.parametrize("n", [3001, 26001])
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("field", ["x", "y", "h"])
def test_particles_without_a_position_or_a_reach(n, sign, field):
    w = _random(n, (1, 1, 1) if field == "x" else (0, 0, 1), seed=1)
    rng = np.random.default_rng(3)
    bad = rng.choice(n, 40, replace=False)
    arr = {k: v.copy() for k, v in w.arrays.items()}
    arr[field][bad] = np.copysign(np.nan, sign)
    cfg, _ = configs(w, ng_max=1000, newton_iters=0)
    r = Run(inputs.Workload(w.name, arr, w.params), cfg)
    sph.step(cfg, r.parts, r.g, r.ws)
    _, bits = r.status()
    # (without a position: alone, a singular tau; without h: a density that is no number)
    assert bits & (sph.ERRBIT_NONFINITE if field == "h" else sph.ERRBIT_SINGULAR_TAU), bits
    assert not bits & sph.ERRBIT_NEIGHBOR_OVERFLOW, bits
    nk_v, _ = sph.candidates_view(cfg, r.ws)
    nk = np.empty(n, np.int64)
    nk[r.ids()] = nk_v.cpu().numpy()
    assert nk.max() <= 1000
    if field != "h":
        assert np.all(nk[bad] == 0)
    P, nc, ns = r.neighbor_pairs()
    # brute force: comparisons with NaN are false, a NaN reach is no reach
    X = np.stack([w.arrays[k] if k != field else arr[k] for k in "xyz"], 1)
    per = np.asarray(w.params["periodic"], dtype=bool)
    h = arr["h"]
    for i in rng.choice(n, 60, replace=False).tolist() + bad[:8].tolist():
        d = X - X[i]
        d = np.where(per, d - np.round(d), d)
        r2 = d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1] + d[:, 2] * d[:, 2]
        r2[i] = np.inf
        with np.errstate(invalid="ignore"):
            gather = r2 < (2.0 * h[i]) ** 2
            both = gather | (r2 < (2.0 * np.fmax(h, h[i])) ** 2)
        mine = P[P[:, 0] == i]
        assert nc[i] == gather.sum() and ns[i] == both.sum(), i
        assert np.array_equal(mine[:, 1], np.nonzero(both)[0]), i


@pytest.mark.parametrize("n,periodic", [(3001, (1, 0, 1)), (70001, (0, 0, 0))])
@pytest.mark.parametrize("e", [-80, 80])
def test_stage_calls_in_other_units(n, periodic, e):
    """update_h and the neighbour lists by the stage calls, and a step with a clamp
    above the fused step's, which uses them."""
    w = _random(n, periodic)
    got = []
    for u in (w, _scaled(w, e)):
        cfg, _ = configs(u, ng_max=600, n_target=60.0, newton_iters=2)
        r = Run(u, cfg)
        sph.build_cells(cfg, r.parts, r.ws)
        sph.update_h(cfg, r.parts, r.ws)
        h = r.by_id("h")
        sph.find_neighbors(cfg, r.parts, r.ws)
        assert r.status() == (0, 0)
        got.append((h, r.neighbor_pairs(), _step(u, h_ratio_max=2.0)))
    (h0, p0, s0), (h1, p1, s1) = got
    assert np.array_equal(h1, h0 * 2.0 ** e)
    assert all(np.array_equal(a, b) for a, b in zip(p0, p1))
    assert s0[2] == s1[2]   # (an open corner may leave a tau singular, in either unit)
    for k, p in POWERS.items():
        assert np.array_equal(s1[0][k], s0[0][k] * 2.0 ** (p * e)), k
    assert all(np.array_equal(a, b) for a, b in zip(s0[1], s1[1]))
