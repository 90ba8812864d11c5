"""Body observables against the oracle's on the same stress and the same nodes: polygons of few and many
edges, round and not convex, either way round, across the periodic boundary, narrower and wider than a wave
of sites.

The stress is the lattice's own (FP32 values, exact in FP64), so only the order of FP64 sums differs: of at
most 1e4 sites with terms of at most D = max |div sigma| a rounding error below 1e4 * 2.2e-16 per unit of
sites * D, and the areas add as much again: 1e-11 * sites * D is five times that."""
import math

import numpy as np
import pytest

from paper_2209_14889_amd import lb
from paper_2209_14889_amd import workload as wl
from tests.helpers import oracle_sim

pytestmark = pytest.mark.gpu


def blob(cx, cy, radius, n, dent, turn):
    a = 2 * math.pi * np.arange(n)[::turn] / n + 0.1
    r = radius * (1.0 + dent * np.cos(5 * a))
    return np.stack([cx + r * np.cos(a), cy + r * np.sin(a)], axis=1)


SHAPES = [(1.2, 3), (4.3, 8), (12.4, 63), (12.4, 65), (31.6, 199), (31.9, 256)]


@pytest.mark.parametrize("walls,radius,n", [(0, *s) for s in [*SHAPES, (40.2, 1024)]] + [(1, *s) for s in SHAPES])
@pytest.mark.parametrize("dent,turn", [(0.0, 1), (0.3, -1)])
def test_observables_of_a_polygon(walls, radius, n, dent, turn):
    nx, ny = 150, 131
    w = wl.small_case(9, nx, ny, n_bodies=2, radius=6.0, walls=walls)
    s = w.sims[0]
    rng = np.random.default_rng(n)
    s.sigma0 = (1e-3 * rng.standard_normal((3, ny, nx))).astype(np.float32).astype(np.float64)
    y = ny / 2 + 0.37 if walls else 5.21      # without walls the second body crosses the lower edge
    s.bodies[1].R = blob(nx - 3.3, y, radius / (1 + dent), n, dent, turn)
    g = lb.Sim(s)
    r = oracle_sim(s)
    got = g.body_forces()
    device = g._torch.zeros(16, dtype=g._torch.float64, device="cuda")
    g.body_forces_device(device)
    g.sync()
    per_body = device.cpu().numpy().reshape(2, 8)
    for b in range(2):
        R = g.nodes()[b]
        r.bodies[b].R = R.copy()
        sites = (np.ptp(R[:, 0]) + 2) * (np.ptp(R[:, 1]) + 2)
        tol = 1e-11 * sites * 4e-3 * 1.5      # |div sigma| <= 2 max |sigma|, max |sigma| about 4e-3
        want = r.body_force(b)
        assert np.max(np.abs(got[b, 0:2] - want[:2])) <= tol
        assert np.max(np.abs(got[b, 4:6] - want[2:4])) <= 1e-11 * nx
        assert np.max(np.abs(got[b, 8:10] - r.body_force_area(b))) <= tol
        np.testing.assert_array_equal(per_body[b], np.concatenate([got[b, 0:2], got[b, 4:10]]))
    g.close()


def test_observables_of_a_body_beyond_its_patch():
    """A body that the flow has drawn out beyond its force patch, which the next synchronising call reports:
    the device's observables are sums over its sites all the same."""
    import oracle
    nx, ny = 128, 64
    s = wl.small_case(9, nx, ny, n_bodies=1, radius=10.0, pull=0.0).sims[0]
    s.bodies[0].k_spring = s.bodies[0].eps_angle = 1e-12
    s.params["Kx"] = (0.0, 0.0, 0.0, 0.0)     # nothing but viscosity holds the flow back
    s.sigma0 = np.zeros((3, ny, nx))
    s.sigma0[0] = 1e-3 * np.sin(2 * math.pi * np.arange(nx) / nx)
    u = 0.12 * np.sin(2 * math.pi * (np.arange(ny)[:, None] - s.bodies[0].R[:, 1].mean()) / ny) * np.ones((ny, nx))
    s.h0 = oracle.equilibrium(np.ones((ny, nx)), u, np.zeros((ny, nx)))
    g = lb.Sim(s)
    out = g._torch.full((8,), float("nan"), dtype=g._torch.float64, device="cuda")
    g.step(500)
    g.body_forces_device(out)
    with pytest.raises(lb.LBError) as e:
        g.sync()
    assert e.value.code == lb.LB_ERANGE
    v = out.cpu().numpy()
    print("observables beyond the patch", v, flush=True)
    assert np.all(np.isfinite(v)) and np.any(v[0:2] != 0.0) and np.any(v[6:8] != 0.0)
    g.close()
