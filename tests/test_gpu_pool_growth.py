"""The particle pool starts smaller than its capacity and grows when a step needs it:
a run that passes the first size mid-call equals the oracle's, its saved state loads into
a context whose pool has not grown, a capacity between the first size and the need still
refuses the step that passes it, and the state of the step before stays."""
import numpy as np
import pytest

import oracle
from paper_2312_16981_amd import ugkwp
from paper_2312_16981_amd import workloads as W
from test_gpu_parity import compare_state

pytestmark = pytest.mark.gpu
FIRST = 1 << 21        # slots a small context's pool starts with


def _thin(dim, **kw):
    p = dict(dt=2e-3, steps=0, w_ref=5e-8, pool_cap=1 << 24, seed=4)
    p.update(kw)
    if dim == 1:
        return W.slab(40, 4, lambda x: np.where(x < 0.5, 0.5, 20.0), name="grow1d", **p)
    return W.c5_lognormal(n=10, G=4, **p)


def _compare_pool(ctx, sim, p):
    """Ids, cells and groups equal, positions, directions and frequencies within 1e-10, and
    the weights by their sum per (cell, group), the survivor density.  (A weight by itself
    is V (rho - rho^p) / N with rho^p the sum of some 1e4 particles: it differs by 1.7e-10
    from the oracle's also where the pool never grows.)"""
    pg, po = ctx.get_pool(), sim.pool()
    assert len(pg["id"]) == len(po["id"])
    i, j = np.argsort(pg["id"]), np.argsort(po["id"])
    for k in ("id", "cell", "g"):
        assert np.array_equal(pg[k][i], po[k][j]), k
    for k in ("x", "ox", "nu") + (("y", "oy") if p.dim == 2 else ()):
        assert np.max(np.abs(pg[k][i] - po[k][j])) <= 1e-10 * np.max(np.abs(po[k])), k
    V = (p.x1 - p.x0) / p.nx * ((p.y1 - p.y0) / p.ny if p.dim == 2 else 1.0)
    dens = np.bincount(pg["cell"] * p.G + pg["g"], pg["w"], p.ncell * p.G) / V
    rhop = ctx.get_fields()[2].reshape(-1)
    assert np.max(np.abs(dens - rhop)) <= 1e-10 * np.max(rhop)


@pytest.mark.parametrize("dim,n", [(1, 8), (2, 4)])
def test_growth_within_a_call(dim, n):
    p = _thin(dim)
    ctx, sim = ugkwp.from_problem(p, sort_interval=1000), oracle.Sim(p)
    ctx.step(n)
    sim.step(n)
    assert ctx.get_diag()["n_pushed"] > FIRST
    compare_state(ctx, sim, p, what=f"grown {dim}-D")
    _compare_pool(ctx, sim, p)
    saved = ctx.get_state()
    other = ugkwp.from_problem(p)
    other.set_state(saved)
    other.step(1)
    sim.step(1)
    compare_state(other, sim, p, what="loaded into a small pool")


def test_capacity_still_refuses():
    p = _thin(1).with_(pool_cap=FIRST + 100000)
    ctx, sim = ugkwp.from_problem(p, sort_interval=1000), oracle.Sim(p)
    assert ctx.step(12, check=False) == ugkwp.EPOOL
    done = ctx.get_counters()[1]
    assert 0 < done < 12
    sim.step(done)
    rho, T, rhop = ctx.get_fields()
    for a, b in zip((rho, T, rhop), sim.fields()):
        assert np.max(np.abs(a - b)) <= 1e-10 * max(np.max(np.abs(b)), 1e-300)
    ctx = ugkwp.from_problem(_thin(1).with_(pool_cap=1))
    assert ctx.step(2, check=False) == ugkwp.EPOOL
