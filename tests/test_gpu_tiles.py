"""GPU vs FP64 oracle where the tiles of the 1-D source iteration can go wrong:
one cell, the cells around a tile's width, the group counts around a power of
two, iterations of many rounds and of exactly the permitted number of sweeps,
and batches whose instances take different numbers of rounds.  Same bar as the
other parity tests: integers and sweep counts equal, every field, tally and
particle within 1e-10 of its array's max-norm."""
import numpy as np
import pytest

import oracle
from paper_2312_16981_amd import ugkwp
from paper_2312_16981_amd import workloads as W
from test_gpu_parity import compare_state, run_pair, say

pytestmark = pytest.mark.gpu
SL, WI, BP, LIN = W.FLAG_SLOPES, W.FLAG_WAVE_ITER, W.FLAG_BOUNDARY_PARTICLES, W.FLAG_SI_LINEARIZED


def _two(nx, G, **kw):
    p = dict(dt=1e-3, steps=0, w_ref=3e-5, pool_cap=1 << 19, name=f"tiles{nx}_g{G}")
    p.update(kw)
    return W.slab(nx, G, lambda x: np.where(x < 0.45, 0.3, 80.0), **p)


@pytest.mark.parametrize("nx,G", [(1, 1), (2, 64), (3, 33), (9, 32), (17, 16), (33, 7), (64, 64), (129, 24), (513, 2)])
@pytest.mark.parametrize("flags", [0, LIN, SL | WI | BP])
def test_tile_edges(nx, G, flags):
    run_pair(_two(nx, G, flags=flags), 4, every=2)


@pytest.mark.parametrize("nx,G", [(1, 5), (31, 64), (130, 12)])
@pytest.mark.parametrize("flags", [0, LIN, LIN | SL | WI])
def test_tile_edges_opacity_of_temperature(nx, G, flags):
    p = _two(nx, G, flags=flags, T_power=0.5, bc_right=W.BC_REFLECT)
    run_pair(p, 4, every=2)


def test_many_rounds():
    """Sweep counts that grow over the run well past one round (one call)."""
    p = W.thick_thin_joint(nx=90, G=12, w_ref=4e-5, pool_cap=1 << 21)
    ctx, sim = ugkwp.from_problem(p), oracle.Sim(p)
    ctx.step(12)
    most = 0
    for _ in range(12):
        sim.step(1)
        most = max(most, sim.diag()["sweeps"])
    assert most > 16
    compare_state(ctx, sim, p, what="many rounds")
    assert ctx.get_diag()["sweeps_max"] == sim.diag()["sweeps"]


@pytest.mark.parametrize("kind", ["literal", "slopes"])
def test_iteration_limit_across_rounds(kind):
    """A limit of exactly the sweeps a step needs lets it through; one less refuses it
    and leaves the state of the step before."""
    if kind == "literal":
        p = W.thick_thin_joint(nx=90, G=12, w_ref=4e-5, pool_cap=1 << 21)
    else:
        p = _two(100, 6, dt=2e-3, flags=SL | WI)
    sim = oracle.Sim(p)
    need = []
    for _ in range(8):
        sim.step(1)
        need.append(sim.diag()["sweeps"])
    most = max(need)
    say("[tiles] sweeps", need)
    assert most > 8
    ctx = ugkwp.from_problem(p.with_(si_max_iters=most))
    ctx.step(8)
    compare_state(ctx, sim, p, what="limit reached")
    ctx = ugkwp.from_problem(p.with_(si_max_iters=most - 1))
    assert ctx.step(8, check=False) == ugkwp.ENOCONV
    first = need.index(most)
    assert ctx.get_counters()[1] == first
    sim = oracle.Sim(p)
    sim.step(first)
    rho, T, rhop = ctx.get_fields()
    for a, b in zip((rho, T, rhop), sim.fields()):
        assert np.max(np.abs(a - b)) <= 1e-10 * max(np.max(np.abs(b)), 1e-300)


@pytest.mark.parametrize("flags,T_power", [(0, 0.0), (LIN, 0.0), (SL | WI, 0.0), (LIN | SL | WI, 0.5), (LIN, 0.5)])
def test_batch_of_different_rounds(flags, T_power):
    probs = []
    for k, (nx, G, kap) in enumerate([(1, 64, 1.0), (57, 32, 2000.0), (300, 16, 0.01), (19, 5, 300.0), (128, 64, 30.0)]):
        probs.append(W.slab(nx, G, lambda x, kap=kap: np.full_like(x, kap), dt=1e-3 if flags & WI else 4e-3,
                            steps=0, w_ref=4e-5, seed=40 + k, pool_cap=1 << 18, flags=flags, T_power=T_power, name=f"bt{k}"))
    ctx = ugkwp.from_batch(probs)
    sims = [oracle.Sim(q) for q in probs]
    ctx.step(10)
    for s in sims:
        s.step(10)
    say("[tiles] sweeps", [s.diag()["sweeps"] for s in sims])
    for k, (q, s) in enumerate(zip(probs, sims)):
        compare_state(ctx, s, q, inst=k, what=f"batch instance {k}")
