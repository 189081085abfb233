"""GPU vs FP64 oracle on 1-D meshes of more tiles than take the stopping test in every block:
a launch of one block decides after each round.  The bar of the other parity tests."""
import numpy as np
import pytest

import oracle
from paper_2312_16981_amd import ugkwp
from paper_2312_16981_amd import workloads as W
from test_gpu_parity import compare_state, run_pair, say
from test_gpu_tiles import _two

pytestmark = pytest.mark.gpu
SL, WI, LIN = W.FLAG_SLOPES, W.FLAG_WAVE_ITER, W.FLAG_SI_LINEARIZED
NX, G = 12300, 33       # 64 lanes a cell: 1025 tiles and more in every shape


def _slab(**kw):
    p = dict(dt=1.4e-4, w_ref=2e-6, pool_cap=1 << 21)
    p.update(kw)
    return _two(NX, G, **p)


@pytest.mark.parametrize("flags,T_power", [(0, 0.0), (LIN, 0.0), (SL | WI, 0.0), (0, 0.5), (LIN | SL | WI, 0.5)])
def test_long_slab(flags, T_power):
    run_pair(_slab(flags=flags, T_power=T_power, dt=2.5e-5 if flags & WI else 1.4e-4), 2)


def test_long_slab_in_one_call_with_captured_launches():
    p = _slab()
    ctx, sim = ugkwp.from_problem(p, extra_flags=ugkwp.FLAG_GRAPH), oracle.Sim(p)
    ctx.step(4)
    sim.step(4)
    compare_state(ctx, sim, p, what="graphs")


def test_iteration_limit_of_a_long_slab():
    p = _slab()
    sim = oracle.Sim(p)
    need = []
    for _ in range(3):
        sim.step(1)
        need.append(sim.diag()["sweeps"])
    most = max(need)
    say("[long] sweeps", need)
    ctx = ugkwp.from_problem(p.with_(si_max_iters=most))
    ctx.step(3)
    compare_state(ctx, sim, p, what="limit reached")
    ctx = ugkwp.from_problem(p.with_(si_max_iters=most - 1))
    assert ctx.step(3, check=False) == ugkwp.ENOCONV
    first = need.index(most)
    assert ctx.get_counters()[1] == first
    sim = oracle.Sim(p)
    if first:
        sim.step(first)
    for a, b in zip(ctx.get_fields(), sim.fields()):
        assert np.max(np.abs(a - b)) <= 1e-10 * max(np.max(np.abs(b)), 1e-300)


def test_failed_temperature_of_a_long_slab():
    """Stiff literal coupling: the temperature's error, as on a short slab."""
    p = _slab(w_ref=1e6).with_(cv=np.full(NX, 1e-6))
    small = _two(40, G, dt=2e-4, w_ref=1e6).with_(cv=np.full(40, 1e-6))
    codes = [ugkwp.from_problem(q).step(1, check=False) for q in (small, p)]
    assert codes[0] == codes[1] == ugkwp.ENONFINITE
