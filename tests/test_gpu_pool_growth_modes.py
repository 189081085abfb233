"""The pool's growth within a call where more than the base method is at stake: the wave
flux of every iterate, a batch, and captured launches.  Against the FP64 oracle."""
import pytest

import oracle
from paper_2312_16981_amd import ugkwp
from paper_2312_16981_amd import workloads as W
from test_gpu_parity import compare_state
from test_gpu_pool_growth import FIRST, _thin

pytestmark = pytest.mark.gpu
SL, WI, LIN = W.FLAG_SLOPES, W.FLAG_WAVE_ITER, W.FLAG_SI_LINEARIZED


@pytest.mark.parametrize("flags", [SL | WI, LIN | WI])
@pytest.mark.parametrize("graph", [False, True])
def test_growth_with_the_wave_flux_of_every_iterate(flags, graph):
    p = _thin(1, flags=flags)
    ctx = ugkwp.from_problem(p, sort_interval=1000, extra_flags=ugkwp.FLAG_GRAPH if graph else 0)
    sim = oracle.Sim(p)
    ctx.step(8)
    sim.step(8)
    assert ctx.get_diag()["n_pushed"] > FIRST
    compare_state(ctx, sim, p, what="grown")


def test_growth_of_a_batch():
    probs = [_thin(1, seed=4 + k) for k in range(3)]
    ctx = ugkwp.from_batch(probs, pool_capacity=1 << 24, sort_interval=1000)
    ctx.step(4)
    assert ctx.get_diag()["n_pushed"] > FIRST
    for k, p in enumerate(probs):
        sim = oracle.Sim(p)
        sim.step(4)
        compare_state(ctx, sim, p, inst=k, what=f"grown batch instance {k}")
