"""2-D sweeps whose opacity is a power of the iterate's temperature, on meshes of more
blocks than run at once: every block takes T^k of the cells around its own, also when
the blocks of those cells have already written T^{k+1}.  Without particles a run is the
same to the last bit each time, and within 1e-10 of the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2312_16981_amd import ugkwp
from paper_2312_16981_amd import workloads as W
from test_gpu_grid import _mesh
from test_gpu_parity import compare_state, say

pytestmark = pytest.mark.gpu
LIN = W.FLAG_SI_LINEARIZED
STEPS = 2


def _problems(batch, flags, stim):
    # 33 groups take 64 lanes a cell: 1530 blocks of the patches, 3030 of the batch's sweep
    p = [_mesh(120, 101, 33, flags=flags, T_power=0.5, opacity_stim=stim, w_ref=1e6)]
    if batch:
        p.append(_mesh(23, 37, 33, flags=flags, T_power=0.5, opacity_stim=stim, w_ref=1e6, seed=9))
    return p


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("flags,stim", [(0, 0), (LIN, 1)])
def test_iterate_of_the_cells_around(batch, flags, stim):
    probs = _problems(batch, flags, stim)
    runs = []
    for _ in range(3):
        ctx = ugkwp.from_batch(probs) if batch else ugkwp.from_problem(probs[0])
        ctx.step(STEPS)
        assert ctx.get_diag()["n_births"] == 0
        runs.append([ctx.get_fields(k) for k in range(len(probs))])
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            for u, v in zip(a, b):
                assert np.array_equal(u, v)
    for k, p in enumerate(probs):
        sim = oracle.Sim(p)
        sim.step(STEPS)
        say("[iterate] sweeps", sim.diag()["sweeps"])
        assert sim.diag()["sweeps"] >= 3
        compare_state(ctx, sim, p, inst=k, what=f"instance {k}")
