"""1-D batches whose material model is set after the context exists (Olson's heat capacity,
an opacity table), with the wave flux of every iterate: the sweeps that hold the most in
LDS.  Against the FP64 oracle at the bar of the other parity tests, and against contexts
of one instance where the model comes and goes between steps."""
import numpy as np
import pytest

import oracle
from paper_2312_16981_amd import ugkwp
from paper_2312_16981_amd import workloads as W
from test_gpu_parity import compare_state, say

pytestmark = pytest.mark.gpu
SL, WI, LIN = W.FLAG_SLOPES, W.FLAG_WAVE_ITER, W.FLAG_SI_LINEARIZED
SIZES = [(1, 64), (97, 33), (260, 16), (19, 5), (70, 64)]


def _slab(k, nx, G, flags):
    return W.slab(nx, G, lambda x: np.where(x < 0.45, 0.3, 80.0), dt=1e-3, steps=0, w_ref=4e-5, seed=70 + k,
                  pool_cap=1 << 18, flags=flags, name=f"bm{k}")


def _olson(p, k):
    return p.with_(olson_H=np.full(p.nx, 0.05 + 0.1 * k), olson_chi=np.full(p.nx, 0.2))


def _table(p):
    nu, T = W.opacity_nodes()
    sigma = np.stack([1e-3 * W.foam_kappa(nu, T), 1e-3 * W.aluminium_kappa(nu, T)])
    return p.with_(opacity_table={"mat": (np.arange(p.nx) % 3 == 0).astype(np.int32), "nu": nu, "T": T, "sigma": sigma},
                   kappa=np.zeros((p.nx, p.G)))


@pytest.mark.parametrize("flags", [LIN | WI, LIN | SL | WI])
@pytest.mark.parametrize("model", ["olson", "table", "olson_table"])
def test_models_with_the_wave_flux_of_every_iterate(model, flags):
    probs = []
    for k, (nx, G) in enumerate(SIZES):
        p = _slab(k, nx, G, flags)
        if "olson" in model:
            p = _olson(p, k)
        if "table" in model:
            p = _table(p)
        probs.append(p)
    ctx = ugkwp.from_batch(probs)
    sims = [oracle.Sim(q) for q in probs]
    ctx.step(6)
    for s in sims:
        s.step(6)
    say("[models] sweeps", [s.diag()["sweeps"] for s in sims])
    for k, (q, s) in enumerate(zip(probs, sims)):
        compare_state(ctx, s, q, inst=k, what=f"{model} instance {k}")


@pytest.mark.parametrize("flags", [0, LIN | SL | WI])
def test_model_set_and_taken_back_between_steps(flags):
    probs = [_slab(k, nx, G, flags) for k, (nx, G) in enumerate(SIZES)]
    H = [np.full(p.nx, 0.05 + 0.1 * k) for k, p in enumerate(probs)]
    ctx = ugkwp.from_batch(probs)
    one = [ugkwp.from_problem(p) for p in probs]
    for on in (False, True, False, True):
        ctx.set_heat_capacity(np.concatenate(H) if on else None, np.concatenate([0.2 + 0 * h for h in H]) if on else None)
        for c, h in zip(one, H):
            c.set_heat_capacity(h if on else None, 0.2 + 0 * h if on else None)
        ctx.step(2)
        for k, c in enumerate(one):
            c.step(2)
            for a, b in zip(ctx.get_fields(k), c.get_fields()):
                assert np.max(np.abs(a - b)) <= 1e-10 * max(np.max(np.abs(b)), 1e-300)
