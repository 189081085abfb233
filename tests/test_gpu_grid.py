"""GPU vs FP64 oracle for the 2-D sweeps whose opacity follows the iterate, where the
patches of cells a block takes can go wrong: one cell, rows and columns, meshes around a
patch's sides for every number of lanes per cell, every wall, a power of the temperature
(with the stimulated-emission factor), and an opacity table with Olson's heat capacity.
Same bar as the other parity tests: integers and sweep counts equal, every field, tally
and particle within 1e-10 of its array's max-norm."""
import numpy as np
import pytest

from paper_2312_16981_amd import workloads as W
from test_gpu_parity import run_pair

pytestmark = pytest.mark.gpu
LIN, SL, WI, BP = W.FLAG_SI_LINEARIZED, W.FLAG_SLOPES, W.FLAG_WAVE_ITER, W.FLAG_BOUNDARY_PARTICLES


def _mesh(nx, ny, G, **kw):
    rng = np.random.default_rng(100 * nx + ny)
    ncell = nx * ny
    p = dict(dt=4e-3, w_ref=2e-4, pool_cap=1 << 18, seed=3, steps=0)
    p.update(kw)
    return W.Problem(name=f"grid{nx}x{ny}_g{G}", dim=2, nx=nx, ny=ny, x0=0.0, x1=0.1 * nx, y0=0.0, y1=0.12 * ny,
                     bc=[W.BC_PLANCK, W.BC_REFLECT, W.BC_VACUUM, W.BC_PLANCK], bcT=[1.0, 0.0, 0.0, 0.7],
                     nu_edges=W.log_edges(0.05, 10.0, G), kappa=np.exp(2.0 * rng.standard_normal((ncell, G))),
                     cv=np.ones(ncell), T0=np.full(ncell, 0.3), Tr0=np.full(ncell, 0.3),
                     pinned=(rng.random(ncell) < 0.1).astype(np.uint8), **p)


@pytest.mark.parametrize("nx,ny,G", [(1, 1, 1), (33, 17, 1), (16, 1, 2), (1, 17, 4), (9, 8, 7), (8, 5, 16),
                                     (5, 9, 24), (4, 4, 32), (7, 3, 33), (5, 4, 64)])
@pytest.mark.parametrize("flags,stim", [(0, 0), (LIN, 0), (LIN, 1), (LIN | SL | WI | BP, 0)])
def test_patches_power_opacity(nx, ny, G, flags, stim):
    run_pair(_mesh(nx, ny, G, flags=flags, T_power=0.5, opacity_stim=stim), 3)


@pytest.mark.parametrize("nx,ny,G", [(1, 1, 1), (17, 9, 8), (9, 5, 13), (5, 6, 32), (6, 3, 50), (3, 5, 64)])
@pytest.mark.parametrize("flags", [LIN, LIN | SL])
def test_patches_table_opacity(nx, ny, G, flags):
    nu, T = W.opacity_nodes()
    ncell = nx * ny
    rng = np.random.default_rng(ncell)
    table = {"mat": rng.integers(0, 2, ncell).astype(np.int32), "nu": nu, "T": T,
             "sigma": np.stack([1e-3 * W.foam_kappa(nu, T), 1e-3 * W.aluminium_kappa(nu, T)])}
    p = _mesh(nx, ny, G, flags=flags).with_(
        opacity_table=table, olson_H=np.where(rng.random(ncell) < 0.7, 0.3, 0.0), olson_chi=np.full(ncell, 0.2),
        kappa=np.zeros((ncell, G)))
    run_pair(p, 3)
