"""GPU vs FP64 oracle on a 2-D mesh of a fixed opacity just above the size up to which every
sweep of the source iteration runs by patches of cells: the first sweep by patches, the
later ones a thread per slot.  The bar of the other parity tests."""
import pytest

from paper_2312_16981_amd import workloads as W
from test_gpu_grid import _mesh
from test_gpu_parity import run_pair

pytestmark = pytest.mark.gpu
LIN, SL, WI, BP = W.FLAG_SI_LINEARIZED, W.FLAG_SLOPES, W.FLAG_WAVE_ITER, W.FLAG_BOUNDARY_PARTICLES


@pytest.mark.parametrize("flags", [0, LIN, WI, SL | WI | BP, LIN | SL | WI | BP])
def test_sweeps_above_the_patches_size(flags):
    nx, ny, G = 112, 110, 32
    assert nx * ny * G > 256 * 3 * 512
    run_pair(_mesh(nx, ny, G, flags=flags, w_ref=1e-4, pool_cap=1 << 24), 2)
