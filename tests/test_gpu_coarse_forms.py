"""The forms of the coarse-level kernel and the launches that a batch shares.

Alone, a grid's coarse levels run with positions looked up once per launch
(the grids sit at the limits of what a thread holds, and past them), and its
middle levels in a launch of their own; beside a grid too small for that form
in a batch, they run with positions computed in every phase, in launches that
both grids share.  Arithmetic and order are the same, so the potential is the
same bit for bit."""
from dataclasses import replace

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def grid(kind, nx, ny):
    if kind == "trench":
        return synth.trench(nx=nx, ny=ny, width=max(2, ny // 8), depth=nx // 8, ppc=1, seed=41, rtol=1e-9)
    base = synth.periodic_square if kind == "periodic" else synth.bounded_square
    return replace(base(n=nx, ppc=1, seed=42), ny=ny, cell_cond=np.zeros((nx, ny), np.uint8), rtol=1e-9)


# first LDS level of 64 x 64 pairs of a node less, odd and even extents on bounded axes, 128 x 48 = 3072 pairs and one
# column more, 128 x 65 of the trench, 128 x 80 = 5120 pairs, three fine levels
@pytest.mark.parametrize("kind,nx,ny", [
    ("periodic", 128, 128), ("bounded", 255, 200), ("bounded", 130, 255), ("periodic", 256, 96), ("trench", 256, 97),
    ("trench", 512, 256), ("periodic", 256, 160), ("trench", 1024, 256), ("bounded", 300, 700)])
def test_forms_of_the_coarse_levels_agree(kind, nx, ny):
    from paper_1610_03918_amd import Pic, PicBatch
    w, small = grid(kind, nx, ny), grid("periodic", 8, 8)
    parts = synth.load(w)
    alone = Pic(w, parts, sort_interval=(0, 0))
    alone.start()
    beside = PicBatch([w, small], [parts, synth.load(small)], sort_interval=(0, 0))
    beside.start()
    # (of the first solve: the length of a later one's first pass follows the slowest instance of a batch)
    a, b = alone.phi.cpu().numpy(), beside.phi(0).cpu().numpy()
    assert np.isfinite(a).all() and np.abs(a).max() > 0
    assert np.array_equal(a, b)
    alone.close()
    beside.close()
