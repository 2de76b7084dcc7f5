"""Several live contexts in one process."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_a_smaller_grid_leaves_a_larger_ones_launch_alone():
    """The one-launch solve of two grids that share a kernel and need different amounts of LDS, both above 64 KiB
    (64 x 64 nodes about 130 KiB, 40 x 40 about 80): the larger one's limit stands when the smaller comes after it."""
    from paper_1610_03918_amd import Pic
    ws = [synth.periodic_square(n=n, ppc=4, seed=81) for n in (64, 40)]
    parts = [synth.load(w) for w in ws]
    alone = []
    for w, p in zip(ws, parts):
        pic = Pic(w, p, sort_interval=(0, 0))
        pic.start()
        pic.pic_step(3)
        alone.append(pic.phi.cpu().numpy())
        pic.close()
    pics = [Pic(w, p, sort_interval=(0, 0)) for w, p in zip(ws, parts)]
    for pic in pics:
        pic.start()
    for _ in range(3):
        for pic in pics:
            pic.pic_step(1)
    for k, pic in enumerate(pics):
        assert pic.pic_cg_pass_info() == (True, 0), k
        assert np.array_equal(pic.phi.cpu().numpy(), alone[k]), k
        pic.close()
