"""A one-launch CG that gives up: the solve goes on with the launched kernels,
the context says so, and after some solves it tries again."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

HOLD = 64


# plain CG over several work-groups; multigrid whose dense coarsest solve other work-groups share
@pytest.mark.parametrize("solver,nx,ny", [(1, 96, 56), (0, 80, 30)])
def test_a_fall_back_shows_and_ends(solver, nx, ny):
    from paper_1610_03918_amd import Pic
    w = synth.trench(nx=nx, ny=ny, width=max(2, ny // 8), depth=nx // 8, ppc=2, seed=71, rtol=1e-8)
    parts = synth.load(w)
    pic = Pic(w, parts, solver=solver, max_iter=50000, sort_interval=(0, 0))
    assert pic.pic_cg_pass_info() == (True, 0)
    for _ in range(4):                         # the length of a pass follows the solves before: let it settle
        want = pic.pic_solve(0)
    phi = pic.phi.cpu().numpy()
    pic.pic_set_cg_pass(-1)                    # a launch that has to wait gives up
    seen = []
    for _ in range(HOLD + 1 + 2 * HOLD + 1):
        pic.pic_solve(0)
        seen.append(pic.pic_cg_pass_info())
    # the first solve, the first after 64 others and the first after twice as many
    tries = (0, HOLD + 1)
    for k, (one, n) in enumerate(seen):
        assert n == sum(k >= t for t in tries), k
        assert one == (k in (HOLD, 3 * HOLD + 1)), k
    assert np.array_equal(pic.phi.cpu().numpy(), phi)
    pic.pic_set_cg_pass(1)
    assert pic.pic_cg_pass_info() == (True, 2)
    got = pic.pic_solve(0)
    assert pic.pic_cg_pass_info() == (True, 2)
    assert np.array_equal(pic.phi.cpu().numpy(), phi) and got["converged"] and want["converged"]
    pic.close()


def test_where_no_launch_fits_the_info_says_so():
    from paper_1610_03918_amd import Pic
    w = synth.trench(nx=256, ny=128, width=8, depth=32, ppc=1, seed=72)
    pic = Pic(w, synth.load(w), sort_interval=(0, 0))
    assert pic.pic_cg_pass_info() == (False, 0)
    pic.start()
    assert pic.pic_cg_pass_info() == (False, 0)
    pic.close()
