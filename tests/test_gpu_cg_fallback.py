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


def few_particles(nx, ny):
    w = synth.trench(nx=nx, ny=ny, width=max(2, ny // 8), depth=nx // 8, ppc=1, seed=73, rtol=1e-6)
    return w, [{k: v[::29].copy() for k, v in p.items()} for p in synth.load(w)]


def same(x, y):
    assert repr(x[0]) == repr(y[0])                # (repr: a residual may be NaN)
    assert np.array_equal(x[1], y[1], equal_nan=True)


# one work-group; several, with one to nine wavefronts each.  1e40: the float32 residual overflows, so that no step
# length is finite.  1e-37: products r z = r^2 / 4 whose float32 z underflows
@pytest.mark.parametrize("nx,ny", [(40, 24), (96, 56), (1024, 512)])
@pytest.mark.parametrize("scale", [1e40, 1e-37])
def test_extreme_sources_as_the_launched_kernels(nx, ny, scale):
    """A pass whose step is not finite is left to the launched kernels, and counts as no fall-back."""
    from paper_1610_03918_amd import Pic
    w, few = few_particles(nx, ny)
    out = {}
    for mode in (0, 1):
        pic = Pic(w, few, solver=1, max_iter=256, sort_interval=(0, 0))
        pic.pic_set_cg_pass(mode)
        pic.b.mul_(scale)
        out[mode] = [(pic.pic_solve(0, allow_unconverged=True), pic.phi.cpu().numpy()) for _ in range(2)]
        assert pic.pic_cg_pass_info() == (mode == 1, 0)
        pic.close()
    for x, y in zip(out[0], out[1]):
        same(x, y)


@pytest.mark.parametrize("mode", [1, -1])
def test_the_iteration_limit_after_a_pass_run_again(mode):
    """Where max_iter cuts a solve short follows the lengths of earlier passes: a first pass that the launched kernels
    ran in the one launch's place counts as a first pass."""
    from paper_1610_03918_amd import Pic
    w, few = few_particles(256, 200)
    out = {}
    for m in (0, mode):
        pic = Pic(w, few, solver=1, max_iter=200, rtol=1e-12, sort_interval=(0, 0))
        pic.pic_set_cg_pass(m)
        b = pic.b.clone()
        if mode == 1:
            pic.b.mul_(1e40)
            pic.pic_solve(0, allow_unconverged=True)
            pic.b.copy_(b)
        out[m] = [(pic.pic_solve(0, allow_unconverged=True), pic.phi.cpu().numpy()) for _ in range(3)]
        pic.close()
    assert not out[0][0][0]["converged"]
    for x, y in zip(out[0], out[mode]):
        same(x, y)
