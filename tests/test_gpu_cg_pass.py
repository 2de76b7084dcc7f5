"""Plain CG as one launch per pass against the launched kernels: the same
potential bit for bit, the same iteration counts, and the fall-back when a
work-group does not wait."""
from dataclasses import replace

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def workload(kind, nx, ny):
    if kind == "periodic":
        w = synth.periodic_square(n=nx, ppc=3, seed=21)
        return replace(w, ny=ny, cell_cond=np.zeros((nx, ny), np.uint8))
    if kind == "bounded":
        w = synth.bounded_square(n=nx, ppc=3, seed=22)
        return replace(w, ny=ny, cell_cond=np.zeros((nx, ny), np.uint8))
    return synth.trench(nx=nx, ny=ny, width=max(2, ny // 8), depth=nx // 8, ppc=2, seed=23)


# one work-group: the smallest grid, a wrap inside one block of columns, two column blocks, ragged rows and
# columns, two blocks per wavefront; several work-groups: just past the limit, a ragged last block, two column
# blocks and more on each axis kind; chains of two, three and of sixteen blocks
@pytest.mark.parametrize("kind,nx,ny,solver", [
    ("periodic", 4, 4, 1), ("bounded", 6, 5, 0), ("trench", 40, 24, 1), ("periodic", 22, 65, 0),
    ("trench", 96, 56, 1), ("bounded", 63, 100, 1), ("trench", 132, 64, 1), ("periodic", 131, 70, 0),
    ("bounded", 200, 129, 0), ("trench", 256, 193, 0), ("trench", 1024, 128, 1), ("periodic", 514, 320, 1),
    ("trench", 2048, 512, 1)])
def test_one_launch_equals_the_launched_kernels(kind, nx, ny, solver):
    from paper_1610_03918_amd import Pic
    w = workload(kind, nx, ny)
    parts = synth.load(w)
    out = {}
    for mode in (0, 1, -1):
        pic = Pic(w, parts, solver=solver, max_iter=50000, rtol=1e-9, sort_interval=(0, 0))
        pic.pic_set_cg_pass(mode)
        infos = [pic.pic_solve(0)]
        pic.pic_rewind()
        for _ in range(2):
            pic.pic_push()
            infos.append(pic.pic_solve(3))
        out[mode] = (infos, pic.phi.cpu().numpy(), [pic.rho(s).cpu().numpy() for s in range(2)])
        pic.close()
    for mode in (1, -1):
        assert out[mode][0] == out[0][0], mode
        assert np.array_equal(out[mode][1], out[0][1]), mode
        assert all(np.array_equal(a, b) for a, b in zip(out[mode][2], out[0][2])), mode


@pytest.mark.parametrize("nx,ny", [(40, 24), (256, 200)])
@pytest.mark.parametrize("max_iter", [1, 17, 64])
def test_iteration_limit(nx, ny, max_iter):
    """A solve cut short by max_iter stops after the same iterations, with the same potential."""
    from paper_1610_03918_amd import Pic
    w = workload("trench", nx, ny)
    parts = synth.load(w)
    out = {}
    for mode in (0, 1):
        pic = Pic(w, parts, solver=1, max_iter=max_iter, rtol=1e-12, sort_interval=(0, 0))
        pic.pic_set_cg_pass(mode)
        info = pic.pic_solve(0, allow_unconverged=True)
        out[mode] = (info, pic.phi.cpu().numpy())
        pic.close()
    assert not out[0][0]["converged"]
    assert out[1][0] == out[0][0]
    assert np.array_equal(out[1][1], out[0][1])


# multigrid in one launch: one tile, ragged tiles, two tiles a thread and more, wraps on both axes, one coarse
# level and several, a coarsest level solved by one work-group, swept (no fixed node), and shared (41 x 15, 33 x 17)
@pytest.mark.parametrize("kind,nx,ny", [
    ("periodic", 8, 8), ("bounded", 16, 8), ("trench", 32, 24), ("periodic", 64, 64), ("trench", 64, 48),
    ("trench", 96, 56), ("bounded", 72, 72), ("periodic", 96, 48), ("trench", 128, 64), ("bounded", 64, 32),
    ("trench", 80, 30), ("trench", 64, 34), ("bounded", 100, 44), ("trench", 192, 40)])
def test_one_launch_multigrid_equals_the_launched_kernels(kind, nx, ny):
    from paper_1610_03918_amd import Pic
    w = workload(kind, nx, ny)
    parts = synth.load(w)
    out = {}
    for mode in (0, 1, -1):
        pic = Pic(w, parts, max_iter=2000, rtol=1e-11, sort_interval=(4, 0))
        pic.pic_set_cg_pass(mode)
        infos = [pic.pic_solve(0)]
        pic.pic_rewind()
        pic.pic_step(6)
        for kind_ in (1, 0, 3):
            infos.append(pic.pic_solve(kind_))
        out[mode] = (infos, pic.phi.cpu().numpy(), [pic.rho(s).cpu().numpy() for s in range(2)])
        pic.close()
    for mode in (1, -1):
        assert out[mode][0] == out[0][0], mode
        assert np.array_equal(out[mode][1], out[0][1]), mode
        assert all(np.array_equal(a, b) for a, b in zip(out[mode][2], out[0][2])), mode


@pytest.mark.parametrize("nx,ny", [(64, 48), (80, 30)])
@pytest.mark.parametrize("max_iter", [1, 5, 13])
def test_iteration_limit_multigrid(nx, ny, max_iter):
    from paper_1610_03918_amd import Pic
    w = workload("trench", nx, ny)
    parts = synth.load(w)
    out = {}
    for mode in (0, 1):
        pic = Pic(w, parts, max_iter=max_iter, rtol=1e-15, sort_interval=(0, 0))
        pic.pic_set_cg_pass(mode)
        infos = [pic.pic_solve(0, allow_unconverged=True) for _ in range(2)]
        out[mode] = (infos, pic.phi.cpu().numpy())
        pic.close()
    assert not out[0][0][0]["converged"]
    assert out[1][0] == out[0][0]
    assert np.array_equal(out[1][1], out[0][1])
