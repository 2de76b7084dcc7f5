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


# every work-group of a one-launch solve has to be on the device at once: 256 of a plain CG pass (1024 x 512, nine
# wavefronts each), 25 (96 x 56), the 17 that share a dense solve (80 x 30)
@pytest.mark.parametrize("kinds", [[(1, 1024, 512), (1, 1024, 512)], [(1, 1024, 512), (0, 80, 30), (1, 96, 56)],
                                   [(0, 80, 30), (0, 80, 30), (0, 64, 48), (0, 256, 128)]])
def test_contexts_on_streams_of_their_own_step_at_once(kinds):
    """Contexts stepped from threads, each on its own stream, end as each does alone."""
    import threading

    import torch

    from paper_1610_03918_amd import Pic

    def make(solver, nx, ny):
        w = synth.trench(nx=nx, ny=ny, width=max(2, ny // 8), depth=nx // 8, ppc=2, seed=82, rtol=1e-8)
        few = [{k: v[::5].copy() for k, v in p.items()} for p in synth.load(w)]
        return Pic(w, few, solver=solver, max_iter=50000)

    def steps(pic):
        pic.start()
        for _ in range(4):
            pic.pic_step(3)

    def result(pic):
        return [pic.phi.cpu().numpy(), *(pic.rho(s).cpu().numpy() for s in range(2))]

    alone = []
    for kind in kinds:
        pic = make(*kind)
        steps(pic)
        alone.append(result(pic))
        pic.close()
    pics = []
    for kind in kinds:
        with torch.cuda.stream(torch.cuda.Stream()):
            pics.append(make(*kind))
    wrong = []

    def body(pic):
        try:
            steps(pic)
        except Exception as e:
            wrong.append(e)

    threads = [threading.Thread(target=body, args=(pic,)) for pic in pics]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
    torch.cuda.synchronize()
    for pic, want in zip(pics, alone):
        assert pic.pic_cg_pass_info()[1] == 0
        assert all(np.array_equal(a, b) for a, b in zip(result(pic), want))
        pic.close()
