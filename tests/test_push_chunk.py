"""The particles per thread block of the push: what the caller asks for, or,
where the choice is left to the library, as few whole passes of 1024 particles
as make at most 1536 blocks of all the context's particles.  The block
size changes no result."""
import ctypes as C

import numpy as np
import pytest

import oracle
import synth
from gpu_util import canonical, live


def _workspace(chunk, cap):
    from paper_1610_03918_amd import pic
    cfg, cc = pic.make_config(synth.workload_for_tests("trench"), chunk=chunk)
    n = C.c_size_t(0)
    assert pic.lib().pic_workspace_size(C.byref(cfg), (C.c_int64 * 2)(*cap), C.byref(n)) == 0
    return n.value


def test_a_callers_chunk_is_laid_out_as_it_is():
    """The table of push blocks (16 bytes each) shrinks with the chunk, however few particles there are, and
    has room for the smallest blocks where the library chooses."""
    cap = [200_000, 200_000]
    size = {c: _workspace(c, cap) for c in (256, 1024, 4096, 8192, 0)}
    for small, large in ((256, 1024), (1024, 4096), (4096, 8192)):
        blocks = sum(-(-n // small) - -(-n // large) for n in cap)
        assert abs(size[small] - size[large] - 16 * blocks) <= 2 * 256, (small, large)
    assert size[0] == size[1024]


# 16 x 16 tiles of 10240 particles: several passes of a block, blocks that start and end inside a pass and (1001) at
# no multiple of four; the last is the library's choice
@pytest.mark.gpu
@pytest.mark.parametrize("unroll", [1, 4])
@pytest.mark.parametrize("chunk", [256, 1001, 2500, 4096, 8192, 0])
def test_block_sizes_against_the_oracle(chunk, unroll):
    from paper_1610_03918_amd import Pic
    w = synth.trench(nx=64, ny=48, width=6, depth=16, ppc=40, seed=51, rtol=1e-9)
    parts = synth.load(w)
    pic = Pic(w, parts, chunk=chunk, push_unroll=unroll, sort_interval=(2, 3))
    assert pic.pic_push_chunk() == (chunk or 1024)
    nc = oracle.node_cond(w)
    phi = synth.random_potential(w, 52, 3.0)
    post = [{k: v.copy() for k, v in p.items()} for p in parts]
    tally, surf = np.zeros((2, 9), np.int64), np.zeros(w.ny, np.int64)
    Ex, Ey = oracle.field(w, nc, phi)
    for _ in range(4):
        pic.phi.copy_(pic.torch.from_numpy(phi))
        pic.pic_push()
        for s in range(2):
            oracle.push(w, s, post[s], Ex, Ey, "f32", tally[s], surf if s == 1 else None)
    for s in range(2):
        assert np.array_equal(canonical(live(pic.particles_numpy(s))), canonical(live(post[s])))
        assert np.array_equal(pic.rho(s).cpu().numpy(), oracle.deposit(w, post[s]))
    assert np.array_equal(np.array(pic.pic_diagnostics()["tally"]), tally)
    pic.close()


@pytest.mark.gpu
def test_the_librarys_choice_counts_the_contexts_particles():
    """Of every instance and species, and of particles rather than of the room for them."""
    from paper_1610_03918_amd import Pic, PicBatch
    ws = [synth.periodic_square(n=64, ppc=90, seed=60 + k) for k in range(3)]
    parts = [synth.load(w) for w in ws]
    n = sum(p["cell"].size for p in parts[0])
    assert n == 737_280                                       # 3 n is more than one pass for each of 1536 blocks
    one = Pic(ws[0], parts[0], capacity=(3_000_000, 3_000_000))
    assert one.pic_push_chunk() == 1024
    one.close()
    three = PicBatch(ws, parts)
    assert [three.pic_push_chunk(i) for i in range(3)] == [2048] * 3
    three.close()
    asked = PicBatch(ws, parts, chunk=3000)
    assert [asked.pic_push_chunk(i) for i in range(3)] == [3000] * 3
    asked.close()
