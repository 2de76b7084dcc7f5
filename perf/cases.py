"""Performance cases of the framework: what its users run, through its public entry points.

Four kinds of work, over the range that the repository's configurations, tests and benchmark cover:

  step    one instance advanced by a re-binning period of steps (solve, field, push, deposit, assembly,
          re-binning), then its diagnostics: from the paper's 80 x 30 trench, where launches and host
          round trips count, to the benchmark's 1024 x 512 trench with 183.9M particles
  batch   a trench-width sweep advanced as captured graphs
  solve   one field solve by plain CG from the learned start: the potential's extrapolation in time, the
          network's input, its inference, the corrected start, the solve
  unet    the warm start's network alone: one inference, or one training step

A case is a dict of plain values.  Particle order in storage is not a result of the method, so a step's
outputs are the charge of both species on every node (exact integers over every particle's position), the
potential, the right-hand side and the diagnostics (kinetic energy, hit classes, impact angles).
"""
from __future__ import annotations

import math
from dataclasses import replace

import numpy as np
import torch

import synth
from paper_1610_03918_amd import Pic, PicBatch
from paper_1610_03918_amd.learned import sample, start_guess, start_of, window
from paper_1610_03918_amd.unet import UNet

DEV = "cuda:0"
CHANNELS = (16, 32, 64, 128)


# ---- cases ----------------------------------------------------------------

def listed():
    return [
        # the paper's wide trench (Sec. III.C), ions recycled: the smallest run, bound by latency
        {"name": "step_paper_trench_80x30", "kind": "step", "geometry": "paper_trench", "width": 15, "nx": 80,
         "ny": 30, "ppc": 100, "see": False, "steps": 16, "sort_e": 8, "sort_i": 64, "halo": 4},
        # the periodic plasma of the cold-oscillation checks, 1e-10 residual
        {"name": "step_periodic_64", "kind": "step", "geometry": "periodic", "width": 0, "nx": 64, "ny": 64,
         "ppc": 16, "see": False, "steps": 16, "sort_e": 8, "sort_i": 64, "halo": 4},
        # four grounded walls, 13M particles
        {"name": "step_bounded_256", "kind": "step", "geometry": "bounded", "width": 0, "nx": 256, "ny": 256,
         "ppc": 100, "see": False, "steps": 16, "sort_e": 8, "sort_i": 64, "halo": 4},
        # the benchmark's trench with its tuned schedule
        {"name": "step_trench_1024x512", "kind": "step", "geometry": "trench", "width": 8, "nx": 1024, "ny": 512,
         "ppc": 200, "see": False, "steps": 16, "sort_e": 16, "sort_i": 128, "halo": 5},
        # the three grid sizes of the trench-width sweep, as one batch of captured steps
        {"name": "batch_sweep_6", "kind": "batch", "widths": "1,4,16,32,48,96", "ppc": 64, "steps": 16,
         "sort_e": 16, "sort_i": 128, "halo": 5},
        # the learned start on the small test trench and on the benchmark's
        {"name": "solve_learned_96x56", "kind": "solve", "nx": 96, "ny": 56, "width": 6, "points": 4, "rtol": 1e-8},
        {"name": "solve_learned_1024x512", "kind": "solve", "nx": 1024, "ny": 512, "width": 8, "points": 4,
         "rtol": 1e-8},
        # inference inside one solve: batch 1, the two grids above (the periodic axis spanned whole)
        {"name": "unet_infer_96x56", "kind": "unet", "train": False, "B": 1, "H": 96, "W": 56, "wrap": True},
        {"name": "unet_infer_1024x512", "kind": "unet", "train": False, "B": 1, "H": 1024, "W": 512, "wrap": True},
        # training steps: the test trench's network, and the benchmark's batch
        {"name": "unet_train_b8_96x56", "kind": "unet", "train": True, "B": 8, "H": 96, "W": 56, "wrap": True},
        {"name": "unet_train_b4_1024x512", "kind": "unet", "train": True, "B": 4, "H": 1024, "W": 512,
         "wrap": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "batch", "solve", "unet", "unet"])
    if kind == "step":
        geometry = rng.choice(["paper_trench", "periodic", "bounded", "trench", "trench"])
        sort_e = rng.choice([8, 16])
        c = {"kind": "step", "geometry": geometry, "width": 0, "see": False, "steps": 16, "sort_e": sort_e,
             "sort_i": 8 * sort_e, "halo": rng.choice([4, 5])}
        if geometry == "paper_trench":
            c.update(nx=80, ny=30, width=rng.randint(3, 20), ppc=_log_int(rng, 20, 400), see=rng.random() < 0.5)
            return c
        # sizes that the multigrid halves several times, and any others (odd ones among them)
        if geometry == "periodic":
            nx = ny = 8 * _log_int(rng, 4, 48)
        elif geometry == "bounded":
            nx, ny = 4 * _log_int(rng, 6, 96), 4 * _log_int(rng, 6, 96)
        else:
            nx, ny = 8 * _log_int(rng, 8, 128), 8 * _log_int(rng, 4, 64)
            if rng.random() < 0.25:
                nx, ny = nx + rng.randint(1, 7), ny + rng.randint(1, 7)
            c["width"] = rng.randint(1, max(1, ny // 6))
        c.update(nx=nx, ny=ny, ppc=min(_log_int(rng, 12, 200), max(12, 30_000_000 // (nx * ny))))
        return c
    if kind == "batch":
        widths = sorted(rng.sample(synth.SWEEP_WIDTHS[:14], rng.randint(2, 8)))
        return {"kind": "batch", "widths": ",".join(str(x) for x in widths), "ppc": _log_int(rng, 12, 64),
                "steps": 16, "sort_e": 16, "sort_i": 128, "halo": 5}
    if kind == "solve":
        nx, ny = 8 * _log_int(rng, 8, 96), 8 * _log_int(rng, 4, 48)
        return {"kind": "solve", "nx": nx, "ny": ny, "width": rng.randint(2, max(2, ny // 6)),
                "points": rng.choice([2, 3, 4, 5]), "rtol": 1e-8}
    H, W = 8 * _log_int(rng, 4, 128), 8 * _log_int(rng, 3, 64)
    train = rng.random() < 0.5
    B = max(1, min(64, _log_int(rng, 1, 64), (1 << 21) // (H * W))) if train else rng.choice([1, 1, 2])
    return {"kind": "unet", "train": train, "B": B, "H": H, "W": W, "wrap": rng.random() < 0.6}


# ---- inputs ---------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _particles(w, gen):
    """The paper's load (uniform offsets in every plasma cell, Gaussian velocities of each species'
    thermal speed), drawn on the GPU, as the host arrays that Pic takes."""
    codes = torch.from_numpy(synth.cell_codes(w.cell_cond)).to(DEV)
    out = []
    for sp in w.species:
        n = codes.numel() * sp.ppc
        p = {"cell": codes.repeat_interleave(sp.ppc).cpu().numpy()}
        for f in ("ox", "oy"):
            p[f] = torch.rand(n, generator=gen, device=DEV).cpu().numpy()
        for f in ("vx", "vy"):
            p[f] = (torch.randn(n, generator=gen, device=DEV) * sp.vth).cpu().numpy()
        out.append(p)
    return out


def _workload(case, seed):
    if case["geometry"] == "paper_trench":
        w = synth.paper_trench(case["width"], ppc=case["ppc"], seed=seed)
        if case["see"]:
            w = replace(w, see_yield=(0.2, 0.2), see_vth=0.4472)
        return w
    if case["geometry"] == "periodic":
        return synth.periodic_square(n=case["nx"], ppc=case["ppc"], seed=seed)
    if case["geometry"] == "bounded":
        w = synth.bounded_square(n=case["nx"], ppc=case["ppc"], seed=seed)
        return replace(w, ny=case["ny"], cell_cond=np.zeros((case["nx"], case["ny"]), np.uint8))
    return synth.trench(nx=case["nx"], ny=case["ny"], width=case["width"], depth=max(2, case["nx"] // 8),
                        ppc=case["ppc"], seed=seed)


def _prepare_step(case, seed):
    w = _workload(case, seed)
    parts = _particles(w, _generator(seed))
    capacity = None
    if case["see"]:
        # room for the emitted electrons
        capacity = (parts[0]["cell"].size + 200_000, parts[1]["cell"].size)
    pic = Pic(w, parts, capacity=capacity, sort_interval=(case["sort_e"], case["sort_i"]), halo=case["halo"])
    pic.start()
    return {"kind": "step", "pic": pic, "steps": case["steps"]}


def _prepare_batch(case, seed):
    ws = [replace(synth.sweep_instance(int(x), ppc=case["ppc"]), seed=seed + k)
          for k, x in enumerate(case["widths"].split(","))]
    gen = _generator(seed)
    batch = PicBatch(ws, [_particles(w, gen) for w in ws], sort_interval=(case["sort_e"], case["sort_i"]),
                     halo=case["halo"])
    batch.start()
    batch.pic_step(2)
    return {"kind": "batch", "batch": batch, "steps": case["steps"]}


def _trench_fixed(nx, ny, width):
    """Node types of synth.trench: 0 free, 1 the grounded plate, 2 the RF electrode (y periodic)."""
    top, lo = nx - max(2, nx // 8), (ny - width) // 2
    fixed = torch.zeros((nx + 1, ny), dtype=torch.int64)
    fixed[0] = 1
    fixed[top:] = 2
    fixed[top:nx, lo + 1:lo + width] = 0
    return fixed


def _problem(case, seed):
    """A solve's data in float64: right-hand side, the potentials of the last steps (latest first) and the
    solution.  The potential is a sheath-like profile that follows the RF drive, with smooth waves that
    drift in time and a rough part of its own at each step (the particles' noise)."""
    nx, ny, K = case["nx"], case["ny"], case["points"]
    gen = _generator(seed)
    fixed = _trench_fixed(nx, ny, case["width"]).to(DEV)
    top = nx - max(2, nx // 8)
    x = torch.arange(nx + 1, dtype=torch.float64, device=DEV)[:, None] / top
    y = torch.arange(ny, dtype=torch.float64, device=DEV)[None, :] * (2 * math.pi / ny)
    mode = torch.rand((12, 3), generator=gen, device=DEV, dtype=torch.float64).tolist()
    seen = []
    for k in range(K + 1):
        t = 40.0 + 20 * mode[0][0] - 0.1 * k
        v = 50.0 * math.sin(0.05 * t)
        phi = v * x.clamp(max=1.0) ** 8 + 6.0 * torch.sin(math.pi * x.clamp(max=1.0)) + 0 * y
        for m, (a, p, q) in enumerate(mode):
            kx, ky = 1 + m % 4, m // 4
            phi = phi + (0.5 * a * math.sin(0.3 * t * (1 + q) + 6 * p)
                         * torch.sin(math.pi * kx * x.clamp(max=1.0)) * torch.cos(ky * y + 6 * q))
        rough = torch.randn((nx + 1, ny), generator=gen, device=DEV, dtype=torch.float64)
        for _ in range(2):
            rough = 0.5 * rough + 0.25 * (rough.roll(1, 1) + rough.roll(-1, 1))
            rough = 0.5 * rough + 0.25 * (rough.roll(1, 0) + rough.roll(-1, 0))
        phi = phi + 0.05 * rough
        phi = torch.where(fixed == 1, 0.0, torch.where(fixed == 2, v, phi))
        seen.append(phi.contiguous())
    now, free = seen[0], fixed == 0
    # A phi on free nodes with the conductors' values on the right-hand side's Dirichlet nodes (eq. 5)
    inner = torch.where(free, now, 0.0)
    near = inner.roll(1, 1) + inner.roll(-1, 1)
    near[1:] += inner[:-1]
    near[:-1] += inner[1:]
    b = torch.where(free, 4.0 * inner - near, now).contiguous()
    return b, seen[1:], now, free


def _params(gen):
    """He-normal weights, small biases, in the network's parameter order."""
    out, cin = [], 3
    shapes = []
    for l, c in enumerate(CHANNELS):
        shapes += [(cin, c), (c, c)]
        cin = c
    for l in (2, 1, 0):
        shapes += [(cin + CHANNELS[l], CHANNELS[l]), (CHANNELS[l], CHANNELS[l])]
        cin = CHANNELS[l]
    for ci, co in shapes:
        out.append(torch.randn((co, 3, 3, ci), generator=gen, device=DEV) * math.sqrt(2.0 / (9 * ci)))
        out.append(torch.randn((co,), generator=gen, device=DEV) * 0.05)
    out.append(torch.randn((16,), generator=gen, device=DEV) * 0.25)
    out.append(torch.randn((1,), generator=gen, device=DEV) * 0.05)
    return out


def _flat(ps):
    return torch.cat([p.reshape(-1) for p in ps])


def _images(case, gen):
    """Network inputs as the residual samples hold them: the scaled residual, zero where the node map holds
    a conductor, the free-node mask, the scaled conductor potentials; and targets of unit size."""
    B, H, W = case["B"], case["H"], case["W"]
    free = torch.ones((B, H, W), device=DEV)
    free[:, 0] = 0
    free[:, H - H // 8:] = 0
    free[:, H - H // 8:, W // 2 - W // 16:W // 2 + W // 16 + 1] = 1
    x = torch.stack([torch.randn((B, H, W), generator=gen, device=DEV) * free, free,
                     (1 - free) * torch.rand((B, 1, 1), generator=gen, device=DEV)], -1).to(torch.bfloat16)
    t = torch.randn((B, H, W), generator=gen, device=DEV)
    for _ in range(3):
        t = (t + t.roll(1, 1) + t.roll(1, 2)) / math.sqrt(3.0)
    return x.contiguous(), (t * free).to(torch.bfloat16).contiguous()


def _prepare_solve(case, seed):
    b, hist, now, free = _problem(case, seed)
    w = synth.trench(nx=case["nx"], ny=case["ny"], width=case["width"], depth=max(2, case["nx"] // 8), ppc=1,
                     rtol=case["rtol"])
    few = [{k: v[::97].copy() for k, v in p.items()} for p in synth.load(w)]
    pic = Pic(w, few, solver=1, max_iter=50000)
    pic.b.copy_(b)
    pic.phi.copy_(torch.where(free, hist[0], now))
    H, W = window(w)
    net = UNet(1, H, W, params=_flat(_params(_generator(seed + 1))), periodic_w=W == w.NY)
    gap = float((hist[0] - now).square().mean().sqrt())
    return {"kind": "solve", "pic": pic, "net": net, "hist": hist, "H": H, "W": W, "points": case["points"],
            # the residual's size in, a correction well below the potential's change per step out
            "scales": (8.0, 1.0 / 64, 2.0 ** round(-math.log2(gap / 256))), "nodes": pic.pic_node_map(),
            "start": torch.empty_like(b), "guess": torch.empty_like(b)}


def _prepare_unet(case, seed):
    gen = _generator(seed)
    net = UNet(case["B"], case["H"], case["W"], params=_flat(_params(gen)), periodic_w=case["wrap"])
    x, t = _images(case, gen)
    if case["train"]:
        return {"kind": "train", "net": net, "x": x, "t": t}
    net.input().copy_(x)
    return {"kind": "infer", "net": net}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _prepare_step(case, seed)
    if kind == "batch":
        return _prepare_batch(case, seed)
    if kind == "solve":
        return _prepare_solve(case, seed)
    return _prepare_unet(case, seed)


# ---- one pass -------------------------------------------------------------

def _diagnostics(d):
    return {k: d[k] for k in ("alive", "charge", "tally", "surf_hits", "kinetic", "field_energy", "iad",
                              "see_emitted")}


def run(state):
    kind = state["kind"]
    if kind == "step":
        pic = state["pic"]
        pic.pic_step(state["steps"])
        d = _diagnostics(pic.pic_diagnostics())
        d["iad"] = np.asarray(d["iad"], np.int64)
        d["tally"] = np.asarray(d["tally"], np.int64)
        d["kinetic"] = np.asarray(d["kinetic"], np.float64)
        d["field_energy"] = np.asarray(d["field_energy"], np.float64)
        return {"rho_e": pic.rho(0), "rho_i": pic.rho(1), "phi": pic.phi, "b": pic.b, "diagnostics": d}
    if kind == "batch":
        batch = state["batch"]
        batch.pic_batch_step(state["steps"], 2, 12, 4, allow_unconverged=True)
        return [{"rho_e": batch.rho(i, 0), "rho_i": batch.rho(i, 1), "phi": batch.phi(i), "b": batch.b(i)}
                for i in range(batch.n)]
    if kind == "solve":
        pic, net, s, guess = state["pic"], state["net"], state["start"], state["guess"]
        start_of(state["hist"], state["points"], s)
        sample(1, pic.b, s, s, None, state["nodes"], (0, 1), state["H"], state["W"], state["scales"],
               net.input()[0])
        net.pic_unet_forward()
        start_guess(1, net, 0, s, s, state["nodes"], (0, 1), state["scales"][2], guess)
        pic.pic_solve(2, guess)
        return {"phi": pic.phi, "guess": guess, "output": net.output()}
    net = state["net"]
    if kind == "infer":
        net.pic_unet_forward()
        return {"output": net.output()}
    for slot in range(net.B):
        net.pic_unet_load(slot, state["x"][slot], state["t"][slot])
    loss = net.train_step(lr=1e-3)
    return {"loss": loss, "output": net.output(), "grads": net.grads, "params": net.params, "m": net.m, "v": net.v}


# ---- what a pass cannot do without ------------------------------------------

def _conv_flops():
    """Flops of one inference, per pixel of the full resolution."""
    per, cin = 2.0 * 16, 3
    for l, c in enumerate(CHANNELS):
        per += 2.0 * 9 * (cin * c + c * c) / 4 ** l
        cin = c
    for l in (2, 1, 0):
        per += 2.0 * 9 * ((cin + CHANNELS[l]) * CHANNELS[l] + CHANNELS[l] ** 2) / 4 ** l
        cin = CHANNELS[l]
    return per


PARAMS = 487297


def _step_work(cells, nodes, ppc, steps):
    # a step reads and writes 20 bytes of each particle, writes both charges, reads them for the source,
    # and reads and writes the potential
    return {"bytes": steps * (2 * cells * ppc * 40.0 + nodes * 48.0), "flops": steps * (2 * cells * ppc * 60.0
                                                                                        + nodes * 100.0)}


def work(case):
    kind = case["kind"]
    if kind == "step":
        w = _workload(case, 1)
        return _step_work(w.plasma_cells(), w.NX * w.NY, case["ppc"], case["steps"])
    if kind == "batch":
        parts = []
        for x in case["widths"].split(","):
            w = synth.sweep_instance(int(x), ppc=case["ppc"])
            parts.append(_step_work(w.plasma_cells(), w.NX * w.NY, case["ppc"], case["steps"]))
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind == "solve":
        nodes = (case["nx"] + 1) * case["ny"]
        # the right-hand side and the past potentials in, the start and the potential out
        return {"bytes": nodes * 8.0 * (3 + case["points"]) + 2 * PARAMS, "flops": nodes * (_conv_flops() + 100.0)}
    P = case["B"] * case["H"] * case["W"]
    if case["train"]:
        # input, target and mask in; parameters and both moments read and written, gradients written
        return {"bytes": P * 12.0 + PARAMS * 28.0, "flops": 3.0 * P * _conv_flops()}
    return {"bytes": P * 10.0 + 4 * PARAMS, "flops": P * _conv_flops()}


# ---- the same in 64 bits ------------------------------------------------------

def _conv(x, wt, bias, wrap):
    """3 x 3 convolution of [B, H, W, Cin] by [Cout, 3, 3, Cin], zero padding (circular along W with wrap), ReLU."""
    B, H, W, C = x.shape
    z = x.new_zeros((B, H, 1, C))
    left, right = (x[:, :, -1:], x[:, :, :1]) if wrap else (z, z)
    x = torch.cat([left, x, right], 2)
    z = x.new_zeros((B, 1, W + 2, C))
    x = torch.cat([z, x, z], 1)
    out = 0
    for dh in range(3):
        for dw in range(3):
            out = out + x[:, dh:dh + H, dw:dw + W].reshape(-1, C) @ wt[:, dh, dw].T
    return torch.relu(out + bias).reshape(B, H, W, -1)


def _pool(x):
    B, H, W, C = x.shape
    return x.reshape(B, H // 2, 2, W // 2, 2, C).mean((2, 4))


def _network(ps, x, wrap):
    h, skips = x, []
    for l in range(4):
        if l:
            h = _pool(h)
        for r in range(2):
            k = 2 * l + r
            h = _conv(h, ps[2 * k], ps[2 * k + 1], wrap)
        skips.append(h)
    for l in (2, 1, 0):
        k = 12 - 2 * l
        h = torch.cat([h.repeat_interleave(2, 1).repeat_interleave(2, 2), skips[l]], -1)
        h = _conv(h, ps[2 * k], ps[2 * k + 1], wrap)
        h = _conv(h, ps[2 * k + 2], ps[2 * k + 3], wrap)
    return h @ ps[28] + ps[29]


def exact(case, seed):
    if case["kind"] == "solve":
        _, _, now, _ = _problem(case, seed)
        return {"phi": now, "guess": None, "output": None}
    if case["kind"] != "unet":
        return None
    gen = _generator(seed)
    ps = [p.double().requires_grad_(case["train"]) for p in _params(gen)]
    x, t = _images(case, gen)
    out = _network(ps, x.double(), case["wrap"])
    if not case["train"]:
        return {"output": out}
    mask = x[..., 1].double()
    loss = (mask * (out - t.double()) ** 2).sum() / mask.sum()
    loss.backward()
    g = _flat([p.grad for p in ps])
    p0 = _flat([p.detach() for p in ps])
    m, v = 0.1 * g, 1e-3 * g * g
    new = p0 - 1e-3 * (m / 0.1) / ((v / 1e-3).sqrt() + 1e-8)
    return {"loss": float(loss), "output": out.detach(), "grads": g, "params": new, "m": m, "v": v}
