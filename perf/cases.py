"""Workloads the library is timed on: calls a user's program makes through the
public entry points, from the smallest fitness call to the 1024-instance
batched frame loop.  All inputs are synthetic and follow from the seed alone
(the generators of paper_2308_10169_amd.inputs).

A case is a dict of plain values; `kind` names the entry point:

  fit     sepso_fitness / sepso_fitness_noalloc on device tensors
  frame   Planner.plan_frame: one planner, one application-phase frame
  batch   BatchPlanner.plan: one frame of many independent instances
  learned the same with the learned initializer attached
  evolve  Evolver.run: the evolution phase on a map
  bf      BFSwarm.step: one large benchmark-function swarm
  bfevo   BFEvolver.run: the evolution phase on a benchmark function
  train   LearnedInit.train: Adam steps on the device-resident training set
"""
from __future__ import annotations

import ctypes as C
import math

import numpy as np
import torch

from paper_2308_10169_amd import ablation, evolve, learned
from paper_2308_10169_amd import inputs as I
from paper_2308_10169_amd import sepso

ALPHA, BETA = I.PARAMS_PATH["alpha"], I.PARAMS_PATH["beta"]
FRAME_ITERS = 35  # iterations a truncated paper-shaped frame runs, on average (work estimates)


def listed():
    return [
        # the static single plan's swarm scored once (4 x 32 paths, 4 rectangles), no workspace:
        # a caller checking candidate paths in its own control loop; launches and latency
        dict(name="fit_static", kind="fit", paths=128, waypoints=8, rects=4, quads=0, stars=0, side=100.0,
             spread=0.1, noalloc=True),
        # the paper-shaped swarm scored once, near a previous plan (8 x 170 paths, 30 rectangles)
        dict(name="fit_paper", kind="fit", paths=1360, waypoints=20, rects=30, quads=0, stars=0, side=366.0,
             spread=0.1, noalloc=False),
        # the stress scene's whole fresh swarm scored once (8 x 4096 uniform paths, 2400 edges)
        dict(name="fit_stress", kind="fit", paths=32768, waypoints=64, rects=500, quads=100, stars=0,
             side=512.0, spread=1.0, noalloc=False),
        # the real-time loop: the paper-shaped dynamic scene, one planner, a frame per call
        dict(name="frame_paper", kind="frame", scene="dynamic", side=366.0, rects=30, groups=8,
             particles=170, waypoints=20, iters=50, at_mode=2, K=4, threads=256),
        # one large swarm on the stress scene (8 x 4096 particles, 64 waypoints, 600 obstacles)
        dict(name="frame_stress", kind="frame", scene="stress", side=512.0, rects=500, groups=8,
             particles=4096, waypoints=64, iters=50, at_mode=2, K=12, threads=256),
        # planning as a service: 1024 uneven dynamic instances, one frame of all of them per call
        dict(name="batch_1024", kind="batch", instances=1024, K=8, threads=256),
        # the same loop with the network's proposals at every frame start
        dict(name="learned_256", kind="learned", instances=256, iters=50, K=12, threads=256),
        # offline tuning on the paper-shaped scene: 64 lower-level runs per evolution
        dict(name="evolve_paper", kind="evolve", scene="paper", h_groups=8, h_particles=8, particles=170,
             waypoints=20, iters=30, evolutions=5),
        # offline tuning on a benchmark function: 32 fresh 80 x 30 swarms of 1400 iterations
        dict(name="bfevo_rastrigin", kind="bfevo", func="rastrigin", h_groups=8, h_particles=4, particles=10,
             dims=30, iters=1400),
        # the paper's large swarm, 16384 x 1000 (its 1400-iteration run in slices of 50)
        dict(name="bf_large", kind="bf", func="rosenbrock", particles=2048, dims=1000, steps=50),
        # training at the default minibatch: many short steps
        dict(name="train_256", kind="train", batch=256, steps=100, samples=4096),
        # training at a throughput minibatch
        dict(name="train_8192", kind="train", batch=8192, steps=20, samples=16384),
    ]


def _log(rng, lo, hi):
    """Integer spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fit", "fit", "frame", "frame", "batch", "learned", "evolve", "bfevo", "bf", "train"])
    if kind == "fit":
        rects, quads, stars = _log(rng, 1, 500), rng.choice([0, _log(rng, 1, 100)]), rng.choice([0, 0, _log(rng, 1, 20)])
        W = rng.randint(1, 64)
        most = 32768 * 65 * 2400 // ((W + 1) * 4 * (rects + quads + 4 * stars))
        return dict(kind="fit", paths=min(most, _log(rng, 1, 32768)), waypoints=W, rects=rects, quads=quads,
                    stars=stars, side=float(rng.randint(128, 512)), spread=rng.choice([0.02, 0.1, 0.3, 1.0]),
                    noalloc=False)
    if kind == "frame":
        K, B = rng.choice([(4, 64), (4, 256), (8, 128), (8, 256)])
        return dict(kind="frame", scene="dynamic", side=float(rng.randint(100, 512)), rects=_log(rng, 4, 100),
                    groups=rng.choice([4, 8]), particles=_log(rng, 32, 1024), waypoints=rng.randint(8, 32),
                    iters=rng.choice([30, 50]), at_mode=rng.choice([0, 2]), K=K, threads=B)
    if kind == "batch":
        K, B = rng.choice([(4, 256), (8, 128), (8, 256)])
        return dict(kind="batch", instances=_log(rng, 8, 800), K=K, threads=B)
    if kind == "learned":
        return dict(kind="learned", instances=_log(rng, 16, 1024), iters=rng.choice([30, 50]), K=12, threads=256)
    if kind == "evolve":
        return dict(kind="evolve", scene=rng.choice(["paper", "ablation"]), h_groups=rng.choice([4, 8]),
                    h_particles=rng.randint(2, 8), particles=_log(rng, 32, 170), waypoints=rng.randint(8, 20),
                    iters=rng.choice([10, 30]), evolutions=rng.randint(1, 5))
    if kind == "bfevo":
        return dict(kind="bfevo", func=rng.choice(sorted(sepso.BF_FUNCS)), h_groups=rng.choice([4, 8]),
                    h_particles=rng.randint(2, 6), particles=rng.randint(5, 12), dims=rng.randint(8, 40),
                    iters=rng.randint(300, 1400))
    if kind == "bf":
        N, D = _log(rng, 16, 2048), _log(rng, 300, 1000)
        return dict(kind="bf", func=rng.choice(sorted(sepso.BF_FUNCS)), particles=N, dims=D,
                    steps=rng.randint(10, 50))
    batch = 32 * _log(rng, 2, 192)
    return dict(kind="train", batch=batch, steps=rng.randint(5, 20), samples=batch + rng.randint(0, batch))


# ---- inputs -----------------------------------------------------------------


def _fit_map(c, rng):
    S = c["side"]
    s, t = I.snap([0.04 * S, 0.06 * S]), I.snap([0.96 * S, 0.94 * S])
    polys = list(I.random_rects(rng, S, S, c["rects"], 0.01 * S, 0.04 * S if c["rects"] > 60 else 0.12 * S,
                                avoid=(s, t)))
    polys += list(I.random_quads(rng, S, S, c["quads"], 0.01 * S, 0.06 * S))
    polys += I.random_stars(rng, S, S, c["stars"], 0.03 * S, 0.1 * S)
    return I.make_map(S, S, polys, s, t)


def _fit_inputs(c, seed):
    """Map arrays and device paths: uniform in the map (a fresh swarm, spread
    1), or the straight line from start to target plus one smooth offset all
    paths share plus each path's own deviations of `spread` of the map (a
    swarm drawn around a previous plan)."""
    rng = np.random.default_rng([11, int(seed)])
    m = _fit_map(c, rng)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    n, W, S = c["paths"], c["waypoints"], c["side"]
    if c["spread"] >= 1.0:
        X = torch.rand((n, 2, W), generator=g, device="cuda") * S
    else:
        u = torch.linspace(0, 1, W + 2, device="cuda")[1:-1]
        s = torch.tensor(m.start, dtype=torch.float32, device="cuda")
        t = torch.tensor(m.target, dtype=torch.float32, device="cuda")
        line = s[:, None] + (t - s)[:, None] * u
        bend = 0.15 * S * torch.randn((2, 1), generator=g, device="cuda") * torch.sin(math.pi * u)
        X = line + bend + c["spread"] * S * 0.5 * torch.randn((n, 2, W), generator=g, device="cuda")
    return m, X.clamp(0.0, S).reshape(n, 2 * W).contiguous()


def _dynamic_specs(c, seed):
    specs, sws = [], []
    for i in range(c["instances"]):
        m, shape = I.batch_instance(i, seed)
        specs.append(m)
        sws.append(I.dynamic_swarm(m.scale, seed=seed, instance=i, **shape))
    return specs, sws


def prepare(case, seed):
    c, kind = case, case["kind"]
    seed = int(seed)
    if kind == "fit":
        m, X = _fit_inputs(c, seed)
        n, dev = c["paths"], "cuda"
        st = dict(kind=kind, c=c, X=X, n_vert=int(m.poly_ptr[-1]), n_polys=m.n_polys,
                  pptr=torch.from_numpy(np.ascontiguousarray(m.poly_ptr, dtype=np.int32)).to(dev),
                  verts=torch.from_numpy(np.ascontiguousarray(m.verts, dtype=np.float32)).to(dev),
                  ends=torch.tensor([*m.start, *m.target], dtype=torch.float32, device=dev),
                  f=torch.zeros(n, dtype=torch.float32, device=dev),
                  L=torch.zeros(n, dtype=torch.float32, device=dev),
                  Q=torch.zeros(n, dtype=torch.int32, device=dev), lib=sepso.lib())
        if not c["noalloc"]:
            nbytes = C.c_size_t()
            sepso._check(st["lib"].sepso_fitness_workspace_bytes(st["n_vert"], n, c["waypoints"], C.byref(nbytes)))
            st["ws"] = torch.empty(max(nbytes.value, 256), dtype=torch.uint8, device=dev)
            st["ws_bytes"] = nbytes.value
        return st
    if kind == "frame":
        if c["scene"] == "stress":
            m = I.stress_map(seed, S=c["side"], n_rects=c["rects"])
        else:
            moving = 2 * c["rects"] // 3
            m = I.dynamic_map(seed, S=c["side"], n_static=c["rects"] - moving, n_moving=moving,
                              side=(0.03 * c["side"], 0.11 * c["side"]))
        sw = I.dynamic_swarm(m.scale, seed=seed, groups=c["groups"], particles=c["particles"],
                             waypoints=c["waypoints"], iters=c["iters"], at_mode=c["at_mode"])
        pl = sepso.Planner(m, sw)
        pl.set_tune(c["K"], c["threads"])
        return dict(kind=kind, c=c, pl=pl)
    if kind == "batch":
        specs, sws = _dynamic_specs(c, seed)
        return dict(kind=kind, c=c, bp=sepso.BatchPlanner(specs, sws, tune=(c["K"], c["threads"])))
    if kind == "learned":
        maps = learned.dynamic_maps(c["instances"], seed)
        sws = [I.learned_swarm(seed=seed, instance=i, iters=c["iters"]) for i in range(c["instances"])]
        for sw in sws:
            sw.use_pi = 1
        lin = sepso.LearnedInit(max_rows=(c["instances"] + 31) // 32 * 32, seed=seed)
        bp = sepso.BatchPlanner(maps, sws, tune=(c["K"], c["threads"]))
        bp.attach(lin)
        return dict(kind=kind, c=c, bp=bp, lin=lin)
    if kind == "evolve":
        spec = I.dynamic_map(seed) if c["scene"] == "paper" else ablation.scene(seed)
        low = evolve.lower_swarm(None, c["particles"], c["waypoints"], c["iters"], seed)
        return dict(kind=kind, c=c, ev=sepso.Evolver(spec, low, c["h_groups"], c["h_particles"], 500, seed=seed))
    if kind == "bfevo":
        return dict(kind=kind, c=c, ev=sepso.BFEvolver(c["func"], 8, c["particles"], c["dims"], c["iters"],
                                                       h_groups=c["h_groups"], h_particles=c["h_particles"],
                                                       evolutions=500, seed=seed, h_seed=seed + 1))
    if kind == "bf":
        return dict(kind=kind, c=c, sw=sepso.BFSwarm(c["func"], 8, c["particles"], c["dims"], 1400, I.HYPER8,
                                                     seed=seed))
    lin = sepso.LearnedInit(max_rows=c["batch"], max_samples=c["samples"], seed=seed)
    learned.generate(lin, c["samples"], seed=1 + seed % 1000)
    return dict(kind=kind, c=c, lin=lin)


# ---- one pass ---------------------------------------------------------------


def _ptr(t):
    return C.c_void_p(t.data_ptr())


def run(state):
    c, kind = state["c"], state["kind"]
    if kind == "fit":
        s, n, W = state, c["paths"], c["waypoints"]
        head = (s["n_polys"], s["n_vert"], _ptr(s["pptr"]), _ptr(s["verts"]), _ptr(s["ends"]), _ptr(s["X"]), n, W,
                ALPHA, BETA, _ptr(s["f"]), _ptr(s["L"]), _ptr(s["Q"]))
        stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        if c["noalloc"]:
            sepso._check(s["lib"].sepso_fitness_noalloc(*head, stream))
        else:
            sepso._check(s["lib"].sepso_fitness(*head, _ptr(s["ws"]), s["ws_bytes"], stream))
        return dict(f=s["f"], L=s["L"], Q=s["Q"])
    if kind == "frame":
        r = state["pl"].plan_frame()
        return {k: r[k] for k in ("path", "cost", "length", "crossings", "iters", "truncated")}
    if kind in ("batch", "learned"):
        r = state["bp"].plan(1, want_paths=True)
        flat = np.concatenate(r["paths"])
        r["paths"] = np.zeros(128 * c["instances"], np.float32)  # one length whatever the waypoint counts
        r["paths"][:flat.size] = flat
        return r
    if kind in ("evolve", "bfevo"):
        ev = state["ev"]
        curve = ev.run(c.get("evolutions", 1))
        st = ev.get_state()
        return dict(curve=curve, X=st["X"], V=st["V"], P=st["P"], Pf=st["Pf"], lfv=st["lfv"],
                    gbest_n=st["gbest_n"], gbest_f=st["gbest_f"])
    if kind == "bf":
        state["sw"].step(c["steps"])
        st = state["sw"].get_state(rows=False)
        return dict(f=st["f"], Pf=st["Pf"], gbest_n=st["gbest_n"], gbest_f=st["gbest_f"], k=st["k"])
    loss = state["lin"].train(c["steps"], c["batch"], 1e-3)
    return dict(loss=loss, weights=state["lin"].get_weights())


# ---- what a pass cannot do without ------------------------------------------


def _swarm_work(elems, segs, polys, iters):
    """Planner iterations over a swarm kept in device memory: X, V and P read
    and X and V written once per element and iteration; about 10 operations
    per element for the update, 10 per segment for its length and line, and a
    box test of 4 comparisons per segment and polygon."""
    return dict(bytes=20.0 * elems * iters, flops=iters * (10.0 * elems + segs * (10.0 + 4.0 * polys)))


def work(case):
    c, kind = case, case["kind"]
    if kind == "fit":
        n, W, polys = c["paths"], c["waypoints"], c["rects"] + c["quads"] + c["stars"]
        verts = 4 * (c["rects"] + c["quads"]) + 13 * c["stars"]
        return dict(bytes=n * (8.0 * W + 12.0) + 8.0 * verts, flops=n * (W + 1.0) * (10.0 + 4.0 * polys))
    if kind == "frame":
        p = c["groups"] * c["particles"]
        polys = c["rects"] + (100 if c["scene"] == "stress" else 0)
        it = c["iters"] if c["scene"] == "stress" or c["at_mode"] == 0 else min(FRAME_ITERS, c["iters"])
        return _swarm_work(p * 2.0 * c["waypoints"], p * (c["waypoints"] + 1.0), polys, it)
    if kind == "batch":  # the generator's means: 8 x 144 particles of 20 waypoints, 52 rectangles
        p = c["instances"] * 8 * 144.0
        return _swarm_work(p * 40.0, p * 21.0, 52, FRAME_ITERS)
    if kind == "learned":
        p, w = c["instances"] * 8 * 32.0, _swarm_work(c["instances"] * 256 * 40.0, c["instances"] * 256 * 21.0, 4,
                                                      c["iters"])
        return dict(bytes=w["bytes"] + 12.0 * p * 40 + 2 * 2.8e6, flops=w["flops"] + c["instances"] * 5.57e6)
    if kind == "evolve":
        p = c["h_groups"] * c["h_particles"] * 8.0 * c["particles"]
        w = _swarm_work(p * 2 * c["waypoints"], p * (c["waypoints"] + 1), 30 if c["scene"] == "paper" else 8,
                        c["iters"] * c["evolutions"])
        return w
    if kind in ("bf", "bfevo"):
        swarms = c["h_groups"] * c["h_particles"] if kind == "bfevo" else 1
        it = c["iters"] if kind == "bfevo" else c["steps"]
        e = swarms * 8.0 * c["particles"] * c["dims"]
        # a swarm of a few kilobytes is read and written once; a large one streams every iteration
        return dict(bytes=20.0 * e * (1 if kind == "bfevo" else it), flops=20.0 * e * it)
    B, macs = float(c["batch"]), 4100 * 512 + 2 * 512 * 512 + 512 * 320
    flops = 2 * B * (3 * macs - 4100 * 512)  # forward, weight gradients, input gradients (not the first layer's)
    # inputs, activations and their gradients once; weights, gradients and both moments once
    return dict(bytes=c["steps"] * (B * (2 * 4100 + 3 * 512 * 4 + 320 * 8) + macs * 30.0), flops=c["steps"] * flops)


# ---- the same in 64 bits ----------------------------------------------------


def exact(case, seed):
    """Fitness in 64-bit torch; None for the iterated swarms and the training
    steps, whose outputs are discrete decisions fed back many times over (no
    64-bit run follows the same ones)."""
    if case["kind"] != "fit":
        return None
    m, X = _fit_inputs(case, int(seed))
    n, W, dev = case["paths"], case["waypoints"], "cuda"
    s = torch.tensor(np.asarray(m.start, np.float32), dtype=torch.float64, device=dev)
    t = torch.tensor(np.asarray(m.target, np.float32), dtype=torch.float64, device=dev)
    pts = torch.cat([s.expand(n, 1, 2), X.double().reshape(n, 2, W).transpose(1, 2), t.expand(n, 1, 2)], 1)
    a, b = pts[:, :-1], pts[:, 1:]
    L = (b - a).square().sum(-1).sqrt().sum(-1)
    v = np.asarray(m.verts, np.float32)
    nxt = np.concatenate([np.roll(np.arange(m.poly_ptr[q], m.poly_ptr[q + 1]), -1) for q in range(m.n_polys)])
    ea = torch.tensor(v, dtype=torch.float64, device=dev)
    eb = torch.tensor(v[nxt], dtype=torch.float64, device=dev)
    a, b = a.reshape(-1, 1, 2), b.reshape(-1, 1, 2)
    Q = torch.zeros(a.shape[0], dtype=torch.int64, device=dev)

    def side(p, q, r):
        return torch.sign((q[..., 0] - p[..., 0]) * (r[..., 1] - p[..., 1])
                          - (q[..., 1] - p[..., 1]) * (r[..., 0] - p[..., 0]))

    rows = max(1, int(6e7) // ea.shape[0])
    for i in range(0, a.shape[0], rows):
        p, q = a[i:i + rows], b[i:i + rows]
        hit = (side(p, q, ea) * side(p, q, eb) < 0) & (side(ea, eb, p) * side(ea, eb, q) < 0)
        Q[i:i + rows] = hit.sum(1)
    Q = Q.reshape(n, W + 1).sum(1)
    return dict(f=L + ALPHA * Q.double() ** BETA, L=L, Q=None)
