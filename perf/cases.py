"""The work that users of the framework have it do, as timed cases.

Every case is one call, or one short sequence of calls, of the public Python
API (``paper_1903_07441_amd.twg``, ``replan``) on seeded synthetic input with
the sizes of the repository's own scenarios, tests and benchmark.  A case is a
dict of plain values; ``kind`` selects what it does:

* ``map``     the map update of one replanning step (``Context.rasterize``).
* ``field``   one converged potential field (``Context.relax``), in FP32 or
              certified in FP64.
* ``sweeps``  a fixed number of sweeps (``Context.sweeps`` / ``sweeps64``).
* ``batch``   many uneven grids at once (``Context.relax_batched``).
* ``paths``   descent on a converged field: index matrix, the robot's path
              and the descent lengths of every cell.
* ``step``    one whole replanning step (``replan.Planner``).
* ``net``     the learned warm start (``UNet.warm_start`` / ``_coarse``).
* ``train``   loss and gradients of one training batch (``UNet.loss_grad``).

``listed`` names the cases, ``draw`` gives more of the same ranges,
``prepare`` makes what a program holds before the call, ``run`` is one pass,
``work`` the bytes and operations a pass cannot do without, and ``exact`` the
outputs in 64 bits by plain torch and numpy.
"""
import math
import os

import numpy as np
import torch

from paper_1903_07441_amd import replan, twg

DEV = torch.device("cuda", 0)
W_RING = 8          # ring width of every scenario
PARAM_SHAPES = [(32, 3, 3), (64, 32, 3), (128, 64, 3), (128, 128, 3), (64, 256, 3), (32, 128, 3), (32, 64, 3),
                (1, 32, 1)]  # (cout, cin, k) in the parameter vector's order


def listed():
    return [
        # the plain method's static map: the smallest call, all latency
        dict(name="map 64", kind="map", nx=64, ny=64, pad=0, n_obs=10, rmin=2.0, rmax=5.0, sigma=0.0, ellipse=False),
        # the map update of the replanning loop at full size
        dict(name="map 2048", kind="map", nx=2048, ny=2048, pad=0, n_obs=500, rmin=3.0, rmax=12.0, sigma=0.5,
             ellipse=False),
        # one small static grid solved in FP64 accuracy, as a first program does it
        dict(name="field 64 certified", kind="field", nx=64, ny=64, pad=0, n_obs=10, rmin=2.0, rmax=5.0, tol=1e-9,
             polish=1, cert=0.0, init="half"),
        # one time-warped grid of ordinary size, polished to the oracle's accuracy, library defaults
        dict(name="field 512 certified", kind="field", nx=512, ny=512, pad=0, n_obs=50, rmin=3.0, rmax=8.0, tol=1e-6,
             polish=1, cert=1e-8, init="zero"),
        # a map of no round size (odd sides and pitch), FP32 only, from the paper's initial 0.5
        dict(name="field 1001x743 ragged", kind="field", nx=1001, ny=743, pad=4, n_obs=150, rmin=3.0, rmax=10.0,
             tol=1e-6, polish=0, cert=0.0, init="half"),
        # the benchmark: one whole replanning step at full size, with the tiling the autotuner keeps there
        dict(name="step 2048", kind="step", side=2048, n_obs=500, rmin=3.0, rmax=12.0, S=6, RH=46),
        # the uneven batch (scenario sets, replanning what-ifs, training targets)
        dict(name="batch 64 grids", kind="batch", n=64, sides="64,128,256,512,1024", rmin=2.0, rmax=5.0, S=8, RH=128),
        # one extra FP64 round of a step whose descent does not resolve yet
        dict(name="sweeps64 2048", kind="sweeps", nx=2048, ny=2048, pad=0, bits=64, count=256, n_obs=500, rmin=3.0,
             rmax=12.0),
        # path extraction and the reachability report on a converged field
        dict(name="paths 1024", kind="paths", nx=1024, ny=1024, pad=0, n_obs=200, rmin=3.0, rmax=10.0),
        # the loop's learned warm start: the network at 1/8 of a full-size map
        dict(name="net coarse 2048", kind="net", nx=2048, ny=2048, factor=8, n_obs=500, rmin=3.0, rmax=12.0),
        # the network at full resolution
        dict(name="net 2048", kind="net", nx=2048, ny=2048, factor=0, n_obs=500, rmin=3.0, rmax=12.0),
        # one training batch of the shipped weights' recipe
        dict(name="train 16x256", kind="train", batch=16, H=256, W=256, n_obs=80, rmin=2.0, rmax=5.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _obs(rng, cells):
    """Obstacles for a grid of `cells` cells at the scenarios' densities."""
    return max(5, min(500, int(cells ** 0.5 * rng.uniform(0.1, 0.3))))


def draw(rng):
    kind = rng.choice(["map", "field", "field", "sweeps", "batch", "paths", "step", "net", "train"])
    if kind in ("map", "field", "sweeps", "paths"):
        nx = _log(rng, *dict(map=(48, 2048), field=(40, 1400), sweeps=(64, 2048), paths=(100, 1400))[kind])
        ny = max(40, int(nx * rng.uniform(0.6, 1.0)))
        c = dict(kind=kind, nx=nx, ny=ny, pad=rng.choice([0, 0, 0, 1, 3, 8]), n_obs=_obs(rng, nx * ny), rmin=3.0,
                 rmax=rng.choice([5.0, 8.0, 12.0]) if nx >= 128 else 5.0)
        if kind == "map":
            c.update(sigma=rng.choice([0.0, 0.5]), ellipse=rng.random() < 0.25)
        elif kind == "field":
            polish = rng.choice([0, 1, 1])
            c.update(tol=1e-6 if max(nx, ny) > 100 else 1e-9, polish=polish, cert=1e-8 if polish else 0.0,
                     init=rng.choice(["half", "zero"]))
        elif kind == "sweeps":
            c.update(bits=rng.choice([32, 64]), count=rng.choice([100, 256]))
        return c
    if kind == "batch":
        return dict(kind="batch", n=_log(rng, 8, 60), sides=rng.choice(["64,128,256,512,1024", "64,96,128,160", "256",
                                                                       "101,333,640"]),
                    rmin=2.0, rmax=5.0, S=rng.choice([4, 6, 8]), RH=rng.choice([32, 64, 128]))
    if kind == "step":
        side = _log(rng, 256, 2048)
        return dict(kind="step", side=side, n_obs=_obs(rng, side * side), rmin=3.0, rmax=12.0, S=0, RH=0)
    if kind == "net":
        factor = rng.choice([0, 8])
        nx, ny = (64 * rng.randint(3, 32) for _ in range(2))
        return dict(kind="net", nx=nx, ny=ny, factor=factor, n_obs=_obs(rng, nx * ny), rmin=3.0, rmax=12.0)
    return dict(kind="train", batch=rng.randint(1, 16), H=8 * rng.randint(8, 32), W=8 * rng.randint(8, 32), n_obs=40,
                rmin=2.0, rmax=5.0)


# ---- inputs -----------------------------------------------------------------

def _world(nx, ny, n_obs, rmin, rmax, seed, sigma=0.5):
    """Robot, goal and moving discs of one scenario (none covers the robot
    or the goal at the start)."""
    rng = np.random.default_rng(seed)
    robot = np.array([rng.integers(1, nx - 1), rng.integers(1, ny - 1)], dtype=np.int32)
    goal = robot
    while (goal == robot).all():
        goal = np.array([rng.integers(1, nx - 1), rng.integers(1, ny - 1)], dtype=np.int32)
    pos, rad = np.empty((n_obs, 2)), rng.uniform(rmin, rmax, n_obs)
    for i in range(n_obs):
        while True:
            pos[i] = rng.uniform(0, nx), rng.uniform(0, ny)
            if min(np.hypot(*(pos[i] - robot)), np.hypot(*(pos[i] - goal))) > rad[i] + 1.5:
                break
    vel = rng.normal(0.0, sigma, (n_obs, 2)) if sigma > 0 else np.zeros((n_obs, 2))
    return dict(nx=nx, ny=ny, robot=robot, goal=goal, W=W_RING, vr=1.0, pos=pos, vel=vel, rad=rad)


def _class_map(w):
    """Class map of a world with its discs where they are now (numpy uint8)."""
    nx, ny = w["nx"], w["ny"]
    cls = np.zeros((ny, nx), dtype=np.uint8)
    for (px, py), r in zip(w["pos"], w["rad"]):
        x0, x1 = max(0, int(px - r)), min(nx, int(px + r) + 2)
        y0, y1 = max(0, int(py - r)), min(ny, int(py + r) + 2)
        ys, xs = np.ogrid[y0:y1, x0:x1]
        cls[y0:y1, x0:x1][(xs - px) ** 2 + (ys - py) ** 2 <= r * r] = twg.OBST
    cls[0, :] = cls[-1, :] = twg.WALL
    cls[:, 0] = cls[:, -1] = twg.WALL
    cls[w["goal"][1], w["goal"][0]] = twg.GOAL
    return cls


def _ring_map(w):
    """Time rings of a world (concentric circles around the robot), int64."""
    ys, xs = np.ogrid[0:w["ny"], 0:w["nx"]]
    d2 = (xs - int(w["robot"][0])) ** 2 + (ys - int(w["robot"][1])) ** 2
    return np.sqrt(d2.astype(np.float64)).astype(np.int64) // W_RING


def _padded(ny, nx, pad, dtype):
    """A zeroed [ny, nx] device grid with a row stride of nx + pad."""
    return torch.zeros((ny, nx + pad), dtype=dtype, device=DEV)[:, :nx]


def _dev(a, dtype=None):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).to(DEV)


def _family(n, c=3.6):
    """SOR factor of the autotuner's family for a grid of side n."""
    return 2.0 / (1.0 + c * math.sin(math.pi / (n + 1)))


def _case_world(case, seed):
    side = case.get("side")
    return _world(case.get("nx", side), case.get("ny", side), case["n_obs"], case["rmin"], case["rmax"], seed,
                  case.get("sigma", 0.5))


def _batch_sides(case):
    sides = [int(s) for s in case["sides"].split(",")]
    return [sides[k % len(sides)] for k in range(case["n"])]


def _batch_maps(case, seed):
    return [_class_map(_world(s, s, 10 + (37 * k) % 191 if s > 128 else 10 + (7 * k) % 20, case["rmin"], case["rmax"],
                              [seed, k])) for k, s in enumerate(_batch_sides(case))]


def _params(seed):
    """He-uniform convolutions, zero biases, head scaled by 0.1: a network
    as training starts it."""
    rng = np.random.default_rng(seed)
    parts = []
    for cout, cin, k in PARAM_SHAPES:
        lim = math.sqrt(6.0 / (cin * k * k)) * (0.1 if k == 1 else 1.0)
        parts += [rng.uniform(-lim, lim, cout * cin * k * k), np.zeros(cout)]
    return np.concatenate(parts).astype(np.float32)


def _shipped(factor):
    name = "unet_coarse8_replan2048.npz" if factor else "unet_learn256.npz"
    path = os.path.join(os.path.dirname(os.path.abspath(twg.__file__)), "weights", name)
    with np.load(path, allow_pickle=False) as z:
        return z["params"].astype(np.float32)


def _train_images(case, seed):
    """Network inputs [B, H, W, 3], targets and class maps of a training batch:
    maps as the field cases have them, targets that fall off from the goal
    and around the obstacles as converged fields do."""
    B, H, W = case["batch"], case["H"], case["W"]
    x, t, c = np.empty((B, H, W, 3), np.float32), np.empty((B, H, W), np.float32), np.empty((B, H, W), np.uint8)
    ys, xs = np.ogrid[0:H, 0:W]
    for b in range(B):
        w = _world(W, H, min(case["n_obs"], W * H // 600), case["rmin"], case["rmax"], [seed, b])
        cls, ring = _class_map(w), _ring_map(w)
        d = np.hypot(xs - w["goal"][0], ys - w["goal"][1])
        x[b, ..., 0] = (cls == twg.OBST) | (cls == twg.WALL)
        x[b, ..., 1] = d / (max(H, W) * math.sqrt(2.0))
        x[b, ..., 2] = ring / max(1, ring.max())
        t[b] = np.where(cls == twg.FREE, np.exp(-d / (0.2 * max(H, W))), cls == twg.GOAL)
        c[b] = cls
    return x, t, c


# ---- prepare and run ----------------------------------------------------------

def prepare(case, seed):
    s = dict(case=case)
    kind = case["kind"]
    ctx = s["ctx"] = twg.Context(0)
    if kind == "train":
        x, t, c = _train_images(case, seed)
        s["net"] = twg.UNet(ctx, _params(seed))
        s.update(x=_dev(x), target=_dev(t), cls=_dev(c), loss=torch.zeros(1, device=DEV),
                 grads=torch.zeros(s["net"].n_params, device=DEV))
        return s
    if kind == "batch":
        maps = _batch_maps(case, seed)
        descs, off = [], 0
        for m in maps:
            n = m.shape[0]
            descs.append((n, n, n, off))
            off += (n * n + 63) // 64 * 64
            ctx.set_tiling(n, n, case["S"], case["RH"], _family(n, 2.8))
        flat = np.full(off, twg.WALL, dtype=np.uint8)
        for m, d in zip(maps, descs):
            flat[d[3]:d[3] + m.size] = m.reshape(-1)
        s.update(descs=descs, cls=_dev(flat), psi=torch.zeros(off, device=DEV))
        return s
    w = _case_world(case, seed)
    nx, ny, pad = w["nx"], w["ny"], case.get("pad", 0)
    s["world"] = w
    if kind == "map":
        s.update(pos=_dev(w["pos"]), vel=_dev(w["vel"]), rad=_dev(w["rad"]), cls=_padded(ny, nx, pad, torch.uint8),
                 ring=_padded(ny, nx, pad, torch.int16).view(torch.uint16))
        return s
    if kind == "step":
        if case["S"]:
            ctx.set_tiling(nx, ny, case["S"], case["RH"], _family(nx), case["S"], case["RH"])
        s.update(pl=replan.Planner(ctx, w), pos=_dev(w["pos"]), vel=_dev(w["vel"]))
        s["pl"].path.zero_()  # the cells past the path's end are never written
        return s
    cls = _class_map(w)
    s["cls"] = _padded(ny, nx, pad, torch.uint8)
    s["cls"].copy_(_dev(cls))
    if kind == "field":
        s.update(psi=_padded(ny, nx, pad, torch.float32),
                 psi64=_padded(ny, nx, pad, torch.float64) if case["polish"] else None)
    elif kind == "sweeps":
        s["psi0"] = _padded(ny, nx, pad, torch.float64 if case["bits"] == 64 else torch.float32)
        s["psi0"].copy_(_start_field(case, cls, w, _dev))
        s["psi"] = _padded(ny, nx, pad, s["psi0"].dtype)
    elif kind == "paths":
        s["psi64"] = _padded(ny, nx, pad, torch.float64)
        s["psi64"].copy_(_harmonic(_dev(cls)[None])[0])
        s.update(idx=_padded(ny, nx, pad, torch.uint8), steps=torch.zeros((ny, nx), dtype=torch.int32, device=DEV),
                 path=torch.zeros((nx * ny, 2), dtype=torch.int32, device=DEV),
                 info=torch.zeros(2, dtype=torch.int32, device=DEV))
    elif kind == "net":
        s.update(net=twg.UNet(ctx, _shipped(case["factor"])), psi=torch.zeros((ny, nx), device=DEV),
                 ring=_dev(_ring_map(w).astype(np.int16)).view(torch.uint16),
                 status=torch.zeros(1, dtype=torch.int32, device=DEV))
    return s


def _start_field(case, cls, w, put):
    """The field the fixed sweeps start from: the paper's 0.5 (FP32), or a
    field that falls off from the goal (FP64 rounds refine a solved one)."""
    nx, ny = w["nx"], w["ny"]
    if case["bits"] == 32:
        u = np.full((ny, nx), 0.5)
    else:
        ys, xs = np.ogrid[0:ny, 0:nx]
        u = np.exp(-np.hypot(xs - w["goal"][0], ys - w["goal"][1]) / 40.0)
    u = np.where(cls == twg.FREE, u, (cls == twg.GOAL) * 1.0)
    return put(u)


def _sweep_omega(case):
    return 1.0 if case["bits"] == 32 else _family(max(case["nx"], case["ny"]))


def run(s):
    case, ctx = s["case"], s.get("ctx")
    kind = case["kind"]
    if kind == "map":
        w = s["world"]
        ctx.rasterize(w["nx"], w["ny"], w["robot"], w["goal"], s["pos"], s["vel"], s["rad"], W=w["W"],
                      robot_speed=w["vr"], cls=s["cls"], ring=s["ring"], ring_mode=int(case["ellipse"]),
                      heading=(0.6, 0.8))
        return {"cls": s["cls"], "ring": s["ring"].view(torch.int16)}
    if kind == "field":
        st = ctx.relax(s["cls"], s["psi"], s["psi64"], tol=case["tol"], tol_cert=case["cert"], polish=case["polish"],
                       init=twg.INIT_ZERO if case["init"] == "zero" else twg.INIT_HALF)
        out = {"psi": s["psi"], "status": st["status"]}
        if case["polish"]:
            out["psi64"] = s["psi64"]
        return out
    if kind == "sweeps":
        s["psi"].copy_(s["psi0"])
        if case["bits"] == 64:
            ctx.sweeps64(s["cls"], s["psi"], _sweep_omega(case), case["count"])
        else:
            ctx.sweeps(s["cls"], s["psi"], _sweep_omega(case), case["count"])
        return {"psi": s["psi"]}
    if kind == "batch":
        st = ctx.relax_batched(s["cls"], s["psi"], s["descs"], tol=1e-6, init=twg.INIT_HALF,
                               sweeps_per_pass=case["S"], rows_per_tile=case["RH"])
        return {"psi": s["psi"], "status": [x["status"] for x in st][:1]}
    if kind == "paths":
        w = s["world"]
        ctx.index_matrix(s["cls"], psi64=s["psi64"], idx=s["idx"])
        ctx.descend(s["cls"], psi64=s["psi64"], start=w["robot"], cap=w["nx"] * w["ny"], path=s["path"],
                    info=s["info"])
        ctx.descent_all(s["cls"], psi64=s["psi64"], steps=s["steps"])
        return {"idx": s["idx"], "path": s["path"], "info": s["info"], "steps": s["steps"]}
    if kind == "step":
        pl, w = s["pl"], s["world"]
        pl.rasterize(w["robot"], s["pos"], s["vel"])
        pl.solve(w["robot"])
        return {"cls": pl.cls, "psi": pl.psi, "psi64": pl.psi64, "path": pl.path, "info": pl.info}
    if kind == "net":
        w = s["world"]
        if case["factor"]:
            s["net"].warm_start_coarse(s["cls"], s["ring"], w["goal"], s["psi"], case["factor"], s["status"])
        else:
            s["net"].warm_start(s["cls"], s["ring"], w["goal"], s["psi"], s["status"])
        return {"psi": s["psi"], "status": s["status"]}
    s["net"].loss_grad(s["x"], s["target"], s["cls"], s["loss"], s["grads"])
    return {"loss": s["loss"], "grads": s["grads"]}


# ---- what a pass cannot do without ---------------------------------------------

def _net_flops(pixels):
    """Products and sums of the network's forward pass."""
    at = [1, 4, 16, 64, 16, 4, 1, 1]
    return sum(2 * co * ci * k * k * pixels / a for (co, ci, k), a in zip(PARAM_SHAPES, at))


def work(case):
    """Inputs read once and outputs written once; a sweep is 7 operations a
    cell (three sums, two fused products).  A converged solve is counted as
    one residual evaluation: how many sweeps it takes is the method's."""
    kind = case["kind"]
    if kind == "batch":
        cells = sum(n * n for n in _batch_sides(case))
        return {"bytes": 5.0 * cells, "flops": 7.0 * cells}
    if kind == "train":
        p = case["batch"] * case["H"] * case["W"]
        return {"bytes": 17.0 * p + 8.0 * 443745, "flops": 3.0 * _net_flops(p)}
    nx, ny = case.get("nx", case.get("side")), case.get("ny", case.get("side"))
    cells = nx * ny
    if kind == "map":
        return {"bytes": 3.0 * cells + 40.0 * case["n_obs"], "flops": 4.0 * cells}
    if kind == "field":
        return {"bytes": (13.0 if case["polish"] else 5.0) * cells, "flops": 7.0 * cells}
    if kind == "sweeps":
        return {"bytes": (2.0 * case["bits"] / 8 + 1) * cells, "flops": 7.0 * case["count"] * cells}
    if kind == "paths":
        return {"bytes": 14.0 * cells, "flops": 4.0 * cells}
    if kind == "step":
        return {"bytes": 15.0 * cells, "flops": 11.0 * cells}
    f = case["factor"]
    return {"bytes": 7.0 * cells + 2.0 * 443745, "flops": _net_flops(cells / f ** 2 if f else cells)}


# ---- the outputs in 64 bits ----------------------------------------------------

def _masks(cls):
    """FREE masks of the two colours, [k, ny, nx] FP64."""
    ny, nx = cls.shape[-2:]
    par = (torch.arange(ny, device=DEV)[:, None] + torch.arange(nx, device=DEV)[None]) % 2
    free = cls == twg.FREE
    return [(free & (par == c)).double() for c in (0, 1)]


def _sweep(u, masks, omega):
    """One red-black sweep of u [k, ny + 2, nx + 2] (a zero frame around)."""
    inner = u[:, 1:-1, 1:-1]
    for m in masks:
        d = (u[:, 1:-1, 2:] + u[:, 1:-1, :-2]).add_(u[:, 2:, 1:-1]).add_(u[:, :-2, 1:-1]).mul_(0.25).sub_(inner)
        inner.addcmul_(m, d, value=omega)
    return u


def _framed(u):
    return torch.nn.functional.pad(u, (1, 1, 1, 1))


def _harmonic(cls):
    """Converged potential of class maps [k, ny, nx] (device), FP64."""
    masks = _masks(cls)
    u = _framed((cls == twg.GOAL).double())
    omega, last = _family(max(cls.shape[-2:]), 3.0), math.inf
    for k in range(200):
        for _ in range(100):
            _sweep(u, masks, omega)
        i = u[:, 1:-1, 1:-1]
        r = ((u[:, 1:-1, 2:] + u[:, 1:-1, :-2] + u[:, 2:, 1:-1] + u[:, :-2, 1:-1]) * 0.25 - i) * (masks[0] + masks[1])
        r = float(r.abs().max())
        if r < 1e-15 or (r < 1e-14 and r > 0.5 * last):
            break
        last = r
    return u[:, 1:-1, 1:-1].contiguous()


def _predicted_map(w):
    """Class map of a replanning step: every cell sees the discs where they
    are predicted for the time the robot needs to the cell's ring."""
    nx, ny = w["nx"], w["ny"]
    ring = _ring_map(w)
    occ = np.zeros((ny, nx), dtype=bool)
    t = np.arange(ring.max() + 1) * float(W_RING) / w["vr"]
    R = np.rint(256.0 * w["rad"]).astype(np.int64)
    for i in range(len(R)):
        c = w["pos"][i] + t[:, None] * w["vel"][i]
        far = np.hypot(c[:, 0] - w["robot"][0], c[:, 1] - w["robot"][1])
        for j in np.nonzero(np.abs(far - (np.arange(len(t)) + 0.5) * W_RING) <= w["rad"][i] + W_RING)[0]:
            x0, x1 = max(0, int(c[j, 0] - w["rad"][i]) - 1), min(nx, int(c[j, 0] + w["rad"][i]) + 2)
            y0, y1 = max(0, int(c[j, 1] - w["rad"][i]) - 1), min(ny, int(c[j, 1] + w["rad"][i]) + 2)
            if x0 >= x1 or y0 >= y1:
                continue
            C = np.rint(256.0 * c[j]).astype(np.int64)
            ys, xs = np.ogrid[y0:y1, x0:x1]
            disc = (256 * xs - C[0]) ** 2 + (256 * ys - C[1]) ** 2 <= R[i] * R[i]
            occ[y0:y1, x0:x1] |= disc & (ring[y0:y1, x0:x1] == j)
    cls = np.where(occ, twg.OBST, twg.FREE).astype(np.uint8)
    cls[w["goal"][1], w["goal"][0]] = twg.GOAL
    cls[0, :] = cls[-1, :] = twg.WALL
    cls[:, 0] = cls[:, -1] = twg.WALL
    return cls


def _conv(x, w, b, relu=True):
    """NHWC 3x3 cross-correlation with zero padding, as nine products."""
    B, H, W, C = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b
    for ky in range(3):
        for kx in range(3):
            y = y + (p[:, ky:ky + H, kx:kx + W].reshape(-1, C) @ w[:, :, ky, kx].t()).reshape(B, H, W, -1)
    return torch.relu(y) if relu else y


def _pool(x):
    return 0.25 * (x[:, ::2, ::2] + x[:, 1::2, ::2] + x[:, ::2, 1::2] + x[:, 1::2, 1::2])


def _up(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2)


def _bf16(x):
    return x.to(torch.bfloat16).to(x.dtype)


def _net(params, x, rnd=lambda v: v):
    """The network in FP64: params the flat vector, x [B, H, W, 3]; rnd rounds
    what the network stores (its input, activations and 3x3 weights)."""
    ws, o = [], 0
    for cout, cin, k in PARAM_SHAPES:
        n = cout * cin * k * k
        w = params[o:o + n].reshape(cout, cin, k, k)
        ws.append((rnd(w) if k == 3 else w, params[o + n:o + n + cout]))
        o += n + cout
    e0 = rnd(_conv(rnd(x), *ws[0]))
    e1 = rnd(_conv(rnd(_pool(e0)), *ws[1]))
    e2 = rnd(_conv(rnd(_pool(e1)), *ws[2]))
    e3 = rnd(_conv(rnd(_pool(e2)), *ws[3]))
    d2 = rnd(_conv(torch.cat([_up(e3), e2], -1), *ws[4]))
    d1 = rnd(_conv(torch.cat([_up(d2), e1], -1), *ws[5]))
    d0 = rnd(_conv(torch.cat([_up(d1), e0], -1), *ws[6]))
    B, H, W, C = d0.shape
    return (d0.reshape(-1, C) @ ws[7][0].reshape(1, C).t()).reshape(B, H, W) + ws[7][1]


def _exact_net(case, seed):
    w = _case_world(case, seed)
    nx, ny, f = w["nx"], w["ny"], case["factor"]
    cls, ring = _dev(_class_map(w)), _dev(_ring_map(w)).double()
    n, far = max(1, f), max(nx, ny) * math.sqrt(2.0)
    if ny % (8 * n) or nx % (8 * n):
        return None
    occ = ((cls == twg.OBST) | (cls == twg.WALL)).double().reshape(ny // n, n, nx // n, n).mean((1, 3))
    ys = torch.arange(ny // n, device=DEV).double() * n + (n - 1) / 2
    xs = torch.arange(nx // n, device=DEV).double() * n + (n - 1) / 2
    dist = torch.hypot(ys[:, None] - float(w["goal"][1]), xs[None] - float(w["goal"][0])) / far
    x = torch.stack([occ, dist, (ring / ring.max())[n // 2::n, n // 2::n]], -1)[None]
    y = _net(_dev(_shipped(f)).double(), x, _bf16)[0]  # the network is defined with bf16 storage
    if f:  # bilinear interpolation back to the grid, clamped to the frame
        def weights(size, frame):
            t = ((torch.arange(size, device=DEV).double() + 0.5) / f - 0.5).clamp(0, frame - 1)
            i = t.floor().clamp(max=frame - 1)
            return i.long(), (i.long() + 1).clamp(max=frame - 1), t - i
        y0, y1, ty = weights(ny, y.shape[0])
        x0, x1, tx = weights(nx, y.shape[1])
        y = y[y0] * (1 - ty)[:, None] + y[y1] * ty[:, None]
        y = y[:, x0] * (1 - tx)[None] + y[:, x1] * tx[None]
    psi = torch.where(cls == twg.FREE, y.clamp(0, 1), (cls == twg.GOAL).double())
    return {"psi": psi, "status": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "field":
        u = _harmonic(_dev(_class_map(_case_world(case, seed)))[None])[0]
        return {"psi": u, "status": None, "psi64": u} if case["polish"] else {"psi": u, "status": None}
    if kind == "sweeps":
        w = _case_world(case, seed)
        cls = _class_map(w)
        u, masks = _framed(_start_field(case, cls, w, _dev)[None]), _masks(_dev(cls)[None])
        for _ in range(case["count"]):
            _sweep(u, masks, _sweep_omega(case))
        return {"psi": u[0, 1:-1, 1:-1].contiguous()}
    if kind == "batch":
        sides, maps, off, at = _batch_sides(case), _batch_maps(case, seed), 0, []
        for n in sides:
            at.append(off)
            off += (n * n + 63) // 64 * 64
        psi = torch.zeros(off, dtype=torch.float64, device=DEV)
        for n in sorted(set(sides)):
            of_size = [k for k in range(len(sides)) if sides[k] == n]
            u = _harmonic(torch.stack([_dev(maps[k]) for k in of_size]))
            for j, k in enumerate(of_size):
                psi[at[k]:at[k] + n * n] = u[j].reshape(-1)
        return {"psi": psi, "status": None}
    if kind == "step":
        cls = _predicted_map(_case_world(case, seed))
        u = _harmonic(_dev(cls)[None])[0]
        return {"cls": None, "psi": u, "psi64": u, "path": None, "info": None}
    if kind == "net":
        return _exact_net(case, seed)
    if kind == "train":
        x, t, c = (_dev(a) for a in _train_images(case, seed))
        p = _dev(_params(seed)).double().requires_grad_()
        y = _net(p, x.double())
        free = (c == twg.FREE).double()
        loss = ((((y - t.double()) ** 2) * free).sum((1, 2)) / free.sum((1, 2)).clamp(min=1)).mean()
        loss.backward()
        return {"loss": loss.detach().reshape(1), "grads": p.grad}
    return None
