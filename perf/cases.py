"""Performance cases: the work a program has the framework do, through its
public entry points (World, Server), from single calls to whole episodes.

listed() holds the cases, draw() makes more of the same ranges, prepare()
builds the world a program keeps, run() is one pass, work() the bytes and
operations the pass cannot do without, and exact() the pass's outputs from
plain torch and numpy in 64 bits where they have such a value.

Kinds:
  step     set the state, advance it, read it back (planning, replay)
  observe  set the state (an episode reset), render it, read the frames
  gym      the observation loop: step, render, read everything, per step
  episode  a reset and an episode of one schedule, then frames and state
  act      the policy on the current frames
  rollout  a reset and an episode of render, act, step
  serve    rollout requests served by continuous batching

Scenes are piles on the ground, as they stand some seconds after the
synthetic drops of scenegen; the draws are seeded.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

BASE = dict(envs=64, bodies=32, bodies_max=0, poisson=0, w=128, h=128, cams=1, ring=False, iters=1, tuned=False,
            schedule="serial", split=0.0, friction=0.0, boxes=False, edge=False, smooth=False, texture=False,
            near_clip=False, metric=False, hidden=0, requests=0)


def _case(name, kind, **kw):
    c = dict(BASE, kind=kind, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a handful of envs stepped one by one with every observation read:
        # interactive use and evaluation, bound by latency and launches
        _case("gym 16 envs, 8 spheres, 64x64", "gym", envs=16, bodies=8, w=64, h=64, iters=10),
        # physics alone over a batch: planning by sampled rollouts, 8 steps
        # a decision (30 Hz control of a 240 Hz simulation)
        _case("step 1024 envs, 32 bodies", "step", envs=1024, bodies=32, cams=0, iters=8),
        # task physics with uneven env sizes: boxes, friction, edge contacts
        _case("step 1500 envs, 4-128 mixed, friction", "step", envs=1500, bodies=4, bodies_max=128, cams=0, iters=4,
              friction=0.5, boxes=True, edge=True),
        # episode reset of a training batch and its first observation
        _case("observe 1024 envs, 128x128", "observe", envs=1024),
        # the 640x480 data-generation camera, textured, with metric depth
        _case("observe 48 envs, 640x480 textured", "observe", envs=48, w=640, h=480, smooth=True, texture=True,
              metric=True),
        # the training batch of the benchmark, co-scheduled
        _case("episode 1024 envs, 32 bodies, 128x128", "episode", envs=1024, iters=100, schedule="pipelined",
              split=2.0, tuned=True),
        # the largest data-generation batch: two 256x256 ring cameras per env
        _case("episode 4096 envs, 64 bodies, 2x256x256", "episode", envs=4096, bodies=64, w=256, h=256, cams=2,
              ring=True, iters=10, schedule="pipelined", split=2.0, tuned=True),
        # uneven batch: Poisson body counts, 64/128/256 frames (w = 0), defaults
        _case("episode 2048 envs, mixed sizes", "episode", envs=2048, bodies=4, bodies_max=128, poisson=24, w=0, h=0,
              iters=50, schedule="interstep", split=2.0),
        # the MLP policies of the RL rollouts on a training batch
        _case("act 1024 envs, hidden 256", "act", envs=1024, hidden=256),
        _case("act 1024 envs, hidden 4096", "act", envs=1024, hidden=4096),
        # a small RL job: render, act, step on one stream
        _case("rollout 250 envs, 64x64, hidden 256", "rollout", envs=250, bodies=17, w=64, h=64, iters=32,
              hidden=256),
        # rollout requests of all shapes with their final states and frames
        _case("serve 8 requests", "serve", envs=16, requests=8, schedule="pipelined", split=2.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "observe", "observe", "gym", "episode", "episode", "act", "rollout", "serve"])
    c = dict(envs=_log(rng, 16, 2048), bodies=_log(rng, 1, 64))
    if kind == "serve":
        return _case("", kind, envs=_log(rng, 8, 32), requests=rng.randint(3, 10), schedule="pipelined", split=2.0)
    if kind in ("act", "rollout"):
        c["w"], c["h"] = 8 * rng.randint(4, 16), 8 * rng.randint(4, 16)
        c["hidden"] = 64 * _log(rng, 1, 64) if rng.random() < 0.5 else _log(rng, 33, 1024)
        c["envs"] = _log(rng, 16, 1200)
        c["iters"] = rng.randint(8, 32) if kind == "rollout" else 1
        if c["w"] * c["h"] * c["hidden"] > 1 << 25:
            c["hidden"] = 256
        return _case("", kind, **c)
    if rng.random() < 0.4:
        c["bodies_max"] = rng.randint(c["bodies"], 128)
    c["friction"] = rng.choice([0.0, 0.0, 0.3, 0.8])
    c["boxes"] = rng.random() < 0.3
    c["edge"] = c["boxes"] and rng.random() < 0.5
    if kind == "step":
        return _case("", kind, cams=0, iters=rng.randint(1, 16), **c)
    look = rng.choice(["flat", "flat", "near_clip", "smooth", "texture"])
    c["near_clip"], c["smooth"], c["texture"] = look == "near_clip", look in ("smooth", "texture"), look == "texture"
    if rng.random() < 0.7:
        c["w"] = c["h"] = rng.choice([64, 100, 128, 200, 256])
        c["cams"], c["ring"] = rng.choice([1, 1, 2]), rng.random() < 0.5
    else:
        c["w"], c["h"] = rng.randint(60, 640), rng.randint(60, 480)
    most = 1 << (24 if kind == "gym" else 26)  # pixels of the batch
    c["envs"] = max(1, min(c["envs"], most // (c["w"] * c["h"] * c.get("cams", 1)), (1 << 18) // max(c["bodies"], 1)))
    if kind == "observe":
        c["metric"] = rng.random() < 0.4
    elif kind == "gym":
        c["iters"] = rng.randint(2, 12)
    else:
        c["iters"] = rng.randint(20, 80)
        c["schedule"] = rng.choice(["serial", "interstep", "intertraj", "pipelined"])
        c["split"] = rng.choice([0.0, 2.0]) if c["schedule"] == "serial" else 2.0
        c["tuned"] = rng.random() < 0.5
    return _case("", kind, **c)


# ---------------------------------------------------------------------------
# scenes
# ---------------------------------------------------------------------------

SHAPES = 2605  # seed of the sizes of uneven batches: a case's shapes are its own, its content the seed's


def _rotation(q, t=np.float64):
    """Rotation matrices [B, 3, 3] of unit quaternions, in type t."""
    w, x, y, z = (q[:, k].astype(t) for k in range(4))
    one, two = t(1), t(2)
    xx, yy, zz, xy, xz, yz, wx, wy, wz = x * x, y * y, z * z, x * y, x * z, y * z, w * x, w * y, w * z
    r = [one - two * (yy + zz), two * (xy - wz), two * (xz + wy), two * (xy + wz), one - two * (xx + zz),
         two * (yz - wx), two * (xz - wy), two * (yz + wx), one - two * (xx + yy)]
    return np.stack(r, 1).reshape(-1, 3, 3)


def _piled(scene, rng):
    """The scene's bodies lying on the ground and on one another: dropped one
    by one straight down onto what lies there, with the small penetrations
    and the motion of a pile half a second to a second after a drop (contact
    counts and speeds between those of the benchmark's 64-body scene after
    100 steps and its 32-body scene after 250)."""
    E, B, n = scene.n_envs, scene.n_bodies, scene.counts()
    q = rng.normal(size=(B, 4))
    q = (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(np.float32)
    size = scene.size.astype(np.float64)
    ext = np.repeat(size[:, None], 3, 1) if scene.ext is None else scene.ext.astype(np.float64)
    round_ = scene.btype == sg.SPHERE
    low = np.where(round_, size, (np.abs(_rotation(q)[:, 2]) * ext).sum(1)) - rng.uniform(1e-4, 2e-3, B)
    reach = np.where(round_, size, 1.3 * size)
    half = np.repeat(0.5 * np.sqrt(np.maximum(n, 4) / 7.0), n)
    pos = np.stack([rng.uniform(-1, 1, B) * half, rng.uniform(-1, 1, B) * half, low], 1)
    off = scene.body_off[:-1].astype(np.int64)
    for k in range(1, int(n.max()) if E else 0):
        e = np.nonzero(n > k)[0]
        b, under = off[e] + k, off[e][:, None] + np.arange(k)
        d2 = ((pos[under, :2] - pos[b, None, :2]) ** 2).sum(2)
        s = reach[under] + reach[b, None] - 1e-3
        top = np.where(d2 < s * s, pos[under, 2] + np.sqrt(np.maximum(s * s - d2, 0.0)), 0.0)
        pos[b, 2] = np.maximum(pos[b, 2], top.max(1))
    return dataclasses.replace(scene, pos=pos.astype(np.float32), quat=q,
                               vel=(rng.normal(size=(B, 3)) * [0.6, 0.6, 0.3]).astype(np.float32),
                               omega=(4.0 * rng.normal(size=(B, 3))).astype(np.float32))


def _scene(case, seed):
    rng = np.random.default_rng(seed)
    shape = np.random.default_rng(SHAPES)
    E, lo, hi = case["envs"], case["bodies"], case["bodies_max"]
    if case["poisson"]:
        counts = np.clip(shape.poisson(case["poisson"], E), lo, hi)
    else:
        counts = shape.integers(lo, hi + 1, E) if hi else np.full(E, lo)
    res = shape.choice([64, 128, 256], E) if case["w"] == 0 else case["w"]
    s = sg.make_scene(int(rng.integers(1 << 20)), counts, res, mixed=lo > 8 or hi > 8, cams_per_env=case["cams"],
                      ring=case["ring"])
    if case["w"] != case["h"] and s.n_cams:
        vp = sg.view_proj(sg.FIXED_EYE, aspect=case["w"] / case["h"]).reshape(16)
        s = dataclasses.replace(s, cam_vp=np.tile(vp, (s.n_cams, 1)), cam_h=np.full(s.n_cams, case["h"], np.int32))
    if case["boxes"]:
        s = sg.with_boxes(s)
    if case["texture"]:
        s = sg.with_texture(s)
    s = dataclasses.replace(s, mu=case["friction"], edge_contacts=case["edge"], smooth=case["smooth"],
                            near_clip=case["near_clip"])
    return _piled(s, rng)


def _policy(case, seed):
    """Seeded weights of order one at every layer (as scenegen's), made on
    the GPU where there is one: layer 1 has up to 2^28 of them."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    g = torch.Generator(device=dev).manual_seed(int(seed))
    K, H, B = 4 * case["w"] * case["h"], case["hidden"], min(case["bodies"], 32)

    def normal(scale, *shape):
        return torch.randn(*shape, generator=g, device=dev) * scale

    w1 = normal(1.0 / (math.sqrt(K) * 128.0), K, H).to(torch.bfloat16)
    P = dict(in_w=case["w"], in_h=case["h"], act_bodies=B, a_max=np.float32(2.0),
             w1_bf16=w1.view(torch.int16).cpu().numpy().view(np.uint16))
    for k, t in (("b1", normal(0.1, H)), ("w2", normal(1.0 / H, H, H)), ("b2", normal(0.5, H)),
                 ("w3", normal(1.0 / H, H, 3 * B)), ("b3", normal(0.3, 3 * B))):
        P[k] = t.cpu().numpy()
    return P


# the launch shapes the benchmark runs co-scheduled
TUNED = ((vuda.TUNE_PHYS_PRIORITY, 3), (vuda.TUNE_TILE_PRIORITY, 1), (vuda.TUNE_RASTER_THREADS, 128),
         (vuda.TUNE_TILE_WAVES, 2))
SCHEDULES = {v: k for k, v in vuda.SCHED_NAMES.items()}


def _requests(case, seed):
    rng, shape = np.random.default_rng(seed), np.random.default_rng(SHAPES)
    out = []
    for _ in range(case["requests"]):
        n = int(math.exp(shape.uniform(math.log(case["envs"]), math.log(16 * case["envs"]))))
        out.append((sg.make_scene(int(rng.integers(1 << 20)), np.full(n, int(shape.integers(8, 65))),
                                  int(shape.choice([64, 128, 256])), mixed=True), int(shape.integers(50, 151))))
    return out


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] == "serve":
        s["requests"] = _requests(case, seed)
        n = case["requests"] * 16 * case["envs"]
        s["server"] = vuda.Server(cap_envs=n, cap_bodies=64 * n, cap_cams=n, cap_pixels=n << 16,
                                  cu_split=case["split"], schedule=SCHEDULES[case["schedule"]], keep_results=True)
        return s
    scene = _scene(case, seed)
    w = vuda.World(scene)
    s.update(world=w, start=scene.state())
    if case["split"]:
        w.cosched(case["split"])
    if case["tuned"]:
        for k, v in TUNED:
            w.set_tuning(k, v)
    buf = lambda what, t: torch.zeros(w.fetch_bytes(what) // torch.empty(0, dtype=t).element_size(), dtype=t,
                                      device="cuda")
    s["state"] = buf(vuda.FETCH_STATE, torch.float32)
    if case["cams"]:
        s["rgb"] = buf(vuda.FETCH_RGB, torch.uint8)
        s["depth"] = buf(vuda.FETCH_DEPTH, torch.float32 if case["metric"] else torch.int32)
    if case["hidden"]:
        w.set_policy(_policy(case, seed))
        s["actions"] = buf(vuda.FETCH_ACTIONS, torch.float32)
    if case["kind"] == "act":
        w.render()
    return s


def _frames(s):
    w, what = s["world"], vuda.FETCH_DEPTH_METRIC if s["case"]["metric"] else vuda.FETCH_DEPTH
    return {"rgb": w.fetch(vuda.FETCH_RGB, out=s["rgb"]), "depth": w.fetch(what, out=s["depth"])}


def run(s):
    case, w, kind = s["case"], s.get("world"), s["case"]["kind"]
    if kind == "serve":
        srv, left = s["server"], len(s["requests"])
        for rid, (scene, horizon) in enumerate(s["requests"]):
            srv.submit(rid, scene, horizon)
        while left:
            left -= srv.tick()
        return [{"state": srv.result(r, vuda.FETCH_STATE), "rgb": srv.result(r, vuda.FETCH_RGB),
                 "depth": srv.result(r, vuda.FETCH_DEPTH).view(np.int32)} for r, _ in enumerate(s["requests"])]
    if kind == "act":
        w.act()
        return {"actions": w.fetch(vuda.FETCH_ACTIONS, out=s["actions"])}
    w.load_state(s["start"])
    if kind == "step":
        w.step(nsteps=case["iters"])
        return {"state": w.fetch(vuda.FETCH_STATE, out=s["state"])}
    if kind == "observe":
        w.render()
        return _frames(s)
    if kind == "gym":
        for _ in range(case["iters"]):
            w.step()
            w.render()
            out = _frames(s)
            out["state"] = w.fetch(vuda.FETCH_STATE, out=s["state"])
        return out
    if kind == "rollout":
        for _ in range(case["iters"]):
            w.render()
            w.act()
            w.step()
        out = {"actions": w.fetch(vuda.FETCH_ACTIONS, out=s["actions"])}
    else:
        w.run(SCHEDULES[case["schedule"]], case["iters"])
        out = {}
    return dict(_frames(s), state=w.fetch(vuda.FETCH_STATE, out=s["state"]), **out)


def work(case):
    """State and body constants once per step, poses in and pixels out once
    per rendered frame, weights and observations once per policy pass."""
    if case["kind"] == "serve":
        # means of the draws: log-uniform envs, 36 bodies, three frame sizes, 100 steps
        n = case["requests"] * case["envs"] * 15 / math.log(16)
        bodies, pixels, iters = 36 * n, 28672 * n, 100
    else:
        per = case["poisson"] or (case["bodies"] + max(case["bodies_max"], case["bodies"])) / 2
        bodies, iters = per * case["envs"], case["iters"]
        pixels = case["envs"] * case["cams"] * (case["w"] * case["h"] or 28672)
    step_b, frame_b = 120 * bodies, 28 * bodies * case["cams"] + 7 * pixels
    # per body and substep: pose, velocities, integration; per pixel: depth and shade
    step_f, frame_f = 4 * 150 * bodies, 20 * pixels
    K, H, A = 4 * case["w"] * case["h"], case["hidden"], 3 * min(case["bodies"], 32)
    act_b = 2 * K * H + 4 * H * (H + A) + 7 * case["envs"] * case["w"] * case["h"]
    act_f = 2 * case["envs"] * (K * H + H * H + H * A)
    if case["kind"] == "step":
        return {"bytes": step_b, "flops": step_f * iters}
    if case["kind"] == "observe":
        return {"bytes": frame_b, "flops": frame_f}
    if case["kind"] == "act":
        return {"bytes": act_b, "flops": act_f}
    b, f = step_b + frame_b, step_f + frame_f
    if case["kind"] == "rollout":
        b, f = b + act_b, f + act_f
    return {"bytes": b * iters, "flops": f * iters}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def exact(case, seed):
    if case["kind"] == "step":
        return {"state": _simulated(_scene(case, seed), case["iters"])}
    if case["kind"] == "observe" and case["metric"] and not case["near_clip"]:
        scene = _scene(case, seed)
        return {"rgb": None, "depth": _metric(scene, _rendered(scene)[1])}
    if case["kind"] == "act":
        P = _policy(case, seed)
        rgb, depth = _rendered(_scene(case, seed))
        n = case["envs"]
        obs = np.concatenate([rgb.reshape(n, -1), (depth >> 16 & 255).astype(np.uint8).reshape(n, -1)], 1)
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
        h, w1 = 0.0, t(P["w1_bf16"].view(np.int16)).view(torch.bfloat16)
        for k in range(0, obs.shape[1], 8192):
            h = h + t(obs[:, k:k + 8192]).double() @ w1[k:k + 8192].double()
        h = torch.relu(h + t(P["b1"]).double())
        h = torch.relu(h @ t(P["w2"]).double() + t(P["b2"]).double())
        y = h @ t(P["w3"]).double() + t(P["b3"]).double()
        return {"actions": (float(P["a_max"]) * y.clamp(-1, 1)).reshape(-1)}
    return None


def _rendered(scene):
    """(rgb [pixels, 3], depth [pixels]) of the scene's cameras with flat
    shading: the float32 transform and shading and the exact integer
    coverage that define a frame, in numpy."""
    f4, t = np.float32, sg.templates()
    R32, kinds = _rotation(scene.quat, f4), scene.btype
    ext = np.repeat(scene.size[:, None], 3, 1) if scene.ext is None else scene.ext
    sizes = scene.cam_w.astype(np.int64) * scene.cam_h
    base = np.concatenate([[0], np.cumsum(sizes)])
    rgb, depth = np.zeros((base[-1], 3), np.uint8), np.full(base[-1], 0xFFFFFFFF, np.uint32)
    for e in range(scene.n_envs):
        ids = np.arange(scene.body_off[e], scene.body_off[e + 1])
        V, F, C, nv = [t.ground_v], [t.ground_f], [np.full((len(t.ground_f), 3), sg.GROUND_ALBEDO, f4)], len(t.ground_v)
        N = [np.tile(np.array([0, 0, 1], f4), (len(t.ground_f), 1))]
        for b in ids:
            tv, tf, tn = (t.sphere_v, t.sphere_f, t.sphere_n) if kinds[b] == 0 else (t.cube_v, t.cube_f, t.cube_n)
            s, R = tv * ext[b], R32[b]
            turn = lambda v: np.stack([(R[k, 0] * v[:, 0] + R[k, 1] * v[:, 1]) + R[k, 2] * v[:, 2] for k in range(3)], 1)
            V.append(scene.pos[b] + turn(s))
            F.append(tf + nv)
            N.append(turn(tn))
            C.append(np.tile(sg.PALETTE[scene.albedo[b]], (len(tf), 1)))
            nv += len(tv)
        V, F, N, C = (np.concatenate(a) for a in (V, F, N, C))
        light = np.maximum(f4(0), (N[:, 0] * sg.LIGHT[0] + N[:, 1] * sg.LIGHT[1]) + N[:, 2] * sg.LIGHT[2])
        col = np.minimum(f4(255), np.rint(C * (f4(0.2) + f4(0.8) * light)[:, None] * f4(255))).astype(np.uint64)
        for c in range(scene.cam_off[e], scene.cam_off[e + 1]):
            W, H, vp = int(scene.cam_w[c]), int(scene.cam_h[c]), scene.cam_vp[c].reshape(4, 4)
            cx, cy, cz, cw = (((m[0] * V[:, 0] + m[1] * V[:, 1]) + m[2] * V[:, 2]) + m[3] for m in vp)
            with np.errstate(all="ignore"):
                px = (cx / cw * f4(0.5) + f4(0.5)) * f4(W)
                py = (f4(0.5) - cy / cw * f4(0.5)) * f4(H)
                z = cz / cw
                ok = (cw >= f4(sg.NEAR)) & ~((np.abs(px) > sg.GUARD_BAND) | (np.abs(py) > sg.GUARD_BAND))
            X = np.where(ok, np.rint(px * f4(256)), 0).astype(np.int64)
            Y = np.where(ok, np.rint(py * f4(256)), 0).astype(np.int64)
            key = _covered(X, Y, z, ok, F[:, [0, 2, 1]], col, W, H)
            hit = key != ~np.uint64(0)
            at = slice(base[c], base[c + 1])
            depth[at] = np.where(hit, key >> np.uint64(40), 0xFFFFFFFF).astype(np.uint32)
            rgb[at] = np.where(hit[:, None], np.stack([key >> np.uint64(8 * k) & np.uint64(255) for k in range(3)], 1), 0)
    return rgb, depth


def _covered(X, Y, z, ok, F, col, W, H):
    """Nearest depth key per pixel of the snapped triangles F."""
    prim = np.nonzero(ok[F].all(1))[0]
    x, y = X[F[prim]], Y[F[prim]]
    area = (x[:, 1] - x[:, 0]) * (y[:, 2] - y[:, 0]) - (y[:, 1] - y[:, 0]) * (x[:, 2] - x[:, 0])
    x0, x1 = np.maximum(0, x.min(1) + 127 >> 8), np.minimum(W - 1, x.max(1) - 128 >> 8)
    y0, y1 = np.maximum(0, y.min(1) + 127 >> 8), np.minimum(H - 1, y.max(1) - 128 >> 8)
    keep = (area > 0) & (x0 <= x1) & (y0 <= y1)
    prim, x, y, area, x0, x1, y0, y1 = (a[keep] for a in (prim, x, y, area, x0, x1, y0, y1))
    zv, inv = z[F[prim]].astype(np.float32), np.float32(1) / area.astype(np.float32)
    n = (x1 - x0 + 1) * (y1 - y0 + 1)
    tri = np.repeat(np.arange(len(n)), n)
    f = np.arange(len(tri)) - np.repeat(np.cumsum(n) - n, n)
    bw = (x1 - x0 + 1)[tri]
    ix, iy = x0[tri] + f % bw, y0[tri] + f // bw
    inside, E = np.ones(len(tri), bool), []
    for e in range(3):
        a, b = (e + 1) % 3, (e + 2) % 3
        dx, dy = x[:, b] - x[:, a], y[:, b] - y[:, a]
        v = dx[tri] * (256 * iy + 128 - y[tri, a]) - dy[tri] * (256 * ix + 128 - x[tri, a])
        inside &= (v > 0) | ((v == 0) & ((dy < 0) | ((dy == 0) & (dx > 0)))[tri])
        E.append(v)
    tri, ix, iy = tri[inside], ix[inside], iy[inside]
    e0, e1, e2 = (v[inside].astype(np.float32) for v in E)
    zz = ((e0 * zv[tri, 0] + e1 * zv[tri, 1]) + e2 * zv[tri, 2]) * inv[tri]
    D = np.rint(np.clip(zz, np.float32(0), np.float32(1)) * np.float32(16777215)).astype(np.uint64)
    c = col[prim[tri]]
    low = c[:, 0] | c[:, 1] << np.uint64(8) | c[:, 2] << np.uint64(16)
    key = D << np.uint64(40) | prim[tri].astype(np.uint64) << np.uint64(24) | low
    out = np.full(W * H, ~np.uint64(0))
    np.minimum.at(out, iy * W + ix, key)
    return out


def _metric(scene, depth):
    out, pos = [], 0
    for c in range(scene.n_cams):
        m, n = scene.cam_vp[c].astype(np.float64).reshape(4, 4), int(scene.cam_w[c]) * int(scene.cam_h[c])
        alpha = m[2, :3] @ m[3, :3] / (m[3, :3] @ m[3, :3])
        D = depth[pos:pos + n]
        d = (m[2, 3] - alpha * m[3, 3]) / (D.astype(np.float64) / 16777215.0 - alpha)
        out.append(np.where(D == 0xFFFFFFFF, np.inf, d))
        pos += n
    return np.concatenate(out)


def _simulated(scene, nsteps):
    """State [B, 13] after nsteps steps in float64: penalty contacts of
    spheres, cubes and boxes, regularized Coulomb friction, edge-edge points
    by the separating-axis test, semi-implicit Euler."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev).double()
    B, n = scene.n_bodies, scene.counts().astype(np.int64)
    p, v, q, w = t(scene.pos), t(scene.vel), t(scene.quat), t(scene.omega)
    size, rb, inv_m, inv_I = t(scene.size), t(scene.rbound), t(scene.inv_m), t(scene.inv_I)
    kind = torch.from_numpy(scene.btype.astype(np.int64)).to(dev)
    boxed = kind != 0
    e = size[:, None].repeat(1, 3) if scene.ext is None else torch.where(kind[:, None] == 2, t(scene.ext), size[:, None])
    I3 = torch.ones_like(p) if scene.inertia is None else torch.where(kind[:, None] == 2, t(scene.inertia), 1.0)
    h32 = np.float32(scene.dt) / np.float32(scene.substeps)
    h, hh, g = float(h32), float(np.float32(0.5) * h32), t(np.array(scene.gravity, np.float32))
    kc, cd, mu, eps = (float(np.float32(a)) for a in (scene.k_contact, scene.c_damp, scene.mu, scene.v_eps))
    # pairs i < j of each env
    i, j = [], []
    for m in np.unique(n):
        a, b = np.triu_indices(int(m), 1)
        at = scene.body_off[:-1][n == m].astype(np.int64)[:, None]
        i.append((at + a).ravel())
        j.append((at + b).ravel())
    I, J = (torch.from_numpy(np.concatenate(a)).to(dev) for a in (i, j))
    corners = t(np.array([[1.0 if c >> a & 1 else -1.0 for a in range(3)] for c in range(8)]))
    up = t(np.array([0.0, 0.0, 1.0]))
    cross = lambda a, b: torch.linalg.cross(a, b, dim=-1)
    dot = lambda a, b: (a * b).sum(-1)
    for _ in range(nsteps * scene.substeps):
        qw, qx, qy, qz = q.unbind(1)
        R = torch.stack([1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                         2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                         2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)], 1).view(-1, 3, 3)
        F, T = torch.zeros_like(p), torch.zeros_like(p)

        def push(A, Bd, nrm, depth, x):
            """Contact points x of body A, pushed along nrm by body Bd (None: the ground)."""
            rel = v[A] + cross(w[A], x - p[A])
            if Bd is not None:
                rel = rel - (v[Bd] + cross(w[Bd], x - p[Bd]))
            vn = dot(rel, nrm)
            f = (kc * depth - cd * vn).clamp(min=0.0)
            force = nrm * f[:, None]
            if mu > 0.0:
                vt = rel - nrm * vn[:, None]
                force = force - vt * (mu * f / dot(vt, vt).sqrt().clamp(min=eps))[:, None]
            F.index_add_(0, A, force)
            T.index_add_(0, A, cross(x - p[A], force))
            if Bd is not None:
                F.index_add_(0, Bd, -force)
                T.index_add_(0, Bd, cross(x - p[Bd], -force))

        d = p[I] - p[J]
        near = dot(d, d) <= (rb[I] + rb[J]) ** 2
        i, j = I[near], J[near]
        # spheres
        m = ~boxed[i] & ~boxed[j]
        a, b = i[m], j[m]
        d = p[a] - p[b]
        L, sr = dot(d, d).sqrt(), size[a] + size[b]
        m = L < sr
        a, b, d, L, sr = a[m], b[m], d[m], L[m], sr[m]
        nrm = torch.where(L[:, None] > 0, d / L[:, None], up)
        push(a, b, nrm, sr - L, p[b] + nrm * (size[b] - 0.5 * (sr - L))[:, None])
        # a sphere and a box
        m = boxed[i] ^ boxed[j]
        a, b = torch.where(boxed[i], j, i)[m], torch.where(boxed[i], i, j)[m]
        u = dot(R[b].transpose(1, 2), (p[a] - p[b])[:, None])
        c = torch.minimum(torch.maximum(u, -e[b]), e[b])
        r = u - c
        L = dot(r, r).sqrt()
        m = L < size[a]
        a, b, u, c, r, L = a[m], b[m], u[m], c[m], r[m], L[m]
        depth, axis = (e[b] - u.abs()).min(1)
        face = torch.nn.functional.one_hot(axis, 3) * torch.where(u.gather(1, axis[:, None]) >= 0, 1.0, -1.0)
        nl = torch.where(L[:, None] > 0, r / L[:, None], face.double())
        push(a, b, dot(R[b], nl[:, None]), torch.where(L > 0, size[a] - L, size[a] + depth), p[b] + dot(R[b], c[:, None]))
        # boxes: the corners of either in the other
        m = boxed[i] & boxed[j]
        bi, bj = i[m], j[m]
        for a, b in ((bi, bj), (bj, bi)):
            x = p[a][:, None] + torch.einsum("prc,pkc->pkr", R[a], corners * e[a][:, None])
            u = torch.einsum("pcr,pkc->pkr", R[b], x - p[b][:, None])
            s, k = (u.abs() < e[b][:, None]).all(2).nonzero(as_tuple=True)
            a2, b2, x2, u2 = a[s], b[s], x[s, k], u[s, k]
            depth, axis = (e[b2] - u2.abs()).min(1)
            face = torch.nn.functional.one_hot(axis, 3) * torch.where(u2.gather(1, axis[:, None]) >= 0, 1.0, -1.0)
            push(a2, b2, dot(R[b2], face.double()[:, None]), depth, x2)
        if scene.edge_contacts and len(bi):
            Ra, Rb, d = R[bi], R[bj], p[bi] - p[bj]
            A3, B3 = Ra.transpose(1, 2), Rb.transpose(1, 2)  # rows: the axes
            L = cross(A3[:, :, None].expand(-1, 3, 3, 3), B3[:, None].expand(-1, 3, 3, 3)).reshape(-1, 9, 3)
            l2 = dot(L, L)
            valid = torch.cat([torch.ones_like(l2[:, :6], dtype=torch.bool), l2 >= 1e-6], 1)
            L = torch.cat([A3, B3, L / l2.clamp(min=1e-30).sqrt()[:, :, None]], 1)
            over = ((L @ Ra).abs() * e[bi][:, None]).sum(2) + ((L @ Rb).abs() * e[bj][:, None]).sum(2) - \
                (L @ d[:, :, None])[:, :, 0].abs()
            sep = (valid & ~(over > 0)).any(1)
            eo, k = torch.where(valid[:, 6:], over[:, 6:], math.inf).min(1)
            s = (~sep & (eo < 0.95 * over[:, :6].min(1).values)).nonzero()[:, 0]
            k, eo, a, b, d = k[s], eo[s], bi[s], bj[s], d[s]
            L = L[s, 6 + k]
            nrm = torch.where(dot(L, d)[:, None] < 0, -L, L)
            ka, kb = torch.nn.functional.one_hot(k // 3, 3).double(), torch.nn.functional.one_hot(k % 3, 3).double()
            ui, uj = dot(R[a].transpose(1, 2), nrm[:, None]), dot(R[b].transpose(1, 2), nrm[:, None])
            ci = p[a] + dot(R[a], ((1 - ka) * torch.where(ui > 0, -e[a], e[a]))[:, None])
            cj = p[b] + dot(R[b], ((1 - kb) * torch.where(uj > 0, e[b], -e[b]))[:, None])
            da, db, y = dot(R[a], ka[:, None]), dot(R[b], kb[:, None]), ci - cj
            bb, dd, ee = dot(da, db), dot(da, y), dot(db, y)
            ha, hb = dot(e[a], ka), dot(e[b], kb)
            sa = torch.minimum(torch.maximum((bb * ee - dd) / (1 - bb * bb), -ha), ha)
            tb = torch.minimum(torch.maximum((ee - bb * dd) / (1 - bb * bb), -hb), hb)
            push(a, b, nrm, eo, 0.5 * ((ci + da * sa[:, None]) + (cj + db * tb[:, None])))
        # the ground
        a = (~boxed & (p[:, 2] < size)).nonzero()[:, 0]
        push(a, None, up.expand(len(a), 3), size[a] - p[a, 2], p[a] - up * size[a][:, None])
        a = (boxed & (p[:, 2] < rb)).nonzero()[:, 0]
        x = p[a][:, None] + torch.einsum("prc,pkc->pkr", R[a], corners * e[a][:, None])
        s, k = (x[:, :, 2] < 0).nonzero(as_tuple=True)
        push(a[s], None, up.expand(len(s), 3), -x[s, k, 2], x[s, k])
        # semi-implicit Euler
        v = v + (F * inv_m[:, None] + g) * h
        p = p + v * h
        wb, tb = dot(R.transpose(1, 2), w[:, None]), dot(R.transpose(1, 2), T[:, None])
        turned = dot(R, (wb + (tb - cross(wb, I3 * wb)) / I3 * h)[:, None])
        w = torch.where(kind[:, None] == 2, turned, w + T * inv_I[:, None] * h)
        wx, wy, wz = w.unbind(1)
        q = q + hh * torch.stack([-wx * qx - wy * qy - wz * qz, wx * qw + wy * qz - wz * qy,
                                  wy * qw + wz * qx - wx * qz, wz * qw + wx * qy - wy * qx], 1)
        q = q / q.norm(dim=1, keepdim=True)
    return torch.cat([p, v, q, w], 1).reshape(-1)
