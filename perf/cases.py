"""Performance cases of the planner library: plan steps, distance fields, occupancy
updates and serving, through the package's public entry points.

Sizes are those of this repository's workloads, tests and benchmark (tiny, mid,
paper-shaped, reactive, the largest tested batch, the serving mix, 200^3 maps with
640x480 images) and ragged neighbours of them.  A case is a dict of plain values with a
``kind``:

* ``step``  one plan step (K rollouts of H steps on an nx x ny x nz grid).  ``bounds``:
  "none", "kept" (built once per map, outside the pass: a static map), "period" (a new map
  each period: bounds of the robot's reach, then the step) or "next" (the step also builds
  the next map's bounds; two maps alternate).  ``receding``: the step executes u*_0 and
  shifts the nominal sequence on the device.  ``noise``: "buffer" or "device" (sampled by
  the step).  ``grid``: "f32" or "f16".  ``gap``: smallest link distance of a
  self-collision pair.
* ``field`` the signed distance field of an occupancy grid (and its squared distances
  with ``d2``).
* ``map``   one occupancy update from a depth image (``mask``: the robot is masked).
* ``serve`` one request of every one of ``n`` controllers, submitted together and served
  until the last result is polled.

The scenes are boxes and spheres around the arm; the distance grids of ``step`` and
``serve`` hold the analytic signed distance of those primitives.
"""
from __future__ import annotations

import ctypes
import math
import random

import numpy as np
import torch

from paper_2512_22575_amd import smpc as S

DEV = "cuda:0"
NDOF = 7

# The 7-DoF arm of the repository's workloads (modified DH) and its limits.
ARM_A = (0.0, 0.0, 0.0, 0.0825, -0.0825, 0.0, 0.088)
ARM_D = (0.333, 0.0, 0.316, 0.0, 0.384, 0.0, 0.0)
ARM_ALPHA = (0.0, -math.pi / 2, math.pi / 2, math.pi / 2, -math.pi / 2, math.pi / 2, math.pi / 2)
Q_MIN = (-2.8973, -1.7628, -2.8973, -3.0718, -2.8973, -0.0175, -2.8973)
Q_MAX = (2.8973, 1.7628, 2.8973, -0.0698, 2.8973, 3.7525, 2.8973)
QD_MAX = (2.175, 2.175, 2.175, 2.175, 2.61, 2.61, 2.61)
QDD_MAX = (15.0, 7.5, 10.0, 12.5, 15.0, 20.0, 20.0)
READY = (0.0, -0.785, 0.0, -2.356, 0.0, 1.571, 0.785)  # a working posture, arm clear of itself

WEIGHTS = dict(w_pose_t=10.0, w_pose_r=2.0, w_term_t=10.0, w_term_r=2.0, w_env=100.0, d_act=0.03,
               w_self=100.0, w_q=10.0, w_qd=10.0, w_qdd=10.0, limit_margin_frac=0.05,
               w_smooth=0.01, w_ns=0.0)
SIGMA = 0.5
LAMBDA = 1.0

MAP_PRM = dict(tol=0.025, l_hit=0.85, l_miss=-0.4, l_min=-2.0, l_max=3.5, l_occ=0.0,
               robot_pad=0.01)


def _step(name, K, H, nx, ny, nz, voxel, dt=0.02, prims=20, **kw):
    c = dict(name=name, kind="step", K=K, H=H, nx=nx, ny=ny, nz=nz, voxel=voxel, dt=dt,
             prims=prims, grid="f32", noise="buffer", bounds="none", receding=False, gap=2)
    c.update(kw)
    return c


def _field(name, nx, ny, nz, voxel, prims, d2=False):
    return dict(name=name, kind="field", nx=nx, ny=ny, nz=nz, voxel=voxel, prims=prims, d2=d2)


def _map(name, nx, ny, nz, voxel, prims, width, height, mask=True, occ=True):
    return dict(name=name, kind="map", nx=nx, ny=ny, nz=nz, voxel=voxel, prims=prims,
                width=width, height=height, mask=mask, occ=occ)


def listed():
    return [
        # The smallest call: a debugging or embedded-size step through the Planner class,
        # where launches and the host path count.
        _step("step_tiny", 64, 16, 32, 32, 32, 0.05, dt=0.05, prims=5),
        # The paper's own setting: M = 512 at 50 Hz on its 3 x 3 x 0.5 m map, a map per
        # period, receding horizon.
        _step("step_paper", 512, 40, 150, 150, 25, 0.02, bounds="period", receding=True),
        # An ordinary step on a static float16 map, disturbances sampled on the device.
        _step("step_mid_f16", 1024, 32, 64, 64, 64, 0.03, grid="f16", noise="device",
              bounds="kept"),
        # Odd sizes everywhere, no bounds, self-collision pairs of neighbouring links too.
        _step("step_ragged", 3001, 37, 101, 83, 67, 0.021, gap=1),
        # Reactive replanning closed loop: K = 4096, H = 40, a new 200^3 map every period.
        _step("loop_reactive", 4096, 40, 200, 200, 200, 0.01, prims=40, bounds="next",
              receding=True),
        # The largest tested batch at the longest horizon, static map, sampled on the device.
        _step("step_large", 65536, 64, 256, 256, 256, 0.008, prims=40, noise="device",
              bounds="kept"),
        # Distance field of a small map.
        _field("field_small", 64, 64, 64, 0.03, 20),
        # Distance field of the reactive map, once per period.
        _field("field_reactive", 200, 200, 200, 0.01, 40),
        # A large ragged map, squared distances wanted as well.
        _field("field_ragged", 333, 257, 141, 0.01, 60, d2=True),
        # Occupancy update of the reactive map from a VGA depth image, robot masked.
        _map("map_reactive", 200, 200, 200, 0.01, 40, 640, 480),
        # A small ragged map from a QVGA image, no robot in view, log-odds only.
        _map("map_ragged", 121, 97, 75, 0.025, 20, 320, 240, mask=False, occ=False),
        # Serving: every one of 64 controllers asks for a plan at once.
        dict(name="serve_burst", kind="serve", n=64, voxel_lo=0.01, voxel_hi=0.03),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi, most):
    while True:
        n = [_logint(rng, lo, hi) for _ in range(3)]
        if n[0] * n[1] * n[2] <= most:
            if rng.random() < 0.5:  # maps are often cubes, and rows often multiples of 4
                n = [n[0] // 4 * 4] * 3 if n[0] ** 3 <= most else [n[0] // 4 * 4, n[1], n[2]]
            return n


def draw(rng: random.Random):
    kind = rng.choice(["step", "step", "step", "field", "field", "map", "serve"])
    if kind == "step":
        while True:
            K, H = _logint(rng, 32, 65536), rng.randint(5, 64)
            if K * H <= 65536 * 64:
                break
        nx, ny, nz = _sides(rng, 24, 256, 200 ** 3)
        bounds = rng.choice(["none", "kept", "period", "next"])
        f16 = rng.random() < 0.25
        c = _step("", K, H, nx, ny, nz, round(2.0 / max(nx, ny, nz), 4), prims=rng.randint(5, 60),
                  bounds=bounds, receding=bounds in ("period", "next"),
                  noise=rng.choice(["buffer", "device"]), grid="f16" if f16 else "f32",
                  gap=rng.choice([2, 2, 2, 1]))
    elif kind == "field":
        nx, ny, nz = _sides(rng, 24, 480, 333 * 257 * 141)
        c = _field("", nx, ny, nz, round(2.0 / max(nx, ny, nz), 4), rng.randint(5, 60),
                   d2=rng.random() < 0.3)
    elif kind == "map":
        nx, ny, nz = _sides(rng, 24, 320, 12_000_000)
        width = rng.choice([160, 320, 424, 640, 848])
        c = _map("", nx, ny, nz, round(2.0 / max(nx, ny, nz), 4), rng.randint(5, 60), width,
                 width * 3 // 4, mask=rng.random() < 0.7, occ=rng.random() < 0.8)
    else:
        c = dict(kind="serve", n=rng.randint(4, 64), voxel_lo=0.01,
                 voxel_hi=round(rng.uniform(0.015, 0.03), 4))
    c.pop("name", None)
    return c


# --- inputs ------------------------------------------------------------------------

class _Robot:
    """The arm with four spheres along each link and the pairs of links `gap` or more apart."""

    def __init__(self, rng, gap):
        self.a, self.d = np.array(ARM_A), np.array(ARM_D)
        self.alpha = np.array(ARM_ALPHA)
        self.q_min, self.q_max = np.array(Q_MIN), np.array(Q_MAX)
        self.qd_max, self.qdd_max = np.array(QD_MAX), np.array(QDD_MAX)
        self.qd_min, self.qdd_min = -self.qd_max, -self.qdd_max
        self.q_ref = 0.5 * (self.q_min + self.q_max)
        link, centre = [], []
        for i in range(NDOF):
            if i + 1 < NDOF:
                al, dn = self.alpha[i + 1], self.d[i + 1]
                end = np.array([self.a[i + 1], -math.sin(al) * dn, math.cos(al) * dn])
            else:
                end = np.array([0.0, 0.0, 0.1])
            for j in range(4):
                link.append(i + 1)
                centre.append((j + 0.5) / 4 * end)
        self.sphere_link = np.array(link, np.int32)
        self.sphere_center = np.array(centre)
        self.sphere_radius = rng.uniform(0.04, 0.08, size=len(link))
        self.pairs = np.array([(i, j) for i in range(28) for j in range(i + 1, 28)
                               if abs(link[i] - link[j]) >= gap], np.int32)


class _Ctx:
    """A library context with a robot, closed with the state that holds it."""

    def __init__(self, robot):
        st, self.h = S.smpc_create(0)
        _ok(st)
        _ok(S.smpc_set_robot(self.h, S.robot_desc(robot)))

    def __del__(self):
        S.smpc_destroy(self.h)


class _Service:
    def __init__(self, ctx, budget, max_batch):
        self.ctx = ctx  # outlives the server
        st, self.h = S.smpc_server_create(ctx.h, budget, max_batch)
        _ok(st)

    def __del__(self):
        S.smpc_server_destroy(self.h)


def _ok(st):
    if st != S.SMPC_OK:
        raise RuntimeError(S.smpc_status_string(st))


def _f32(x):
    return np.asarray(x, np.float32)


def _origin(nx, ny, nz, voxel):
    return _f32([-0.5 * nx * voxel, -0.5 * ny * voxel, 0.0])


def _scene(rng, nx, ny, nz, voxel, n):
    """Boxes and spheres in the map's inner 90 %, clear of the arm's base column."""
    ext = np.array([nx, ny, nz]) * voxel
    lo = np.array([-0.45 * ext[0], -0.45 * ext[1], 0.05 * ext[2]])
    hi = np.array([0.45 * ext[0], 0.45 * ext[1], 0.95 * ext[2]])
    prims = []
    for i in range(n):
        for _ in range(200):
            c = rng.uniform(lo, hi)
            box = i % 2 == 0
            half = 0.5 * rng.uniform(0.1, 0.4, size=3) if box else rng.uniform(0.05, 0.2, size=1)
            reach = math.hypot(half[0], half[1]) if box else half[0]
            if math.hypot(c[0], c[1]) - reach > 0.2:
                prims.append((box, c, half))
                break
    return prims


def _sdf(prims, nx, ny, nz, voxel):
    """Signed distance of the primitives at the voxel centres, float32 [nz][ny][nx]."""
    o = _origin(nx, ny, nz, voxel)
    ax = [torch.arange(n, device=DEV, dtype=torch.float32) * voxel + (float(o[k]) + 0.5 * voxel)
          for k, n in enumerate((nx, ny, nz))]
    out = torch.full((nz, ny, nx), 10.0, device=DEV)
    for box, c, half in prims:
        r = [(ax[k] - float(c[k])).abs() for k in range(3)]
        if box:
            q = [r[k] - float(half[k]) for k in range(3)]
            p = [x.clamp(min=0.0).square() for x in q]
            outer = (p[2][:, None, None] + p[1][None, :, None] + p[0][None, None, :]).sqrt()
            inner = torch.maximum(torch.maximum(q[2][:, None, None], q[1][None, :, None]),
                                  q[0][None, None, :]).clamp(max=0.0)
            d = outer + inner
        else:
            s = [x.square() for x in r]
            d = (s[2][:, None, None] + s[1][None, :, None] + s[0][None, None, :]).sqrt()
            d = d - float(half[0])
        out = torch.minimum(out, d)
    return out


def _pose(rng):
    q = rng.normal(size=4)
    w, x, y, z = q / np.linalg.norm(q)
    T = np.eye(4)
    T[:3, :3] = [[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                 [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                 [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]]
    T[:3, 3] = rng.uniform([0.25, -0.45, 0.15], [0.65, 0.45, 0.85])
    return _f32(T)


def _normal(seed, *shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return torch.randn(shape, generator=g, device=DEV)


def _step_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 1])
    nx, ny, nz, vox = case["nx"], case["ny"], case["nz"], float(np.float32(case["voxel"]))
    K, H = case["K"], case["H"]
    i = dict(robot=_Robot(rng, case["gap"]), K=K, H=H, voxel=vox, origin=_origin(nx, ny, nz, vox),
             q0=_f32(np.array(READY) + rng.uniform(-0.3, 0.3, size=NDOF)),
             qd0=_f32(rng.uniform(-0.2, 0.2, size=NDOF)), T_goal=_pose(rng),
             dt=float(np.float32(case["dt"])), seed=int(rng.integers(1 << 62)))
    prims = _scene(rng, nx, ny, nz, vox, case["prims"])
    grids = [_sdf(prims, nx, ny, nz, vox)]
    if case["bounds"] == "next":  # the map one period later: everything drifted a little
        moved = [(b, c + rng.normal(size=3) * 0.004, h) for b, c, h in prims]
        grids.append(_sdf(moved, nx, ny, nz, vox))
    i["grids"] = grids
    i["U"] = 0.1 * _normal(seed * 4 + 1, H, NDOF)
    i["noise"] = SIGMA * _normal(seed * 4 + 2, K, H, NDOF) if case["noise"] == "buffer" else None
    return i


def _prepare_step(case, seed):
    i = _step_inputs(case, seed)
    K, H, nx, ny, nz = case["K"], case["H"], case["nx"], case["ny"], case["nz"]
    stream = torch.cuda.current_stream().cuda_stream
    f16 = case["grid"] == "f16"
    dtype = S.GRID_F16 if f16 else S.GRID_F32
    grids = []
    for g in i["grids"]:
        if f16:
            h = torch.empty((nz, ny, nx), dtype=torch.float16, device=DEV)
            _ok(S.smpc_grid_to_f16(g.data_ptr(), h.data_ptr(), g.numel(), 1.0, stream))
            g = h
        grids.append(g)
    planner = S.Planner(i["robot"], device=0)
    s = dict(case=case, planner=planner, inputs=i, grids=grids, dtype=dtype, stream=stream, at=0)
    s["reach"] = planner.robot_reach()
    cells = S.smpc_grid_coarse_cells(nx, ny, nz)
    kept = case["bounds"]
    s["tables"] = [torch.empty(cells, device=DEV) for _ in range(2 if kept == "next" else 1)]
    s["costs"] = torch.empty(K, device=DEV)
    s["weights"] = torch.empty(K, device=DEV)
    s["stats"] = torch.empty(4, device=DEV)
    # Receding: two nominal sequences and two joint states alternate, all on the device.
    s["U"] = [i["U"].clone(), torch.empty_like(i["U"])]
    s["X"] = [torch.from_numpy(np.concatenate([i["q0"], i["qd0"]])).to(DEV),
              torch.zeros(2 * NDOF, device=DEV)]
    s["u0"] = torch.zeros(NDOF, device=DEV)
    if kept == "kept":
        _ok(S.smpc_grid_coarse_min(grids[0], dtype, s["tables"][0].data_ptr(), stream))
    elif kept == "next":
        _ok(S.smpc_grid_coarse_min_ball(grids[0], dtype, i["origin"], i["voxel"], *s["reach"],
                                        s["tables"][0].data_ptr(), stream))
    rec = case["receding"]
    s["args"] = [
        S.plan_args(i["q0"], i["qd0"], i["T_goal"], grids[p % len(grids)], i["origin"], i["voxel"],
                    i["noise"], s["U"][p], s["U"][1 - p], K, H, i["dt"], LAMBDA, WEIGHTS,
                    costs_out=s["costs"], weights_out=s["weights"], stats_out=s["stats"],
                    seed=i["seed"], sigma=[SIGMA] * NDOF, grid_dtype=dtype,
                    coarse=s["tables"][p % len(s["tables"])] if kept != "none" else None,
                    receding=rec, u0_out=s["u0"] if rec else None,
                    state_in=s["X"][p] if rec else None, state_out=s["X"][1 - p] if rec else None)
        for p in (0, 1)]
    return s


def _run_step(s):
    case, i, p = s["case"], s["inputs"], s["at"]
    kept = case["bounds"]
    if case["K"] * case["H"] <= 1024 and kept == "none" and i["noise"] is not None:
        # The smallest steps come from interactive programs: the Planner class, tensors in hand.
        s["planner"].plan_step(q0=i["q0"], qd0=i["qd0"], T_goal=i["T_goal"], grid=s["grids"][0],
                               origin=i["origin"], voxel=i["voxel"], noise=i["noise"],
                               U_in=s["U"][0], U_out=s["U"][1], dt=i["dt"], lam=LAMBDA,
                               weights=WEIGHTS, costs_out=s["costs"], weights_out=s["weights"],
                               stats_out=s["stats"], grid_dtype=s["dtype"], stream=s["stream"])
    elif kept == "next":
        q = (p + 1) % 2
        _ok(S.smpc_plan_step_then_bounds(s["planner"]._ctx, s["args"][p], s["grids"][q], s["dtype"],
                                         i["origin"], i["voxel"], *s["reach"],
                                         s["tables"][q].data_ptr(), s["stream"]))
    else:
        if kept == "period":
            _ok(S.smpc_grid_coarse_min_ball(s["grids"][0], s["dtype"], i["origin"], i["voxel"],
                                            *s["reach"], s["tables"][0].data_ptr(), s["stream"]))
        _ok(S.smpc_plan_step(s["planner"]._ctx, s["args"][p], s["stream"]))
    out = dict(U=s["U"][1 - p], costs=s["costs"], weights=s["weights"], stats=s["stats"])
    if case["receding"]:
        out.update(u0=s["u0"], state=s["X"][1 - p])
        s["at"] = 1 - p
    if kept in ("period", "next"):
        out["bounds"] = s["tables"][(p + 1) % 2 if kept == "next" else 0]
    return out


def _field_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 2])
    nx, ny, nz, vox = case["nx"], case["ny"], case["nz"], float(np.float32(case["voxel"]))
    prims = _scene(rng, nx, ny, nz, vox, case["prims"])
    return (_sdf(prims, nx, ny, nz, vox) <= 0.0).to(torch.uint8), vox


def _prepare_field(case, seed):
    occ, vox = _field_inputs(case, seed)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    need = S.smpc_edt_workspace_bytes(nx, ny, nz)
    return dict(case=case, occ=occ, voxel=vox, need=need,
                phi=torch.empty((nz, ny, nx), device=DEV),
                d2=torch.empty((2, nz, ny, nx), dtype=torch.int32, device=DEV) if case["d2"] else None,
                work=torch.empty((need + 3) // 4, dtype=torch.int32, device=DEV),
                stream=torch.cuda.current_stream().cuda_stream)


def _run_field(s):
    c, d2 = s["case"], s["d2"]
    _ok(S.smpc_edt(s["occ"].data_ptr(), c["nx"], c["ny"], c["nz"], s["voxel"], s["phi"].data_ptr(),
                   d2.data_ptr() if d2 is not None else None, s["work"].data_ptr(), s["need"],
                   s["stream"]))
    return dict(phi=s["phi"], d2=d2) if d2 is not None else dict(phi=s["phi"])


def _camera(case):
    """Pinhole camera above a corner of the workspace, looking at the arm."""
    w, h = case["width"], case["height"]
    eye, target = np.array([1.2, -0.9, 0.9]), np.array([0.0, 0.0, 0.35])
    z = (target - eye) / np.linalg.norm(target - eye)
    x = np.cross(z, [0.0, 0.0, 1.0])
    x /= np.linalg.norm(x)
    T = np.eye(4)
    T[:3, 0], T[:3, 1], T[:3, 2], T[:3, 3] = x, np.cross(z, x), z, eye
    return dict(f=float(np.float32(0.9 * w)), cx=w / 2.0, cy=h / 2.0, w=w, h=h, T=_f32(T),
                lo=0.1, hi=4.0)


def _depth(prims, cam):
    """z-depth of the first surface along each pixel's ray, 0 where nothing is in range."""
    T = torch.from_numpy(cam["T"].astype(np.float64)).to(DEV)
    u = (torch.arange(cam["w"], device=DEV, dtype=torch.float64) + 0.5 - cam["cx"]) / cam["f"]
    v = (torch.arange(cam["h"], device=DEV, dtype=torch.float64) + 0.5 - cam["cy"]) / cam["f"]
    d = u[None, :, None] * T[:3, 0] + v[:, None, None] * T[:3, 1] + T[:3, 2]
    o, best = T[:3, 3], torch.full((cam["h"], cam["w"]), math.inf, device=DEV, dtype=torch.float64)
    for box, c, half in prims:
        m = torch.from_numpy(np.asarray(c, np.float64)).to(DEV)
        if box:
            hs = torch.from_numpy(np.asarray(half, np.float64)).to(DEV)
            a, b = (m - hs - o) / d, (m + hs - o) / d
            near, far = torch.minimum(a, b).amax(-1), torch.maximum(a, b).amin(-1)
            t = torch.where((far >= near) & (near > 0), near, torch.full_like(near, math.inf))
        else:
            oc = o - m
            A, B = (d * d).sum(-1), (d * oc).sum(-1)
            disc = B * B - A * (float((oc * oc).sum()) - float(half[0]) ** 2)
            t = (-B - disc.clamp(min=0.0).sqrt()) / A
            t = torch.where((disc >= 0) & (t > 0), t, torch.full_like(t, math.inf))
        best = torch.minimum(best, t)
    ok = (best >= cam["lo"]) & (best <= cam["hi"])
    return torch.where(ok, best, torch.zeros_like(best)).float()


def _map_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 3])
    nx, ny, nz, vox = case["nx"], case["ny"], case["nz"], float(np.float32(case["voxel"]))
    robot = _Robot(rng, 2)
    q = _f32(np.array(READY) + rng.uniform(-0.3, 0.3, size=NDOF))
    cam = _camera(case)
    prims = _scene(rng, nx, ny, nz, vox, case["prims"])
    depth = _depth(prims, cam)
    # Dropouts of the sensor, and a map that earlier images have already touched.
    depth[_normal(seed * 4 + 1, cam["h"], cam["w"]) > 2.3] = 0.0
    L = (_normal(seed * 4 + 2, nz, ny, nx) * 1.2 - 0.4).clamp(MAP_PRM["l_min"], MAP_PRM["l_max"])
    return dict(robot=robot, q=q, cam=cam, depth=depth, L=L, voxel=vox,
                origin=_origin(nx, ny, nz, vox))


def _prepare_map(case, seed):
    i = _map_inputs(case, seed)
    cam = i["cam"]
    need = S.smpc_ogm_workspace_bytes(cam["w"], cam["h"])
    return dict(case=case, inputs=i, planner=S.Planner(i["robot"], device=0),
                cam=S.make_camera(cam["f"], cam["f"], cam["cx"], cam["cy"], cam["w"], cam["h"],
                                  cam["T"], cam["lo"], cam["hi"]),
                prm=S.make_ogm_params(**MAP_PRM), L=i["L"],
                occ=torch.empty(i["L"].shape, dtype=torch.uint8, device=DEV) if case["occ"] else None,
                work=torch.empty(need // 4, device=DEV),
                stream=torch.cuda.current_stream().cuda_stream)


def _run_map(s):
    i = s["inputs"]
    s["planner"].ogm_update(depth=i["depth"], cam=s["cam"], log_odds=s["L"], origin=i["origin"],
                            voxel=i["voxel"], prm=s["prm"], work=s["work"],
                            q=i["q"] if s["case"]["mask"] else None, occ_out=s["occ"],
                            stream=s["stream"])
    return dict(L=s["L"], occ=s["occ"]) if s["occ"] is not None else dict(L=s["L"])


def _serve_inputs(case, seed):
    """Controllers of the serving mix: K, H, map size and clutter differ from one to the next."""
    rng = np.random.default_rng([int(seed), 4])
    robot = _Robot(rng, 2)
    mix = np.random.default_rng(case["n"])  # the fleet is the case's, its maps are the seed's
    ctl = []
    for k in range(case["n"]):
        n, vox = int(mix.integers(64, 161)), float(np.float32(mix.uniform(case["voxel_lo"], case["voxel_hi"])))
        K, H = int(mix.choice([256, 1024, 2048, 4096])), int(mix.choice([16, 32, 64]))
        prims = _scene(rng, n, n, n, vox, int(mix.integers(10, 61)))
        ctl.append(dict(robot=robot, n=n, voxel=vox, K=K, H=H, prims=prims,
                        origin=_origin(n, n, n, vox), dt=float(np.float32(0.02)),
                        q0=_f32(np.array(READY) + rng.uniform(-0.3, 0.3, size=NDOF)),
                        qd0=_f32(np.zeros(NDOF)), T_goal=_pose(rng),
                        seed=int(rng.integers(1 << 62))))
    return robot, ctl


def _prepare_serve(case, seed):
    robot, ctl = _serve_inputs(case, seed)
    service = _Service(_Ctx(robot), 512 << 20, 64)
    s = dict(case=case, service=service, grids=[], reqs=[],
             stream=torch.cuda.current_stream().cuda_stream)
    s["U"] = torch.empty(sum(c["H"] for c in ctl), NDOF, device=DEV)
    s["costs"] = torch.empty(sum(c["K"] for c in ctl), device=DEV)
    h = k = 0
    for tag, c in enumerate(ctl):
        g = _sdf(c["prims"], c["n"], c["n"], c["n"], c["voxel"])
        s["grids"].append(g)
        st, cid = S.smpc_server_add_controller(service.h, S.controller_desc(
            g, c["origin"], c["voxel"], c["K"], c["H"], c["dt"], LAMBDA, WEIGHTS, SIGMA,
            U_star_out=s["U"][h:h + c["H"]], costs_out=s["costs"][k:k + c["K"]]))
        _ok(st)
        s["reqs"].append(S.request(tag, cid, c["q0"], c["qd0"], c["T_goal"], c["seed"]))
        h, k = h + c["H"], k + c["K"]
    return s


def _run_serve(s):
    h, stream = s["service"].h, s["stream"]
    for r in s["reqs"]:
        _ok(S.smpc_server_submit(h, r))
    n = len(s["reqs"])
    u0, stats, left = np.empty((n, NDOF), np.float32), np.empty((n, 3), np.float32), n
    while left:
        st, _ = S.smpc_server_pump(h, stream)
        _ok(st)
        st, done = S.smpc_server_poll(h)
        _ok(st)
        for c in done:
            u0[c.tag] = c.u0[:]
            stats[c.tag] = c.S_min, c.Z, c.ess
        left -= len(done)
    return dict(u0=u0, stats=stats, U=s["U"], costs=s["costs"])


def prepare(case, seed):
    return {"step": _prepare_step, "field": _prepare_field, "map": _prepare_map,
            "serve": _prepare_serve}[case["kind"]](case, int(seed))


def run(state):
    kind = "serve" if "service" in state else state["case"]["kind"]
    return {"step": _run_step, "field": _run_field, "map": _run_map,
            "serve": _run_serve}[kind](state)


# --- work --------------------------------------------------------------------------

FLOP_PER_ROLLOUT_STEP = 4300.0  # FK, 28 sphere centres and lookups, 240 pairs, pose, limits


def work(case):
    if case["kind"] == "step":
        K, H, vox = case["K"], case["H"], case["nx"] * case["ny"] * case["nz"]
        elem = 2 if case["grid"] == "f16" else 4
        grid = vox * elem if case["bounds"] in ("period", "next") else min(vox * elem, K * H * 28 * 8 * elem)
        noise = K * H * NDOF * 4 if case["noise"] == "buffer" else 0
        return {"bytes": noise + grid + 2 * H * NDOF * 4 + 2 * K * 4,
                "flops": FLOP_PER_ROLLOUT_STEP * K * H}
    if case["kind"] == "field":
        vox = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": vox * (1 + 4 + (8 if case["d2"] else 0)), "flops": 20.0 * vox}
    if case["kind"] == "map":
        vox, pix = case["nx"] * case["ny"] * case["nz"], case["width"] * case["height"]
        return {"bytes": vox * (8 + (1 if case["occ"] else 0)) + pix * 4, "flops": 30.0 * vox}
    mix, by, fl = np.random.default_rng(case["n"]), 0.0, 0.0
    for _ in range(case["n"]):
        n = int(mix.integers(64, 161))
        mix.uniform(case["voxel_lo"], case["voxel_hi"])
        K, H = int(mix.choice([256, 1024, 2048, 4096])), int(mix.choice([16, 32, 64]))
        mix.integers(10, 61)
        by += 4.0 * min(n ** 3, K * H * 28 * 8) + K * 4 + H * NDOF * 8
        fl += FLOP_PER_ROLLOUT_STEP * K * H
    return {"bytes": by, "flops": fl}


# --- 64-bit values -------------------------------------------------------------------

def _t64(x):
    return torch.as_tensor(np.asarray(x, np.float64), device=DEV)


def _frames64(robot, q):
    """Rotation columns and origins of the seven link frames for joint values q (n, 7)."""
    n = q.shape[0]
    X = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
    X[:, 0] = 1.0
    Y, Z, t = X.roll(1, 1), X.roll(2, 1), torch.zeros_like(X)
    out = []
    for j in range(NDOF):
        ca, sa = math.cos(robot.alpha[j]), math.sin(robot.alpha[j])
        t = t + float(np.float32(robot.a[j])) * X
        Y, Z = ca * Y + sa * Z, ca * Z - sa * Y
        c, s = q[:, j:j + 1].cos(), q[:, j:j + 1].sin()
        X, Y = c * X + s * Y, c * Y - s * X
        t = t + float(np.float32(robot.d[j])) * Z
        out.append((X, Y, Z, t))
    return out


def _centres64(robot, frames):
    out = []
    for i in range(len(robot.sphere_link)):
        X, Y, Z, t = frames[int(robot.sphere_link[i]) - 1]
        c = _f32(robot.sphere_center[i]).astype(np.float64)
        out.append(X * c[0] + Y * c[1] + Z * c[2] + t)
    return out


def _phi64(grid, origin, voxel, p):
    nz, ny, nx = grid.shape
    u = (p - _t64(origin)) / voxel - 0.5
    u = torch.minimum(u.clamp(min=0.0), _t64([nx - 1, ny - 1, nz - 1]))
    i = torch.minimum(u.floor(), _t64([nx - 2, ny - 2, nz - 2])).long()
    f = u - i
    flat, base = grid.reshape(-1), (i[:, 2] * ny + i[:, 1]) * nx + i[:, 0]
    v = 0.0
    for b in range(8):
        bx, by, bz = b & 1, b >> 1 & 1, b >> 2
        w = (f[:, 0] if bx else 1 - f[:, 0]) * (f[:, 1] if by else 1 - f[:, 1])
        w = w * (f[:, 2] if bz else 1 - f[:, 2])
        v = v + w * flat[base + (bz * ny + by) * nx + bx].double()
    return v


def _pose64(frame, T_goal, wt, wr):
    X, Y, Z, t = frame
    G = _t64(T_goal)
    R = torch.stack([X, Y, Z], -1)
    D = G[:3, :3].T @ R
    e = (t - G[:3, 3]) @ G[:3, :3]
    vee = torch.stack([D[:, 2, 1] - D[:, 1, 2], D[:, 0, 2] - D[:, 2, 0], D[:, 1, 0] - D[:, 0, 1]], -1)
    theta = torch.atan2(0.5 * vee.norm(dim=-1), 0.5 * (D.diagonal(dim1=1, dim2=2).sum(-1) - 1))
    x = 0.5 * theta
    gain = (x * x - x.sin() ** 2) / (2 * x.sin() ** 4)  # |V^-1 t|^2 = |t|^2 + gain t'(I - R)t
    gain = torch.where(theta < 1e-3, torch.full_like(gain, 1 / 6), gain)
    lost = (e * e).sum(-1) - (e * (D @ e[:, :, None])[:, :, 0]).sum(-1)
    return 0.5 * (wt * ((e * e).sum(-1) + gain * lost.clamp(min=0.0)) + wr * theta * theta)


def _over64(x, lo, hi):
    m = WEIGHTS["limit_margin_frac"] * (np.asarray(hi) - np.asarray(lo))
    lo, hi = _t64(np.asarray(lo) + m), _t64(np.asarray(hi) - m)
    return ((x - hi).clamp(min=0.0) + (x - lo).clamp(max=0.0)).square().sum(-1)


def _state64(i, grid, q, qd):
    """Running cost of states (n, 7) without the control terms."""
    w, rob = WEIGHTS, i["robot"]
    fr = _frames64(rob, q)
    c = _pose64(fr[-1], i["T_goal"], w["w_pose_t"], w["w_pose_r"])
    c = c + w["w_q"] * _over64(q, rob.q_min, rob.q_max) + w["w_qd"] * _over64(qd, rob.qd_min, rob.qd_max)
    p, r = _centres64(rob, fr), rob.sphere_radius
    for k in range(len(p)):
        h = w["d_act"] - (_phi64(grid, i["origin"], i["voxel"], p[k]) - float(r[k]))
        c = c + w["w_env"] * h.clamp(min=0.0).square()
    own = torch.zeros_like(c)
    for a, b in rob.pairs:
        h = float(r[a] + r[b]) - (p[a] - p[b]).norm(dim=-1)
        own += h.clamp(min=0.0).square()
    return c + w["w_self"] * own


def _philox64(seed, K, H):
    """Standard normals of the library's documented generator (Philox4x32-10, Box-Muller)."""
    m32 = np.uint64(0xFFFFFFFF)
    z = []
    for b in (0, 1):
        n = np.arange(K * H, dtype=np.uint64) * np.uint64(2) + np.uint64(b)
        c = [n & m32, n >> np.uint64(32), np.zeros_like(n), np.zeros_like(n)]
        k = [seed & 0xFFFFFFFF, seed >> 32]
        for _ in range(10):
            x, y = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
            c = [(y >> np.uint64(32)) ^ c[1] ^ np.uint64(k[0]), y & m32,
                 (x >> np.uint64(32)) ^ c[3] ^ np.uint64(k[1]), x & m32]
            k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
        u = [((v >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0 ** -23 for v in c]
        for a, d in ((0, 1), (2, 3)):
            r, t = np.sqrt(-2 * np.log(u[a])), 2 * np.pi * u[d]
            z += [r * np.cos(t), r * np.sin(t)]
    return torch.from_numpy(np.stack(z[:NDOF], -1).reshape(K, H, NDOF)).to(DEV)


def _plan64(i, grid, Ubar, eps):
    """One plan step: costs, weights, U*, statistics."""
    K, H, dt, w, rob = i["K"], i["H"], i["dt"], WEIGHTS, i["robot"]
    q0, qd0 = _t64(i["q0"]), _t64(i["qd0"])
    S_ = torch.empty(K, dtype=torch.float64, device=DEV)
    c0 = _state64(i, grid, q0[None], qd0[None])[0]
    step = max(1, (1 << 20) // H)
    for lo in range(0, K, step):
        u = Ubar + eps[lo:lo + step]
        qd = qd0 + (u * dt).cumsum(1)
        q = q0 + (qd * dt).cumsum(1)
        c = (w["w_smooth"] * u.square().sum(-1) + w["w_qdd"] * _over64(u, rob.qdd_min, rob.qdd_max)).sum(1)
        if H > 1:
            run_ = _state64(i, grid, q[:, :-1].reshape(-1, NDOF), qd[:, :-1].reshape(-1, NDOF))
            c = c + run_.reshape(-1, H - 1).sum(1)
        c = c + _pose64(_frames64(rob, q[:, -1])[-1], i["T_goal"], w["w_term_t"], w["w_term_r"])
        S_[lo:lo + step] = c + c0
    e = (-(S_ - S_.min()) / LAMBDA).exp()
    p = e / e.sum()
    U = Ubar + (p[None] @ eps.reshape(K, -1)).reshape(H, NDOF)
    return S_, p, U, torch.stack([S_.min(), e.sum(), 1 / p.square().sum(), torch.zeros_like(c0)])


def _exact_step(case, seed):
    i = _step_inputs(case, seed)
    grid = i["grids"][0]
    if case["grid"] == "f16":
        grid = grid.clamp(-1.0, 1.0).half()
    if case["noise"] == "buffer":
        eps = i["noise"].double()
    else:
        eps = SIGMA * _philox64(i["seed"], case["K"], case["H"])
    costs, weights, U, stats = _plan64(i, grid, i["U"].double(), eps)
    out = dict(U=U, costs=costs, weights=weights, stats=stats)
    if case["receding"]:
        qd = _t64(i["qd0"]) + U[0] * i["dt"]
        out.update(U=torch.cat([U[1:], torch.zeros_like(U[:1])]), u0=U[0],
                   state=torch.cat([_t64(i["q0"]) + qd * i["dt"], qd]))
    if case["bounds"] in ("period", "next"):
        out["bounds"] = None
    return out


def _squared64(src):
    """Squared index distance to the nearest set voxel (int32)."""
    nz, ny, nx = src.shape
    far = 1 << 28
    d = torch.where(src, 0, far).to(torch.int32)
    for ax, n in ((2, nx), (1, ny), (0, nz)):
        best = d.clone()
        for k in range(1, n):
            a, b = d.narrow(ax, 0, n - k) + k * k, d.narrow(ax, k, n - k) + k * k
            lo, hi = best.narrow(ax, k, n - k), best.narrow(ax, 0, n - k)
            torch.minimum(lo, a, out=lo)
            torch.minimum(hi, b, out=hi)
        d = best
    return torch.where(d >= far, nx * nx + ny * ny + nz * nz, d)


def _exact_field(case, seed):
    occ, vox = _field_inputs(case, seed)
    out, inn = _squared64(occ != 0), _squared64(occ == 0)
    phi = vox * (out.double().sqrt() - inn.double().sqrt())
    return dict(phi=phi, d2=torch.stack([out, inn])) if case["d2"] else dict(phi=phi)


def _exact_map(case, seed):
    i = _map_inputs(case, seed)
    cam, prm, vox = i["cam"], MAP_PRM, i["voxel"]
    T, o = _t64(cam["T"]), i["origin"].astype(np.float64)
    depth, f = i["depth"].double(), cam["f"]
    if case["mask"]:
        p = _centres64(i["robot"], _frames64(i["robot"], _t64(i["q"])[None]))
        balls = [(x[0], float(r) + prm["robot_pad"]) for x, r in zip(p, i["robot"].sphere_radius)]
        u = (torch.arange(cam["w"], device=DEV, dtype=torch.float64) + 0.5 - cam["cx"]) / f
        v = (torch.arange(cam["h"], device=DEV, dtype=torch.float64) + 0.5 - cam["cy"]) / f
        at = (u[None, :, None] * T[:3, 0] + v[:, None, None] * T[:3, 1] + T[:3, 2]) * depth[..., None] + T[:3, 3]
        for c, r in balls:
            depth = torch.where((at - c).square().sum(-1) <= r * r, torch.zeros_like(depth), depth)
    ax = [(torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) * vox + o[k]
          for k, n in enumerate((case["nx"], case["ny"], case["nz"]))]
    p = torch.stack(torch.broadcast_tensors(ax[0][None, None], ax[1][None, :, None], ax[2][:, None, None]), -1)
    c = (p - T[:3, 3]) @ T[:3, :3]
    z = c[..., 2]
    zs = torch.where(z > 0, z, torch.ones_like(z))
    u, v = (f * c[..., 0] / zs + cam["cx"]).floor(), (f * c[..., 1] / zs + cam["cy"]).floor()
    seen = (z > 0) & (u >= 0) & (u < cam["w"]) & (v >= 0) & (v < cam["h"])
    at = v.clamp(0, cam["h"] - 1).long() * cam["w"] + u.clamp(0, cam["w"] - 1).long()
    d = torch.where(seen, depth.reshape(-1)[at], torch.zeros_like(z))
    e, L = z - d, i["L"].double()
    hit, free = (d > 0) & (e.abs() <= prm["tol"]), (d > 0) & (e < -prm["tol"])
    new = (L + torch.where(hit, prm["l_hit"], prm["l_miss"])).clamp(prm["l_min"], prm["l_max"])
    L = torch.where(hit | free, new, L)
    if case["mask"]:
        for b, r in balls:
            L = torch.where((p - b).square().sum(-1) <= r * r, torch.full_like(L, prm["l_min"]), L)
    return dict(L=L, occ=(L > prm["l_occ"]).to(torch.uint8)) if case["occ"] else dict(L=L)


def _exact_serve(case, seed):
    _, ctl = _serve_inputs(case, seed)
    u0, stats, U, costs = [], [], [], []
    for c in ctl:
        grid = _sdf(c["prims"], c["n"], c["n"], c["n"], c["voxel"])
        eps = SIGMA * _philox64(c["seed"], c["K"], c["H"])
        S_, _, Us, st = _plan64(c, grid, torch.zeros(c["H"], NDOF, dtype=torch.float64, device=DEV), eps)
        u0.append(Us[0])
        stats.append(st[:3])
        U.append(Us)
        costs.append(S_)
    return dict(u0=torch.stack(u0).cpu().numpy(), stats=torch.stack(stats).cpu().numpy(),
                U=torch.cat(U), costs=torch.cat(costs))


def exact(case, seed):
    return {"step": _exact_step, "field": _exact_field, "map": _exact_map,
            "serve": _exact_serve}[case["kind"]](case, int(seed))
