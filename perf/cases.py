"""The calls a program makes of this library, as measurable cases.

Every case goes through the package's public entry points on seeded synthetic
scenes (`workloads`: boxes on a ground, or a displaced terrain with spheres)
and G-buffers of them; the camera pose and the sample seed follow the seed.

  listed()            the named cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) scene, acceleration structure, G-buffer and buffers
  run(state)          one pass; returns its outputs whole
  work(case)          bytes and operations a pass cannot do without
  exact(case, seed)   the outputs in 64 bits (boxes scenes, uniform light)
"""
import functools
import math

import numpy as np
import torch

import paper_2607_23122_amd as ocr
import workloads as w

# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------


def _frame(name=None, **kw):
    """A single-view pass: trace, then one estimator."""
    c = dict(kind="frame", scene="terrain", cells=512, spheres=2000, width=1920, height=1080, mode="ao", ao_radius=2.0,
             pattern="window", r=3, group=8, estimator="biased", lights=1, pdf=0, samples=1)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the plain CPU-sized frame of the repository (770 triangles, 5x5
        # window): a few microseconds of GPU work, so launches and the host
        # side of a call count
        _frame("ao_256_boxes", scene="boxes", cells=0, spheres=64, width=256, height=256, ao_radius=1.0, r=2),
        # a small frame of odd size whose tiles, runs and list groups all end
        # in partial groups; unbiased, so every launch of the path is made
        _frame("shadow_333x197_unbiased", scene="boxes", cells=0, spheres=64, width=333, height=197, mode="shadow", r=2,
               estimator="unbiased"),
        # interactive AO at 1080p: one sample, biased 7x7 reuse
        _frame("ao_1080p_biased"),
        # the same with first-hit validation: the headline frame step
        _frame("ao_1080p_unbiased", estimator="unbiased"),
        # soft shadows of one rectangular light at 1080p
        _frame("shadow_1080p_biased", mode="shadow"),
        _frame("shadow_1080p_unbiased", mode="shadow", estimator="unbiased"),
        # the paper's own reuse pattern, fixed groups of eight, with validation
        _frame("ao_1080p_group8", pattern="group", estimator="unbiased"),
        # direct illumination, light sampled by the receiver-dependent density
        _frame("di_900p_bilinear", mode="di", pdf=1, width=1600, height=900),
        # shadows of two lights, 5x5 window, validated
        _frame("shadow2_720p_unbiased", mode="shadow", lights=2, r=2, estimator="unbiased", width=1280, height=720),
        # sixteen views of uneven size over four scenes in one plan launch
        dict(name="plan_16_views", kind="plan", views=16),
        # a burst of mixed requests to the server, drained
        dict(name="served_burst_24", kind="served", requests=24, slots=8),
        # the largest frame: 1440p over 2M triangles, two accumulated samples
        _frame("ao_1440p_render2", cells=768, spheres=2560, width=2560, height=1440, estimator="unbiased", samples=2),
    ]


def draw(rng):
    big = 2.0 * 2560 * 1440 * 169  # pairs of the largest listed case
    while True:
        width = round(math.exp(rng.uniform(math.log(40), math.log(2561))))
        height = max(17, round(width * rng.uniform(0.45, 1.1)))
        scene = rng.choice(["boxes", "terrain", "terrain"])
        mode = rng.choice(["ao", "ao", "ao", "shadow", "shadow", "shadow_sa", "di"])
        pattern = rng.choice(["window", "window", "window", "group"])
        r = rng.choice([1, 2, 2, 3, 3, 3, 4])
        c = _frame(scene=scene, width=width, height=height, mode=mode, pattern=pattern, r=r,
                   group=rng.choice([2, 4, 8]), estimator=rng.choice(["none", "biased", "biased", "unbiased", "unbiased"]),
                   samples=1)
        if scene == "boxes":
            c.update(cells=0, spheres=rng.randint(8, 96), ao_radius=rng.choice([0.5, 1.0, 1.0]))
        else:
            cells = rng.randint(96, 768)
            c.update(cells=cells, spheres=round(cells * cells * 2000 / 512 ** 2), ao_radius=rng.choice([1.0, 2.0, 2.0]))
        if mode == "shadow":
            c["lights"] = rng.choice([1, 1, 2])
        if mode != "ao" and c["lights"] == 1:
            c["pdf"] = rng.choice([0, 0, 1])
        if width * height * (4 * r + 1) ** 2 <= big and width * height <= 2560 * 1440:
            return c


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------
@functools.lru_cache(maxsize=12)
def _mesh(scene, cells, spheres):
    return w.boxes_scene(1, spheres) if scene == "boxes" else w.terrain_scene(2 + cells % 7, cells, spheres)


def _pose(seed):
    return (seed * 0.6180339887498949) % 1.0


def _inputs(case, seed):
    mesh = _mesh(case["scene"], case["cells"], case["spheres"])
    if case["scene"] == "boxes":
        cam = w.orbit_camera(_pose(seed), 1, case["width"], case["height"], (0.0, 12.0, -8.0), (0.0, 0.0, 0.0))
        lights = [w.RectLight(np.array([1.0, 7.0, -1.0], np.float32), np.array([1.0, 0.0, 0.0], np.float32),
                              np.array([0.0, 0.0, 1.0], np.float32)),
                  w.RectLight(np.array([-6.0, 5.0, 3.0], np.float32), np.array([0.0, 0.6, 0.8], np.float32),
                              np.array([0.0, -0.8, 0.6], np.float32))]
        # the second light's emitting side faces the middle of the scene
        e = lights[1]
        if np.dot(np.cross(e.edge_u, e.edge_v), -e.center) < 0:
            e.edge_u, e.edge_v = e.edge_v, e.edge_u
    else:
        cam = w.orbit_camera(_pose(seed), 1, case["width"], case["height"])
        lights = w.two_lights()
    gb = w.render_gbuffer(mesh, cam)
    if case["mode"] == "ao":
        light = None
    elif case["lights"] == 2:
        light = lights
    else:
        light = lights[0]
        light.pdf = case["pdf"]
    return mesh, gb, light


def _params(case):
    return ocr.reuse_params(case["pattern"], case["r"], case["group"], case["estimator"])


def prepare(case, seed):
    if case["kind"] == "plan":
        return _prepare_plan(case, seed)
    if case["kind"] == "served":
        return _prepare_served(case, seed)
    mesh, gb, light = _inputs(case, seed)
    p = _params(case)
    g = ocr.DeviceGBuffer.from_host(gb)
    need = ocr.workspace_bytes(g.width, g.height, p)
    return dict(case=case, seed=seed, light=light, gbuf=g, params=p, bvh=ocr.build_bvh(mesh.V, mesh.F),
                occ=ocr.Occluders.empty(g.height, g.width),
                ws=torch.zeros(need, dtype=torch.uint8, device="cuda") if need else None,
                out=torch.empty((g.height, g.width), dtype=torch.float32, device="cuda"))


def _prepare_plan(case, seed):
    bvhs = [ocr.build_bvh(s.V, s.F) for s in (_mesh("terrain", c["cells"], c["spheres"]) for c in w.BATCH_SCENES)]
    light, views, outs, keep = w.terrain_light(), [], [], []
    for v, (i, cam, mode) in enumerate(w.batch_views()[:case["views"]]):
        c = w.BATCH_SCENES[i]
        cam = w.orbit_camera(v + 16 * _pose(seed), 16, cam.width, cam.height)
        g = ocr.DeviceGBuffer.from_host(w.render_gbuffer(_mesh("terrain", c["cells"], c["spheres"]), cam))
        out = torch.empty((g.height, g.width), dtype=torch.float32, device="cuda")
        views.append(ocr.view_desc(bvhs[i], g, out, mode, 2.0, light if mode == "shadow" else None, seed, v,
                                   ocr.reuse_params("window", 3, 8, "biased")))
        outs.append(out)
        keep.append(g)
    # the knobs are given: an autotuned choice varies from run to run
    plan = ocr.Plan(views, ocr.plan_tuning((8, 8), "block8"), keep=(bvhs, keep))
    return dict(case=case, plan=plan, outs=outs)


def _prepare_served(case, seed):
    rng = np.random.Generator(np.random.PCG64(7))  # the mix; poses and samples follow the seed
    light, srv, outs, reqs = w.terrain_light(), ocr.Server(2 << 30, case["slots"]), [], []
    pools, sizes = [], [(1280, 720), (1920, 1080), (2560, 1440)]
    for c in w.BATCH_SCENES[:3]:
        mesh = _mesh("terrain", c["cells"], c["spheres"])
        pool = [ocr.DeviceGBuffer.from_host(w.render_gbuffer(mesh, w.orbit_camera(k / 3 + _pose(seed), 1, *s)))
                for k, s in enumerate(sizes)]
        pools.append((srv.add_scene(ocr.build_bvh(mesh.V, mesh.F), pool), pool))
    # one request of each third is validated; sizes, scenes and effects mixed
    for k in range(case["requests"]):
        sid, pool = pools[int(rng.integers(len(pools)))]
        view = int(rng.integers(len(pool)))
        mode = "ao" if rng.integers(2) == 0 else "shadow"
        out = torch.empty((pool[view].height, pool[view].width), dtype=torch.float32, device="cuda")
        reqs.append(ocr.request(sid, view, mode, 2.0, light, seed + k, 0, ocr.reuse_params(
            "window", 3, 8, "unbiased" if k % 3 == 0 else "biased"), out))
        outs.append(out)
    return dict(case=case, server=srv, reqs=reqs, outs=outs)


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] == "plan":
        state["plan"].launch()
        return state["outs"]
    if case["kind"] == "served":
        srv = state["server"]
        for r in state["reqs"]:
            srv.submit(r)
        srv.drain()
        srv.poll()
        return state["outs"]
    bvh, g, occ, p, light = (state[k] for k in ("bvh", "gbuf", "occ", "params", "light"))
    mode = case["mode"]
    if case["samples"] > 1:
        return {"image": ocr.render(bvh, g, mode, case["ao_radius"], light, state["seed"], case["samples"], 0, p)}
    ocr.trace_occluders(bvh, g, "ao" if mode == "ao" else "shadow", case["ao_radius"], light, state["seed"], 0, occ)
    if mode == "ao":
        ocr.reuse_ao(bvh, g, occ, case["ao_radius"], p, state["out"], state["ws"])
    elif mode == "shadow":
        ocr.reuse_shadow(bvh, g, occ, light, p, state["out"], state["ws"])
    elif mode == "shadow_sa":
        ocr.reuse_shadow_solid_angle(bvh, g, occ, light, p, state["out"], state["ws"])
    else:
        ocr.reuse_direct_illumination(bvh, g, occ, light, p, 100.0, 0.8, state["out"], state["ws"])
    return {"hit": occ.hit, "dz": occ.dz, "nz": occ.nz, "image": state["out"]}


# --------------------------------------------------------------------------
# Work
# --------------------------------------------------------------------------
# Useful work per unit on the terrain frames (counted by the library's
# accounting entry points): box and triangle tests of 26 and 59 FP32
# operations a ray or a validation segment needs, segments and hits per pixel,
# and the operations of one pair density.
_RAY = {"ao": 49 * 26 + 2.4 * 59, "shadow": 69 * 26 + 4.1 * 59}
_SEGMENT = 64 * 26 + 5 * 59
_HIT = {"ao": 0.11, "shadow": 0.23}
_PAIR_SHARE = {"ao": 0.7, "shadow": 0.008}
_DENSITY = {"ao": 28, "shadow": 42}


def _pixel_work(mode, estimator, pattern, r, group):
    """(bytes, operations) of a pixel: G-buffer 28 B read once, a record of
    4 B and 24 B more for a hit written, an estimate of 4 B written."""
    m = "ao" if mode == "ao" else "shadow"
    f = _RAY[m]
    if estimator != "none":
        n = (4 * r + 1) ** 2 if pattern == "window" else group
        f += _HIT[m] * n * _DENSITY[m]
        if estimator == "unbiased":
            f += _HIT[m] * n * (_PAIR_SHARE[m] * _SEGMENT + _DENSITY[m])
    return 28 + 4 + 24 * _HIT[m] + 4, f


def work(case):
    total = [0.0, 0.0]

    def add(px, *args):
        b, f = _pixel_work(*args)
        total[0] += b * px
        total[1] += f * px

    if case["kind"] == "plan":
        for _, cam, mode in w.batch_views()[:case["views"]]:
            add(cam.width * cam.height, mode, "biased", "window", 3, 8)
    elif case["kind"] == "served":
        px = (1280 * 720 + 1920 * 1080 + 2560 * 1440) / 3.0
        for k in range(case["requests"]):
            for mode in ("ao", "shadow"):
                add(px / 2, mode, "unbiased" if k % 3 == 0 else "biased", "window", 3, 8)
    else:
        add(case["width"] * case["height"] * case["samples"], case["mode"], case["estimator"], case["pattern"],
            case["r"], case["group"])
    return {"bytes": total[0], "flops": total[1]}


# --------------------------------------------------------------------------
# The outputs in 64 bits.  The samples are a specification in 32 bits (hash,
# operation order), followed here in numpy; tracing is brute force over the
# triangles and the estimators follow the paper's equations in torch, float64.
# --------------------------------------------------------------------------
_F = np.float32


def _fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(_F)


def _pcg4d(px, py, s, seed):
    with np.errstate(over="ignore"):
        v = [np.asarray(x, np.uint32) * np.uint32(1664525) + np.uint32(1013904223) for x in (px, py, s, seed)]

        def mix(v):
            v[0] = v[0] + v[1] * v[3]
            v[1] = v[1] + v[2] * v[0]
            v[2] = v[2] + v[0] * v[1]
            v[3] = v[3] + v[1] * v[2]
            return v

        v = mix(v)
        v = [x ^ (x >> np.uint32(16)) for x in v]
        return mix(v)


def _unit(h):
    return (h >> np.uint32(8)).astype(_F) * _F(2.0 ** -24)


def _directions(gb, case, seed, light):
    """(o, d, traced): FP32 offset points and ray vectors of every pixel."""
    H, W = gb.prim.shape
    py, px = np.meshgrid(np.arange(H, dtype=np.uint32), np.arange(W, dtype=np.uint32), indexing="ij")
    zero = np.zeros_like(px)
    sd = np.uint32((seed & 0xFFFFFFFF) ^ (seed >> 32))
    x, n = gb.pos, gb.nrm
    eps = (_F(1) + np.abs(x).max(-1)) * _F(2.0 ** -16)
    o = _fma(eps[..., None], n, x)
    if case["mode"] == "ao":
        al, be, q = (np.zeros((H, W), _F) for _ in range(3))
        done = np.zeros((H, W), bool)
        for a in range(16):
            with np.errstate(over="ignore"):
                h = _pcg4d(px, py, zero, zero + sd + np.uint32((a * 0x9E3779B9) & 0xFFFFFFFF))
            ta, tb = _F(2) * _unit(h[0]) - _F(1), _F(2) * _unit(h[1]) - _F(1)
            tq = _fma(tb, tb, ta * ta)
            take = ~done & (tq < 1)
            al, be, q = np.where(take, ta, al), np.where(take, tb, be), np.where(take, tq, q)
            done |= take
        g = np.sqrt(_F(1) - q)
        sign = np.copysign(_F(1), n[..., 2])
        a = _F(-1) / (sign + n[..., 2])
        b = n[..., 0] * n[..., 1] * a
        t = np.stack([_F(1) + sign * n[..., 0] * n[..., 0] * a, sign * b, -sign * n[..., 0]], -1)
        u = np.stack([b, sign + n[..., 1] * n[..., 1] * a, -n[..., 1]], -1)
        d = (al[..., None] * t + be[..., None] * u) + g[..., None] * n
        return o, d.astype(_F), gb.valid
    h = _pcg4d(px, py, zero, zero + sd)
    a, b = _unit(h[0]) - _F(0.5), _unit(h[1]) - _F(0.5)
    y = _fma(b[..., None], light.edge_v, _fma(a[..., None], light.edge_u, light.center))
    d = y - o
    nl = np.cross(light.edge_u.astype(np.float64), light.edge_v.astype(np.float64))
    front = (n.astype(np.float64) * d).sum(-1) > 0
    lit = ((o.astype(np.float64) - light.center) * nl).sum(-1) > 0
    return o, d, gb.valid & front & lit


def _triangles(mesh, dev):
    T = torch.from_numpy(mesh.V[mesh.F.astype(np.int64)].astype(np.float64)).to(dev)
    a, e1, e2 = T[:, 0], T[:, 1] - T[:, 0], T[:, 2] - T[:, 0]
    return a, e1, e2, torch.linalg.cross(e1, e2)


def _distances(tri, o, d):
    """Ray parameters [rays, triangles] of the crossings, inf where there is none."""
    a, e1, e2, n = tri
    det = -(d @ n.T)
    s = o[:, None] - a[None]
    t = (s * n[None]).sum(-1) / det
    c = torch.linalg.cross(s, d[:, None].expand_as(s))
    u = (c * e2[None]).sum(-1) / det
    v = -(c * e1[None]).sum(-1) / det
    ok = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t > 0)
    return torch.where(ok, t, torch.full_like(t, math.inf))


def _closest(tri, o, d, prim, tmax):
    ids = torch.full((o.shape[0],), -1, dtype=torch.int64, device=o.device)
    ts = torch.zeros(o.shape[0], dtype=torch.float64, device=o.device)
    step = max(1, 20_000_000 // tri[0].shape[0])
    for i in range(0, o.shape[0], step):
        t = _distances(tri, o[i:i + step], d[i:i + step])
        t.scatter_(1, prim[i:i + step, None], math.inf)
        best, at = t.min(1)
        hit = best <= tmax
        ids[i:i + step] = torch.where(hit, at, -torch.ones_like(at))
        ts[i:i + step] = torch.where(hit, best, torch.zeros_like(best))
    return ids, ts


def _blocked(tri, o, d, skip0, skip1):
    out = torch.zeros(o.shape[0], dtype=torch.bool, device=o.device)
    step = max(1, 20_000_000 // tri[0].shape[0])
    for i in range(0, o.shape[0], step):
        t = _distances(tri, o[i:i + step], d[i:i + step])
        t.scatter_(1, skip0[i:i + step, None], math.inf)
        t.scatter_(1, skip1[i:i + step, None], math.inf)
        out[i:i + step] = (t < 1 - 1e-4).any(1)
    return out


def _front_fraction(o, n, light):
    """Share of the rectangle in front of the tangent plane of (o, n): the
    unit square clipped by a half-plane, by the shoelace formula."""
    c, eu, ev = (torch.from_numpy(np.asarray(v, np.float64)).to(o.device) for v in (light.center, light.edge_u, light.edge_v))
    f0, fu, fv = (n * (c - o)).sum(-1), n @ eu, n @ ev
    corner = [(-0.5, -0.5), (0.5, -0.5), (0.5, 0.5), (-0.5, 0.5)]
    area = torch.zeros_like(f0)
    # twice the area as a sum of cross products about the first corner: each
    # edge's inside part, plus the chord joining the two crossing points
    cross_in, cross_out = [torch.zeros_like(f0) for _ in range(2)], [torch.zeros_like(f0) for _ in range(2)]
    cut = torch.zeros_like(f0, dtype=torch.bool)
    for (ax, ay), (bx, by) in zip(corner, corner[1:] + corner[:1]):
        fa, fb = f0 + ax * fu + ay * fv, f0 + bx * fu + by * fv
        t = torch.where((fa > 0) != (fb > 0), fa / (fa - fb), torch.zeros_like(fa))
        mx, my = ax + t * (bx - ax), ay + t * (by - ay)
        sx, sy = torch.where(fa > 0, torch.full_like(fa, ax), mx), torch.where(fa > 0, torch.full_like(fa, ay), my)
        ex, ey = torch.where(fb > 0, torch.full_like(fa, bx), mx), torch.where(fb > 0, torch.full_like(fa, by), my)
        some = (fa > 0) | (fb > 0)
        area += torch.where(some, sx * ey - ex * sy, torch.zeros_like(fa))
        leave, enter = (fa > 0) & ~(fb > 0), (fb > 0) & ~(fa > 0)
        cross_out = [torch.where(leave, v, k) for v, k in zip((mx, my), cross_out)]
        cross_in = [torch.where(enter, v, k) for v, k in zip((mx, my), cross_in)]
        cut |= leave
    area += torch.where(cut, cross_out[0] * cross_in[1] - cross_in[0] * cross_out[1], torch.zeros_like(area))
    nl = torch.linalg.cross(eu, ev)
    return torch.where(((o - c) @ nl) > 0, 0.5 * area.abs(), torch.zeros_like(area))


def _shifted(v, dy, dx, fill):
    """v at (y + dy, x + dx), `fill` outside the image."""
    H, W = v.shape[:2]
    out = torch.full_like(v, fill)
    y0, y1, x0, x1 = max(0, -dy), min(H, H - dy), max(0, -dx), min(W, W - dx)
    if y1 > y0 and x1 > x0:
        out[y0:y1, x0:x1] = v[y0 + dy:y1 + dy, x0 + dx:x1 + dx]
    return out


def exact(case, seed):
    if case["kind"] != "frame" or case["scene"] != "boxes" or case["samples"] > 1 or case["lights"] > 1 or \
            case["pdf"] or case["mode"] not in ("ao", "shadow") or case["width"] * case["height"] > 800_000:
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    mesh, gb, light = _inputs(case, seed)
    H, W = gb.prim.shape
    tri = _triangles(mesh, dev)
    put = lambda v: torch.from_numpy(np.asarray(v, np.float64)).to(dev)  # noqa: E731
    o32, d32, traced = _directions(gb, case, seed, light)
    o, d, n = put(o32), put(d32), put(gb.nrm)
    valid = torch.from_numpy(gb.valid).to(dev)
    prim = torch.from_numpy(np.where(gb.valid, gb.prim, 0).astype(np.int64)).to(dev)
    sent = torch.from_numpy(traced).to(dev).reshape(-1).nonzero()[:, 0]
    flat = lambda v: v.reshape((H * W,) + v.shape[2:])  # noqa: E731
    ao = case["mode"] == "ao"
    ids, ts = _closest(tri, flat(o)[sent], flat(d)[sent], flat(prim)[sent], case["ao_radius"] if ao else 1.0 - 1e-15)
    hit = torch.full((H * W,), -1, dtype=torch.int64, device=dev)
    dz, nz = torch.zeros((H * W, 3), dtype=torch.float64, device=dev), torch.zeros((H * W, 3), dtype=torch.float64, device=dev)
    hit[sent] = ids
    got = sent[ids >= 0]
    dz[got] = ts[ids >= 0, None] * flat(d)[got]
    nn = tri[3][hit[got]]
    nn = nn / nn.norm(dim=-1, keepdim=True)
    nz[got] = torch.where((nn * flat(d)[got]).sum(-1, keepdim=True) > 0, -nn, nn)
    hit, dz, nz = hit.reshape(H, W), dz.reshape(H, W, 3), nz.reshape(H, W, 3)
    miss = torch.zeros(H * W, dtype=torch.bool, device=dev)
    miss[sent] = ids < 0
    miss = miss.reshape(H, W)
    res = lambda img: {"hit": None, "dz": dz, "nz": nz, "image": img}  # noqa: E731
    if case["estimator"] == "none":
        if ao:
            return res(torch.where(valid & (hit >= 0), 0.0, 1.0).double())
        return res(miss.double())

    # densities p_k(j) of each candidate j at its receivers k = j + (dy, dx)
    if case["pattern"] == "window":
        D, T = 2 * case["r"], case["r"]
        offs = [(y, x) for y in range(-D, D + 1) for x in range(-D, D + 1)]
    else:
        gw, gh = {1: (1, 1), 2: (2, 1), 4: (2, 2), 8: (4, 2)}[case["group"]]
        offs = [(y, x) for y in range(1 - gh, gh) for x in range(1 - gw, gw)]
    jy, jx = (hit >= 0).nonzero(as_tuple=True)
    oj, dj, nzj = o[jy, jx], dz[jy, jx], nz[jy, jx]
    p = {}
    if not ao:
        lc, leu, lev = put(light.center), put(light.edge_u), put(light.edge_v)
        nl = torch.linalg.cross(leu, lev)
        nl = nl / nl.norm()
    for dy, dx in offs:
        ky, kx = jy + dy, jx + dx
        ok = (ky >= 0) & (ky < H) & (kx >= 0) & (kx < W)
        if case["pattern"] == "group":
            ok &= (torch.div(ky, gh, rounding_mode="floor") == jy // gh) & (torch.div(kx, gw, rounding_mode="floor") == jx // gw)
        ky, kx = ky.clamp(0, H - 1), kx.clamp(0, W - 1)
        ok &= valid[ky, kx]
        ow, nw = o[ky, kx], n[ky, kx]
        v = (oj - ow) + dj
        front, zw, d2 = (nw * v).sum(-1), (nzj * v).sum(-1), (v * v).sum(-1)
        if ao:
            q = front * -zw / (d2 * d2)
            ok &= (front > 0) & (zw < 0) & (d2 <= case["ao_radius"] ** 2)
        else:
            lw = v @ nl
            s = ((lc - ow) @ nl) / lw
            y = ow + s[:, None] * v - lc
            al, be = (y @ leu) / (leu @ leu), (y @ lev) / (lev @ lev)
            q = s * s * zw / lw
            ok &= (front > 0) & (lw < 0) & (zw < 0) & (s > 1) & (al.abs() <= 0.5) & (be.abs() <= 0.5)
        q = torch.where(ok, q, torch.zeros_like(q))
        if case["estimator"] == "unbiased" and (dy or dx):
            k = (q > 0).nonzero()[:, 0]
            b = _blocked(tri, ow[k], v[k], hit[jy[k], jx[k]], prim[ky[k], kx[k]])
            q[k[b]] = 0.0
        p[dy, dx] = q
    B = torch.zeros((H, W), dtype=torch.float64, device=dev)

    def add(dy, dx, P):
        q = p[dy, dx]
        k = ((q > 0) & (P > 0)).nonzero()[:, 0]
        B.index_put_((jy[k] + dy, jx[k] + dx), q[k] / P[k], accumulate=True)

    none = torch.ones((H, W), dtype=torch.bool, device=dev)  # no unblocked sample in the set
    if case["pattern"] == "window":
        for dy in range(-T, T + 1):
            for dx in range(-T, T + 1):
                add(dy, dx, sum(p[dy + y, dx + x] for y in range(-T, T + 1) for x in range(-T, T + 1)))
                none &= ~_shifted(miss, dy, dx, False)
    else:
        P = sum(p.values())
        for dy, dx in offs:
            add(dy, dx, P)
            near = _shifted(miss, dy, dx, False)
            yy, xx = torch.meshgrid(torch.arange(H, device=dev), torch.arange(W, device=dev), indexing="ij")
            same = (torch.div(yy + dy, gh, rounding_mode="floor") == yy // gh) & (torch.div(xx + dx, gw, rounding_mode="floor") == xx // gw)
            none &= ~(near & same)
    if ao:
        return res(torch.where(valid, 1.0 - B, torch.ones_like(B)))
    F = _front_fraction(o.reshape(-1, 3), n.reshape(-1, 3), light).reshape(H, W)
    img = F - B
    if case["estimator"] == "biased":
        img = torch.where(none, torch.zeros_like(img), img)
    return res(torch.where(valid, img, torch.zeros_like(img)))
