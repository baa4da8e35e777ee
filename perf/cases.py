"""The calls that are timed: render and reverse-mode gradient through the package's public entry points, from
the smallest image to the batches the benchmark runs.

A case names a scene family of scenegen and sizes:
  tiny     plane, three analytic spheres, one light (4 materials' worth of branches, 7 primitives)
  ring     16 icospheres on a textured ground, 20.5k triangles, cameras on a ring x polarizer angles
  maps     32 icospheres, blended ground with 256^2 albedo and roughness maps, two lights (inverse rendering)
  stage    light stage: circular lights, normal, specular and roughness maps, four analyzers
  terrain  uneven worlds of 1e5 to 1e6 triangles in one scene, four analyzers
  stack    85 linear polarizer sheets in front of a diffuse room (deep paths)
`op` is what the program calls: render, backward (the gradient alone), step (both), noalloc (the gradient
without a workspace) or fit (the autograd function under a squared loss).  The scene's geometry and the plan
are what a program keeps between calls; the parameters, the random seed and dL/dI come from the case's seed.
"""
import functools
import math

import numpy as np
import torch

import paper_2607_13265_amd as ppt
import scenegen as sg


def listed():
    return [
        # the smallest step: a 32 x 32 image of the three-sphere scene, 4 samples, depth 3 (launch latency)
        dict(name="tiny_step", family="tiny", op="step", width=32, height=32, spp=4, depth=3, views=1,
             sensor="polarizer", chunk=0, interval=0, counters=True),
        # a one-sample preview of odd size, whole Stokes vectors, no gradient (interactive view)
        dict(name="preview_render", family="ring", op="render", width=97, height=61, spp=1, depth=4, views=1,
             sensor="none", chunk=0, interval=0, counters=True),
        # four low-resolution views: the first, coarse iterations of an optimisation
        dict(name="coarse_views_step", family="ring", op="step", width=33, height=27, spp=8, depth=6, views=4,
             sensor="polarizer", chunk=0, interval=0, counters=False),
        # a gradient inside a program that may not allocate device memory, two views
        dict(name="noalloc_backward", family="ring", op="noalloc", width=128, height=128, spp=32, depth=6, views=2,
             sensor="polarizer", chunk=0, interval=0, counters=True),
        # one view at full size: 256 x 256, 64 samples, depth 8
        dict(name="single_view_step", family="ring", op="step", width=256, height=256, spp=64, depth=8, views=1,
             sensor="polarizer", chunk=0, interval=0, counters=False),
        # whole Stokes vectors of one view at 512 x 512 (a polarimetric ground-truth image)
        dict(name="stokes_render", family="maps", op="render", width=512, height=512, spp=16, depth=6, views=1,
             sensor="none", chunk=0, interval=0, counters=True),
        # the benchmark's batch: 4 poses x 32 polarizer angles in one launch sequence, default chunk size
        dict(name="batched_views_step", family="ring", op="step", width=128, height=128, spp=32, depth=6, views=128,
             sensor="polarizer", chunk=0, interval=0, counters=False),
        # one iteration of inverse rendering: image, squared loss, decorrelated gradient of the maps and lights
        dict(name="inverse_rendering_step", family="maps", op="fit", width=512, height=512, spp=16, depth=6, views=8,
             sensor="polarizer", chunk=1 << 23, interval=0, counters=False),
        # multi-view light-stage capture with all maps
        dict(name="light_stage_step", family="stage", op="step", width=256, height=256, spp=16, depth=6, views=8,
             sensor="lightstage", chunk=0, interval=0, counters=False),
        # worlds of different sizes, resolutions and sample counts in one call
        dict(name="uneven_worlds_step", family="terrain", op="step", width=0, height=0, spp=0, depth=12, views=3,
             sensor="analyzer", chunk=0, interval=0, counters=False),
        # deep paths: 85 sheets at depth 128, cached suffixes
        dict(name="deep_stack_step", family="stack", op="step", width=1280, height=720, spp=1, depth=128, views=1,
             sensor="none", chunk=0, interval=0, counters=False),
        # the same deep paths with bounded memory: checkpoints every 16 vertices
        dict(name="deep_stack_hybrid", family="stack", op="backward", width=640, height=360, spp=1, depth=128, views=1,
             sensor="none", chunk=0, interval=16, counters=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same families and ranges: sizes log-uniform (odd ones among them), up to the listed largest."""
    family = rng.choice(["tiny", "ring", "ring", "ring", "maps", "stage", "stack"])
    c = dict(family=family, chunk=0, interval=0, counters=rng.random() < 0.5, views=1)
    if family == "stack":
        c["op"] = rng.choice(["render", "step", "backward"])
        c["depth"] = rng.randint(87, 128)
        c["width"], c["height"], c["spp"] = _log(rng, 64, 1280), _log(rng, 36, 720), 1
        c["sensor"] = "none"
        c["interval"] = rng.choice([0, 0, 8, 16])
        return c
    c["op"] = rng.choice(["render", "backward", "step", "step"] + (["noalloc"] if family == "ring" else []))
    c["depth"] = rng.randint(2, 4) if family == "tiny" else rng.randint(3, 8)
    c["width"] = _log(rng, 24, 384)
    c["height"] = _log(rng, max(16, c["width"] // 2), c["width"])
    c["spp"] = _log(rng, 1, 64)
    if family in ("ring", "maps", "stage"):
        c["views"] = _log(rng, 1, 64 if family == "ring" else 8)
    most = 1 << (20 if c["op"] == "noalloc" else 24)
    while c["width"] * c["height"] * c["spp"] * c["views"] > most:
        if c["spp"] > 1:
            c["spp"] = (c["spp"] + 1) // 2
        else:
            c["views"] = (c["views"] + 1) // 2
    c["sensor"] = "lightstage" if family == "stage" else rng.choice(["polarizer", "polarizer", "none", "analyzer"])
    if rng.random() < 0.25:
        c["chunk"] = 1 << rng.randint(16, 20)
    return c


SENSORS = {"none": sg.SENSOR_NONE, "polarizer": sg.SENSOR_POLARIZER, "analyzer": sg.SENSOR_ANALYZER4,
           "lightstage": sg.SENSOR_LIGHTSTAGE4}
# parameters whose gradient the programs of each family ask for
WANTED = {"tiny": ("theta", "albedo", "ior"), "ring": ("albedo_tex", "roughness", "theta_views"),
          "maps": ("albedo_tex", "roughness_tex", "light_Le"),
          "stage": ("ground_normal", "ground_specular", "ground_roughness", "object_normal", "object_specular",
                    "object_roughness", "glass_normal", "metal_normal", "metal_specular"),
          "terrain": ("albedo_tex", "roughness", "light_Le"), "stack": ("floor_albedo", "wall_albedo")}
VERTICES = {"tiny": 1.3, "ring": 0.93, "maps": 1.3, "stage": 1.07, "terrain": 1.29}  # mean vertices of a path


@functools.lru_cache(maxsize=16)
def _workload(family, width, height, spp, depth, views, sensor):
    """The scene (host data) and the view records of a case."""
    kind = SENSORS[sensor]
    if family == "terrain":
        wl = sg.config5(range(50, 50 + views))
        return wl.scene, wl.views
    if family == "stack":
        wl = sg.polarizer_stack(width=width, height=height, spp=spp, max_depth=depth)
        return wl.scene, wl.views
    if family == "stage":
        wl = sg.lightstage(res=256, spp=spp, n_views=views)
        sc, recs = wl.scene, wl.views.copy()
        recs["width"], recs["height"], recs["crop_w"], recs["crop_h"] = width, height, width, height
        return sc, recs
    if family == "tiny":
        sc = sg.config1().scene
        recs = [sg.make_view(0, width, height, spp, (0, 1, 6), (0, -0.5, 0), (0, 1, 0), 40.0, kind,
                             sc.slot("theta") if sensor == "polarizer" else -1, 0, 0)]
    elif family == "ring":
        sc, _ = sg.scene2()
        angles = min(views, 32)
        th = sc.add_slot("theta_views", [k * np.pi / angles + 0.1 for k in range(angles)])
        recs = [sg.make_view(0, width, height, spp, sg.ring_pose(k // angles), (0, 0, 0), (0, 1, 0), 45.0, kind,
                             th if sensor == "polarizer" else -1, k % angles if sensor == "polarizer" else 0, k)
                for k in range(views)]
    else:
        sc = sg.scene4()
        th = sc.slot("theta_views")
        recs = [sg.make_view(0, width, height, spp, (0.0, 6.0, 7.0), (0, -1, 0), (0, 1, 0), 50.0, kind,
                             th if sensor == "polarizer" else -1, k if sensor == "polarizer" else 0, k)
                for k in range(views)]
    return sc, np.asarray(recs, sg.VIEW_DTYPE)


@functools.lru_cache(maxsize=4)
def _blob(*key):
    return _workload(*key)[0].to_blob()


def _key(case):
    return (case["family"], case["width"], case["height"], case["spp"], case["depth"], case["views"], case["sensor"])


def _wanted(case, names):
    bases = WANTED[case["family"]]
    return [any(n == b or n.endswith("_" + b) and n[0] == "w" for b in bases) for n in names]


def _inputs(case, seed):
    """Parameter values (float32 arrays, one per slot) and dL/dI of a seed: per-pixel positive weights on the
    intensities of a radiance loss, weaker signed ones on the other Stokes components."""
    sc, views = _workload(*_key(case))
    rng = np.random.default_rng([int(seed), 7])
    params = [(p * rng.uniform(0.9, 1.1, p.shape)).astype(np.float32) for p in sc.params()]
    n = sg.image_numel(views)
    g = torch.Generator().manual_seed(int(seed) * 2 + 1)
    d = None
    if case["op"] in ("backward", "step", "noalloc"):
        d = torch.empty(n // 4, 4).uniform_(-0.25, 0.25, generator=g)
        d[:, 0] = d[:, 0] * 2 + 1.0
        d = (d / (n / 12)).reshape(-1)
    return params, d


class _State:
    pass


def prepare(case, seed):
    sc, views = _workload(*_key(case))
    s = _State()
    s.op, s.seed = case["op"], int(seed)
    params, d = _inputs(case, seed)
    s.scene = ppt.Scene(_blob(*_key(case)))
    s.plan = ppt.Plan(s.scene, views, case["depth"], chunk_paths=case["chunk"], checkpoint_interval=case["interval"])
    if not case["counters"]:
        s.plan.set_stats(False)
    s.params = [torch.from_numpy(p).cuda() for p in params]
    s.want = _wanted(case, sc.slot_names)
    s.d = None if d is None else d.cuda()
    if s.op == "noalloc":
        s.grads = [torch.empty_like(p) if w else None for p, w in zip(s.params, s.want)]
    if s.op == "fit":
        # the target: the same views under brighter lights, another random stream
        le = sc.slot("light_Le")
        brighter = [p * 1.5 if k == le else p for k, p in enumerate(s.params)]
        s.target = s.plan.render(brighter, s.seed + 5000)
        s.params = [p.requires_grad_(w) for p, w in zip(s.params, s.want)]
    return s


def run(s):
    if s.op == "render":
        return {"image": s.plan.render(s.params, s.seed)}
    if s.op == "noalloc":
        return {"grads": [g for g in s.plan.backward_noalloc(s.params, s.seed, s.d, s.grads) if g is not None]}
    if s.op == "fit":
        for p in s.params:
            p.grad = None
        image = ppt.render(s.plan, s.params, s.seed, backward_seed=s.seed + 1000003)
        (image - s.target).square().mean().backward()
        return {"image": image.detach(), "grads": [p.grad for p in s.params if p.grad is not None]}
    out = {}
    if s.op == "step":
        out["image"] = s.plan.render(s.params, s.seed)
    grads = s.plan.backward(s.params, s.seed, s.d, want=s.want)
    out["grads"] = [g for g in grads if g is not None]
    return out


def work(case):
    """Arrays in and out once; arithmetic of the node and primitive tests and of shading (about 3000 operations a
    vertex to render, 3900 with its derivatives)."""
    sc, views = _workload(*_key(case))
    paths = int(np.sum(views["crop_w"].astype(np.int64) * views["crop_h"] * views["spp"]))
    per = case["depth"] * 0.6 if case["family"] == "stack" else VERTICES[case["family"]]
    image = 4 * sg.image_numel(views)
    params = 4 * sum(p.size for p in sc.slot_values)
    wanted = 4 * sum(p.size for p, w in zip(sc.slot_values, _wanted(case, sc.slot_names)) if w)
    geometry = sum(w.n_tris() * 36 for w in sc.worlds)
    ahead, back = case["op"] in ("render", "step", "fit"), case["op"] != "render"
    return {"bytes": (image + params + geometry) * ahead + (image + params + geometry + wanted) * back,
            "flops": paths * per * (3000 * ahead + 3900 * back)}


# ---------------------------------------------------------------------------- the estimator in 64 bits
# A plain path tracer in torch (float64): the same Philox counters, so the same paths; every triangle is tested;
# the gradient is torch's own reverse mode of the sum of dL/dI times the image, with sampling detached.  It knows
# the materials without normal or specular maps and without circular light.
MOST_TESTS = 2.5e10  # ray-triangle tests beyond which it would take too long


def _philox(c, seed):
    m = 0xFFFFFFFF
    c = [x & m for x in c]
    k0, k1 = seed & m, (seed >> 32) & m

    def mul(a, x):
        hi = (a * (x >> 16) + ((a * (x & 0xFFFF)) >> 16)) >> 16
        return hi & m, (a * x) & m

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return [(x >> 8).double() * 2.0 ** -24 for x in c]


def _dot(a, b):
    return (a * b).sum(-1)


def _unit(a):
    return a / a.norm(dim=-1, keepdim=True)


def _basis(n):
    """The orthonormal basis of Duff et al. 2017."""
    sg_ = torch.where(torch.signbit(n[:, 2]), -1.0, 1.0).double()
    a = -1.0 / (sg_ + n[:, 2])
    b = n[:, 0] * n[:, 1] * a
    x = torch.stack([1 + sg_ * n[:, 0] ** 2 * a, sg_ * b, -sg_ * n[:, 0]], -1)
    return x, torch.stack([b, sg_ + n[:, 1] ** 2 * a, -n[:, 1]], -1)


def _rotator(k, x0, x1):
    c, s = _dot(x0, x1), _dot(torch.cross(k, x0, dim=-1), x1)
    return c * c - s * s, 2 * c * s


def _rotation(c, s):
    r = torch.zeros(c.shape[0], 4, 4, dtype=torch.float64, device=c.device)
    r[:, 0, 0] = r[:, 3, 3] = 1
    r[:, 1, 1] = r[:, 2, 2] = c
    r[:, 1, 2], r[:, 2, 1] = s, -s
    return r


def _retarder_diattenuator(a, b, c, d):
    z = torch.zeros_like(a)
    return torch.stack([torch.stack(r, -1) for r in ((a, b, z, z), (b, a, z, z), (z, z, c, d), (z, z, -d, c))], -2)


def _fresnel(ci, m, transmit):
    """Mueller entries (a, b, c, d) of the Born and Wolf amplitudes at incidence cosine ci, relative index m."""
    st2 = (1 - ci * ci) / (m * m)
    ct = torch.sqrt(torch.complex((1 - st2).real, (1 - st2).imag + 0.0))
    if transmit:
        s, p = 2 * ci / (ci + m * ct), 2 * ci / (m * ci + ct)
        scale = (m * ct).real / ci
    else:
        s, p = (ci - m * ct) / (ci + m * ct), (m * ci - ct) / (m * ci + ct)
        scale = 1.0
    A, B, z = s.real ** 2 + s.imag ** 2, p.real ** 2 + p.imag ** 2, s * p.conj()
    return [scale * v for v in (0.5 * (A + B), 0.5 * (A - B), z.real, z.imag)]


class _World:
    def __init__(self, w, offsets, dev):
        t = lambda x: torch.as_tensor(np.ascontiguousarray(x), device=dev)  # noqa: E731
        v = t(np.concatenate(w.tri_v).astype(np.float64))
        self.uv = t(np.concatenate(w.tri_uv).astype(np.float64))
        self.v0, self.e1, self.e2 = v[:, 0], v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]
        n = torch.cross(self.e1, self.e2, dim=-1)
        self.n = _unit(n)
        # det, t det, u det and v det of the triangle test as products with (o, d) and (o x d, d)
        self.gdet, self.gt = -n, torch.cat([n, -_dot(self.v0, n)[:, None]], -1)
        self.gu = torch.cat([self.e2, -torch.cross(self.e2, self.v0, dim=-1)], -1)
        self.gv = torch.cat([-self.e1, -torch.cross(self.v0, self.e1, dim=-1)], -1)
        sph = np.asarray(w.spheres, np.float32).astype(np.float64).reshape(-1, 5)
        self.spheres = t(sph[:, :4])
        self.n_tris = self.v0.shape[0]
        self.mat = torch.cat([t(np.concatenate(w.tri_mat).astype(np.int64)), t(sph[:, 4].astype(np.int64))])
        m = np.asarray(w.materials, sg.MAT_DTYPE)
        off = lambda slot, o: t(np.where(m[slot] >= 0, offsets[m[slot]] + m[o].astype(np.int64), -1))  # noqa: E731
        self.type = t(m["type"].astype(np.int64))
        self.alb, self.alb_w, self.alb_h = off("albedo_slot", "albedo_off"), t(m["albedo_tw"].astype(np.int64)), t(m["albedo_th"].astype(np.int64))
        self.alp, self.alp_w, self.alp_h = off("alpha_slot", "alpha_off"), t(m["alpha_tw"].astype(np.int64)), t(m["alpha_th"].astype(np.int64))
        self.eta, self.kap, self.emit = off("eta_slot", "eta_off"), off("kappa_slot", "kappa_off"), off("emit_slot", "emit_off")
        self.axis, self.blend = t(m["axis"].astype(np.float64)), t(m["blend"].astype(np.float32).astype(np.float64))
        li = np.asarray(w.lights, sg.LIGHT_DTYPE)
        self.lp, self.lu, self.lv = (t(li[k].astype(np.float64)) for k in ("p0", "eu", "ev"))
        ln = torch.cross(self.lu, self.lv, dim=-1)
        self.area = ln.norm(dim=-1)
        self.ln = ln / self.area[:, None]
        self.le = t(offsets[li["le_slot"]] + li["le_off"].astype(np.int64))

    def hit(self, o, d, tmax):
        """Nearest hit in (0, tmax): distance, primitive (-1: none), barycentrics."""
        n = o.shape[0]
        best = tmax.clone()
        prim = torch.full((n,), -1, dtype=torch.int64, device=o.device)
        bu, bv = torch.zeros_like(best), torch.zeros_like(best)
        step = max(1, int(2e7 // max(self.n_tris, 1)))
        for a in range(0, n, step):
            oo, dd = o[a:a + step], d[a:a + step]
            pl = torch.cat([torch.cross(oo, dd, dim=-1), dd], -1)
            inv = 1.0 / (dd @ self.gdet.T)
            u, v = (pl @ self.gu.T) * inv, (pl @ self.gv.T) * inv
            tt = (oo @ self.gt[:, :3].T + self.gt[:, 3]) * inv
            ok = (u >= 0) & (v >= 0) & (u + v <= 1) & (tt > 0)
            tt = torch.where(ok, tt, math.inf)
            t, k = tt.min(-1)
            got = t < best[a:a + step]
            best[a:a + step] = torch.where(got, t, best[a:a + step])
            prim[a:a + step] = torch.where(got, k, -1)
            bu[a:a + step] = torch.where(got, u.gather(1, k[:, None])[:, 0], 0.0)
            bv[a:a + step] = torch.where(got, v.gather(1, k[:, None])[:, 0], 0.0)
        for j in range(self.spheres.shape[0]):
            oc, r = o - self.spheres[j, :3], self.spheres[j, 3]
            b, c = _dot(d, oc), _dot(oc, oc) - r * r
            disc = b * b - c
            sq = disc.clamp(min=0).sqrt()
            t = torch.where(-b - sq > 0, -b - sq, -b + sq)
            got = (disc >= 0) & (t > 0) & (t < best)
            best, prim = torch.where(got, t, best), torch.where(got, self.n_tris + j, prim)
        return best, prim, bu, bv


def _texture(P, off, tw, th, u, v, ch):
    """Constant (tw = 0) or bilinear texture, clamped at the edges, texel centres at (i + 1/2) / N."""
    w, h = tw.clamp(min=1), th.clamp(min=1)
    x, y = u * w - 0.5, v * h - 0.5
    x0, y0 = x.floor(), y.floor()
    fx, fy = x - x0, y - y0
    k = torch.arange(ch, device=P.device)
    out = 0
    for dx, wx in ((0, 1 - fx), (1, fx)):
        for dy, wy in ((0, 1 - fy), (1, fy)):
            xi = torch.minimum((x0.long() + dx).clamp(min=0), w - 1)
            yi = torch.minimum((y0.long() + dy).clamp(min=0), h - 1)
            out = out + (wx * wy)[:, None] * P[((off + (yi * w + xi) * ch)[:, None] + k)]
    return torch.where((tw > 0)[:, None], out, P[off[:, None] + k])


def _glossy(W, P, m, q, wi, eta):
    """Mueller matrix of the microfacet lobe for light along -wi to wo, and cos_i."""
    h = _unit(wi + q["wo"])
    ci, co, ch = _dot(q["ns"], wi), _dot(q["ns"], q["wo"]), _dot(q["ns"], h)
    a2 = q["alpha"] ** 2
    D = a2 / (math.pi * ((a2 - 1) * ch * ch + 1) ** 2)
    g1 = lambda c: 1 / (1 + 0.5 * (torch.sqrt(1 + a2 * (1 - c * c) / (c * c)) - 1))  # noqa: E731
    kappa = D * g1(ci) * g1(co) / (4 * ci * co)
    F = _retarder_diattenuator(*_fresnel(_dot(wi, h).abs(), eta, False))
    return kappa[:, None, None] * _framed(F, -wi, h, q["wo"]), ci


def _framed(F, k_in, n_inc, k_out):
    s = torch.cross(k_in, n_inc, dim=-1)
    l2 = _dot(s, s)
    s = torch.where((l2 < 1e-16)[:, None], _basis(k_in)[0], s / l2.clamp(min=1e-300).sqrt()[:, None])
    return _rotation(*_rotator(k_out, s, _basis(k_out)[0])) @ F @ _rotation(*_rotator(k_in, _basis(k_in)[0], s))


def _eps(p):
    return 1e-4 * (1 + p.abs().amax(-1))


def _leave(p, ng, d):
    return p + ng * torch.where(_dot(d, ng) > 0, _eps(p), -_eps(p))[:, None]


def _half_vector_sample(ns, wo, alpha, u1, u2):
    ch = 1 / torch.sqrt(1 + alpha ** 2 * u1 / (1 - u1))
    sh = (1 - ch * ch).clamp(min=0).sqrt()
    x, y = _basis(ns)
    h = x * (sh * torch.cos(2 * math.pi * u2))[:, None] + y * (sh * torch.sin(2 * math.pi * u2))[:, None] + ns * ch[:, None]
    woh = _dot(wo, h)
    wi = h * (2 * woh)[:, None] - wo
    D = alpha ** 2 / (math.pi * ((alpha ** 2 - 1) * ch * ch + 1) ** 2)
    return wi, D * ch / (4 * woh), (woh > 0) & (_dot(ns, wi) > 0)


def _paths(W, P, view, depth, seed, pix, smp):
    """Stokes radiance (paths, 3, 4) in the sensor frame of one view's paths."""
    dev = pix.device
    vid = int(view["view_id"])
    n = pix.shape[0]
    f64 = lambda k: torch.as_tensor(view[k].astype(np.float64), device=dev)  # noqa: E731
    f = _unit(f64("target") - f64("origin"))
    r = _unit(torch.cross(f, f64("up"), dim=-1))
    up = torch.cross(r, f, dim=-1)
    th = math.tan(0.5 * math.radians(float(view["fov_y_deg"])))
    wd, ht = int(view["width"]), int(view["height"])
    u = _philox([pix, smp, torch.full_like(pix, vid << 8), torch.zeros_like(pix)], seed)
    sx = (2 * ((pix % wd).double() + u[0]) / wd - 1) * th * (wd / ht)
    sy = (1 - 2 * ((pix // wd).double() + u[1]) / ht) * th
    d = _unit(f + r * sx[:, None] + up * sy[:, None])
    o = f64("origin").expand(n, 3)
    k = -d
    sensor = _rotation(*_rotator(k, _basis(k)[0], _unit(r - k * _dot(k, r)[:, None])))
    M = torch.eye(4, dtype=torch.float64, device=dev).expand(n, 4, 4)
    scale = torch.ones(n, 3, dtype=torch.float64, device=dev)
    total = torch.zeros(n, 3, 4, dtype=torch.float64, device=dev)
    ids = torch.arange(n, device=dev)
    delta = torch.zeros(n, dtype=torch.bool, device=dev)
    c3 = torch.arange(3, device=dev)
    for b in range(1, depth + 1):
        t, prim, hu, hv = W.hit(o, d, torch.full((ids.shape[0],), math.inf, dtype=torch.float64, device=dev))
        live = prim >= 0
        ids, o, d, M, scale, delta, t, prim, hu, hv = (x[live] for x in (ids, o, d, M, scale, delta, t, prim, hu, hv))
        if ids.numel() == 0:
            break
        tri = prim < W.n_tris
        pt = torch.where(tri, prim, 0)
        p, ng = o + d * t[:, None], W.n[pt]
        b0 = 1 - hu - hv
        uv = b0[:, None] * W.uv[pt, 0] + hu[:, None] * W.uv[pt, 1] + hv[:, None] * W.uv[pt, 2]
        p = torch.where(tri[:, None], W.v0[pt] + W.e1[pt] * hu[:, None] + W.e2[pt] * hv[:, None], p)
        if W.spheres.shape[0]:
            ps = torch.where(tri, 0, prim - W.n_tris)
            no = _unit(p - W.spheres[ps, :3])
            ng = torch.where(tri[:, None], ng, torch.where((W.spheres[ps, 3] < 0)[:, None], -no, no))
            suv = torch.stack([0.5 + torch.atan2(no[:, 2], no[:, 0]) / (2 * math.pi), torch.acos(no[:, 1].clamp(-1, 1)) / math.pi], -1)
            uv = torch.where(tri[:, None], uv, suv)
        m = W.mat[prim]
        ty = W.type[m]
        wo = -d
        front = _dot(ng, wo) > 0
        ns = torch.where(front[:, None], ng, -ng)

        def add(sel, stokes):  # radiance of the paths sel of this bounce: throughput times a Stokes vector per channel
            nonlocal total
            lo = scale[sel][..., None] * (M[sel][:, None] @ stokes[..., None])[..., 0]
            total = total.index_add(0, ids[sel], lo)

        e = torch.nonzero((W.emit[m] >= 0) & front & (delta | (b == 1)))[:, 0]
        if e.numel():
            s = torch.zeros(e.numel(), 3, 4, dtype=torch.float64, device=dev)
            s[..., 0] = P[W.emit[m[e]][:, None] + c3]
            add(e, s)
        if b == depth:
            break
        ctr = [pix[ids], smp[ids], torch.full_like(ids, (vid << 8) | b)]
        ua, ub = (_philox(ctr + [torch.full_like(ids, c)], seed) for c in (0, 1))
        alpha = torch.where(W.alp[m] >= 0, _texture(P, W.alp[m].clamp(min=0), W.alp_w[m], W.alp_h[m], uv[:, 0], uv[:, 1], 1)[:, 0], 0.5)
        alpha = alpha.clamp(1e-3, 1)
        rho = _texture(P, W.alb[m].clamp(min=0), W.alb_w[m], W.alb_h[m], uv[:, 0], uv[:, 1], 3)
        eta = torch.where(W.eta[m] >= 0, P[W.eta[m].clamp(min=0)], 1.5)
        kap = torch.where((W.kap[m] >= 0) & (ty == sg.MAT_GGX_CONDUCTOR), P[W.kap[m].clamp(min=0)], 0.0)
        q = dict(ns=ns, wo=wo, alpha=alpha)
        pick = lambda sel: {key: v[sel] for key, v in q.items()}  # noqa: E731
        # next-event estimation
        nl = W.lp.shape[0]
        if nl:
            li = (ua[3] * nl).long().clamp(max=nl - 1)
            y = W.lp[li] + W.lu[li] * ub[0][:, None] + W.lv[li] * ub[1][:, None]
            dv = y - p
            dist = dv.norm(dim=-1)
            wl = dv / dist[:, None]
            cy, cx = -_dot(W.ln[li], wl), _dot(ns, wl)
            no_nee = (ty == sg.MAT_EMITTER) | (ty == sg.MAT_DIELECTRIC) | (ty == sg.MAT_SHEET)
            a = torch.nonzero(~no_nee & (cy > 0) & (cx > 0))[:, 0]
            so = _leave(p[a], ng[a], wl[a])
            sv = y[a] - so
            sl = sv.norm(dim=-1)
            a = a[W.hit(so, sv / sl[:, None], sl - _eps(y[a]))[1] < 0]
            if a.numel():
                geom = (cy * W.area[li] * nl / dist ** 2 * cx)[a]
                le = P[W.le[li[a]][:, None] + c3] * geom[:, None]
                wd_ = torch.where(ty[a] == sg.MAT_LAMBERT, 1.0, torch.where(ty[a] == sg.MAT_BLEND, W.blend[m[a]], 0.0))
                s = torch.zeros(a.numel(), 3, 4, dtype=torch.float64, device=dev)
                s[..., 0] = wd_[:, None] * rho[a] / math.pi * le
                g = torch.nonzero(wd_ < 1)[:, 0]
                if g.numel():
                    col, _ = _glossy(W, P, m[a[g]], pick(a[g]), wl[a[g]], torch.complex(eta[a[g]], kap[a[g]]))
                    s = s.index_add(0, g, ((1 - wd_[g])[:, None] * le[g])[..., None] * col[:, None, :, 0])
                add(a, s)
        # continuation: direction and selection detached, weights differentiated
        wi = torch.zeros_like(d)
        w4 = torch.zeros(ids.numel(), 4, 4, dtype=torch.float64, device=dev)
        wr = torch.ones(ids.numel(), 3, dtype=torch.float64, device=dev)
        cont = torch.zeros(ids.numel(), dtype=torch.bool, device=dev)
        blend = ty == sg.MAT_BLEND
        dif = torch.nonzero((ty == sg.MAT_LAMBERT) | (blend & (ua[0] < W.blend[m])))[:, 0]
        if dif.numel():
            x, yv = _basis(ns[dif])
            rr, ph = ua[1][dif].sqrt(), 2 * math.pi * ua[2][dif]
            wi[dif] = x * (rr * ph.cos())[:, None] + yv * (rr * ph.sin())[:, None] + ns[dif] * (1 - ua[1][dif]).clamp(min=0).sqrt()[:, None]
            e00 = torch.zeros(4, 4, dtype=torch.float64, device=dev)
            e00[0, 0] = 1
            w4 = w4.index_copy(0, dif, e00.expand(dif.numel(), 4, 4))
            wr = wr.index_copy(0, dif, rho[dif])
            cont[dif] = True
        glo = torch.nonzero((ty == sg.MAT_GGX_DIELECTRIC) | (ty == sg.MAT_GGX_CONDUCTOR) | (blend & ~(ua[0] < W.blend[m])))[:, 0]
        if glo.numel():
            w_, pdf, ok = _half_vector_sample(ns[glo], wo[glo], alpha[glo].detach(), ua[1][glo], ua[2][glo])
            glo, w_, pdf = glo[ok], w_[ok], pdf[ok]
            wi[glo] = w_
            mat, ci = _glossy(W, P, m[glo], pick(glo), w_, torch.complex(eta[glo], kap[glo]))
            w4 = w4.index_copy(0, glo, (ci / pdf)[:, None, None] * mat)
            cont[glo] = True
        die = torch.nonzero(ty == sg.MAT_DIELECTRIC)[:, 0]
        if die.numel():
            one = torch.ones_like(eta[die])
            mr = torch.where(front[die], eta[die], 1 / eta[die])
            mrd = mr.detach()
            co = _dot(ns[die], wo[die])
            st2 = (1 - co * co) / mrd ** 2
            PR = torch.where(st2 < 1, _fresnel(co, torch.complex(mrd, 0 * one), False)[0], 1.0)
            re = ua[0][die] < PR
            wr_ = ns[die] * (2 * co)[:, None] - wo[die]
            wt = _unit(-wo[die] / mrd[:, None] + ns[die] * (co / mrd - (1 - st2).clamp(min=0).sqrt())[:, None])
            wi[die] = torch.where(re[:, None], wr_, wt)
            for sel, refl in ((torch.nonzero(re)[:, 0], True), (torch.nonzero(~re)[:, 0], False)):
                if sel.numel():
                    g = die[sel]
                    cc = co[sel] if refl else _dot(wi[g], ns[g]).abs()
                    mm = mr[sel] if refl else 1 / mr[sel]
                    F = _retarder_diattenuator(*_fresnel(cc, torch.complex(mm, 0 * mm), not refl))
                    F = F / (PR[sel] if refl else 1 - PR[sel])[:, None, None]
                    w4 = w4.index_copy(0, g, _framed(F, -wi[g], ns[g] if refl else -ns[g], wo[g]))
            cont[die] = True
        she = torch.nonzero(ty == sg.MAT_SHEET)[:, 0]
        if she.numel():
            wi[she] = -wo[she]
            kk, ax = wo[she], W.axis[m[she]]
            xt, xc = _unit(ax - kk * _dot(ax, kk)[:, None]), _basis(kk)[0]
            h, z = torch.full_like(kk[:, 0], 0.5), torch.zeros_like(kk[:, 0])
            F = _rotation(*_rotator(kk, xt, xc)) @ _retarder_diattenuator(h, h, z, z) @ _rotation(*_rotator(kk, xc, xt))
            w4 = w4.index_copy(0, she, F)
            cont[she] = True
        M, scale = M[cont] @ w4[cont], scale[cont] * wr[cont]
        delta = ((ty == sg.MAT_DIELECTRIC) | (ty == sg.MAT_SHEET))[cont]
        o, d, ids = _leave(p[cont], ng[cont], wi[cont]), wi[cont], ids[cont]
    return (sensor[:, None] @ total[..., None])[..., 0]


def _analyzers(view, P, theta, dev):
    """The sensor's Mueller matrices, (analyzers, 4, 4)."""
    def linear(c, s):
        q = torch.stack([torch.ones_like(c), c, s, torch.zeros_like(c)])
        return 0.5 * q[:, None] * q[None, :]
    if view["sensor"] == sg.SENSOR_NONE:
        return torch.eye(4, dtype=torch.float64, device=dev)[None]
    if view["sensor"] == sg.SENSOR_POLARIZER:
        return linear(torch.cos(2 * P[theta]), torch.sin(2 * P[theta]))[None]
    at = lambda c, s: linear(*(torch.tensor(float(x), dtype=torch.float64, device=dev) for x in (c, s)))  # noqa: E731
    plate = torch.zeros(4, 4, dtype=torch.float64, device=dev)  # quarter wave: s2 <- s3
    plate[0, 0] = plate[1, 1] = plate[2, 3] = 1
    plate[3, 2] = -1
    return torch.stack([at(1, 0), at(0, 1), at(-1, 0), at(0, 1) @ plate])


def exact(case, seed):
    sc, views = _workload(*_key(case))
    paths = sum(int(v["crop_w"]) * int(v["crop_h"]) * int(v["spp"]) for v in views)
    tests = paths * VERTICES.get(case["family"], 90) * 2.5 * max(w.n_tris() for w in sc.worlds)
    if case["family"] not in ("tiny", "ring", "maps", "stack") or case["op"] == "fit" or tests > MOST_TESTS:
        return None
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    params, d = _inputs(case, seed)
    sizes = np.asarray([p.size for p in params])
    offsets = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    back = case["op"] != "render"
    P = torch.from_numpy(np.concatenate(params).astype(np.float64)).to(dev).requires_grad_(back)
    W = _World(sc.worlds[0], offsets, dev)
    blocks, at, grad = [], 0, torch.zeros_like(P)
    for view in views:
        n_pix, spp = int(view["crop_w"]) * int(view["crop_h"]), int(view["spp"])
        theta = int(offsets[view["theta_slot"]] + view["theta_off"]) if view["theta_slot"] >= 0 else None
        i = torch.arange(n_pix * spp, device=dev)
        lo = _paths(W, P, view, case["depth"], int(seed), i // spp, i % spp).reshape(n_pix, spp, 3, 4).mean(1)
        image = (_analyzers(view, P, theta, dev)[:, None, None] @ lo[None, ..., None])[..., 0].reshape(-1)
        if back:
            grad += torch.autograd.grad((image * d[at:at + image.numel()].to(dev, torch.float64)).sum(), P)[0]
        blocks.append(image.detach())
        at += image.numel()
    out = {}
    if case["op"] in ("render", "step"):
        out["image"] = torch.cat(blocks)
    if back:
        out["grads"] = [grad[o:o + s] for o, s, w in zip(offsets, sizes, _wanted(case, sc.slot_names)) if w]
    return out
