"""Small calls, whose paths run all their bounces in one launch, against the launches per bounce (which
per-kernel timing keeps): the same paths through the same records, so images, signatures and counts are equal
and gradients differ by the order of their additions only."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# about 200 FP32 operations of a path's share of a gradient in another order: 200 * 2^-24
TOL = 1.2e-5


def _two_worlds():
    """A dielectric and a conductor sphere over a ground, and a closed box of polarizer sheets: one scene."""
    sc = sg.Scene()
    s_alb, s_ior, s_rgh = sc.add_slot("albedo", [0.6, 0.5, 0.4]), sc.add_slot("ior", [1.5, 0.6]), sc.add_slot("rough", [0.2])
    s_kap, s_le, s_th = sc.add_slot("kappa", [3.0]), sc.add_slot("Le", [6.0, 5.0, 4.0]), sc.add_slot("theta", [0.3, 1.1])
    for k in range(2):
        w = sc.add_world()
        lam = w.add_material(type=sg.MAT_LAMBERT, albedo_slot=s_alb)
        w.add_quad((-5, -1, -5), (0, 0, 10), (10, 0, 0), lam)
        w.add_light((-1, 4, -1), (2, 0, 0), (0, 0, 2), s_le)
        if k == 0:
            w.add_sphere((-0.7, 0, 0), 0.8, w.add_material(type=sg.MAT_DIELECTRIC, eta_slot=s_ior))
            w.add_sphere((1.0, 0, 0.5), 0.7, w.add_material(type=sg.MAT_GGX_CONDUCTOR, alpha_slot=s_rgh, eta_slot=s_ior,
                                                            eta_off=1, kappa_slot=s_kap))
        else:
            for i in range(3):
                w.add_quad((-3, -1, 1.0 + i), (6, 0, 0), (0, 4, 0),
                           w.add_material(type=sg.MAT_SHEET, axis=(np.cos(0.3 * i), np.sin(0.3 * i), 0.0)))
    return sc, s_th


def _views(kind, sensor, sizes, theta):
    cam = {"tiny": ((0, 1, 6), (0, -0.5, 0), 40.0), "ring": (sg.ring_pose(0), (0, 0, 0), 45.0),
           "worlds": ((0, 1.5, 6), (0, 0, 0), 45.0)}[kind]
    pol = sensor == sg.SENSOR_POLARIZER
    views = np.asarray([sg.make_view(k % 2 if kind == "worlds" else 0, max(w, 1), h, spp, cam[0], cam[1], (0, 1, 0), cam[2],
                                     sensor, theta if pol else -1, 0, k) for k, (w, h, spp) in enumerate(sizes)], sg.VIEW_DTYPE)
    views["crop_w"] = [w for w, _, _ in sizes]  # (a width of 0: a view without paths)
    return views


@pytest.mark.parametrize("kind,sensor,sizes,depth,flags,kw", [
    ("tiny", sg.SENSOR_POLARIZER, [(1, 1, 1)], 3, 0, {}),
    ("tiny", sg.SENSOR_NONE, [(31, 1, 1), (0, 5, 3), (33, 2, 1)], 4, 0, {}),
    ("tiny", sg.SENSOR_ANALYZER4, [(64, 32, 4)], 1, 0, {}),
    ("ring", sg.SENSOR_POLARIZER, [(37, 29, 3)] * 3, 6, 0, dict(chunk_paths=1000)),
    ("ring", sg.SENSOR_NONE, [(256, 128, 8)], 3, 0, {}),  # (above the limit of one chunk)
    ("ring", sg.SENSOR_NONE, [(256, 128, 6)], 3, 0, {}),  # (the largest small call)
    ("ring", sg.SENSOR_ANALYZER4, [(128, 128, 16)], 4, 0, dict(chunk_paths=100000)),  # (a larger call in small chunks)
    ("worlds", sg.SENSOR_NONE, [(256, 256, 5)], 32, 0, {}),  # (the limit of deep plans)
    ("ring", sg.SENSOR_POLARIZER, [(64, 64, 2)], 5, 1, {}),  # (no next-event estimation)
    ("worlds", sg.SENSOR_POLARIZER, [(23, 17, 5)] * 4, 6, 0, {}),
    ("worlds", sg.SENSOR_ANALYZER4, [(40, 30, 1), (11, 7, 9)], 8, 0, {}),
    ("worlds", sg.SENSOR_NONE, [(40, 30, 2), (40, 30, 2)], 7, 0, dict(checkpoint_interval=3)),
])
def test_small_call_equals_launches_per_bounce(kind, sensor, sizes, depth, flags, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_13265_amd as ppt
    if kind == "worlds":
        sc, th = _two_worlds()
    else:
        sc = sg.config1().scene if kind == "tiny" else sg.scene2()[0]
        th = sc.slot("theta")
    params = [torch.from_numpy(p).cuda() for p in sc.params()]
    plan = ppt.Plan(ppt.Scene(sc.to_blob()), _views(kind, sensor, sizes, th), depth, flags, **kw)
    rng = np.random.default_rng(depth)
    d = rng.uniform(-0.25, 0.25, (plan.image_numel // 4, 4)).astype(np.float32)
    d[:, 0] = rng.uniform(0.5, 1.5, d.shape[0])
    d = torch.from_numpy(d.ravel()).cuda()
    mask = torch.from_numpy((rng.uniform(size=plan.num_paths) < 0.8).astype(np.uint8)).cuda()
    for m in (None, mask):
        plan.set_path_mask(m)
        got = []
        for timing in (False, True):  # (timed calls keep the launches per bounce)
            plan.set_timing(timing)
            image = plan.render(params, 23, out=torch.full((plan.image_numel,), 7.0, device="cuda"))
            counts = plan.stats(0)
            grads = plan.backward(params, 23, d)
            got.append((image, counts, plan.signatures(params, 23), grads, plan.stats(1)))
        (i0, c0, s0, g0, b0), (i1, c1, s1, g1, b1) = got
        assert torch.equal(s0, s1)
        # (a pixel whose samples span wavefronts of the reduction sums them by atomics in any order)
        assert float((i0 - i1).double().norm()) <= 4 * 2.0 ** -24 * float(i1.double().norm())
        for key in ("vertices", "paths", "rays", "shadow_rays"):
            assert c0[key] == c1[key] and b0[key] == b1[key], key
        for name, a, b in zip(sc.slot_names, g0, g1):
            a, b = a.double(), b.double()
            assert float((a - b).norm()) <= TOL * float(b.norm()), name
