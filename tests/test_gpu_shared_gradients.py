"""Gradients of small calls whose additions meet in few addresses: constants packed in one slot, small maps, maps of
which little is in view.  The same values as the launches per bounce (which per-kernel timing keeps) give, and in no
more time than those take."""
import time

import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the workgroup accumulators add in FP32: 2^14 additions of one sign to an address, whose rounding averages to
# sqrt(2^14) 2^-24 = 8e-6 of the sum
TOL = 8e-6


def _scene(kind, size):
    """A floor, a wall and 20 quads with one blended material.  packed: its constants, and the light's, at the end of
    one slot of `size` values; map: albedo and roughness maps of size x size; full: the same behind a slot that
    fills the workgroup accumulators (none is left for the maps)."""
    rng = np.random.default_rng(size)
    sc = sg.Scene()
    kw = dict(type=sg.MAT_BLEND, blend=0.5)
    if kind == "packed":
        v = rng.uniform(0.2, 0.8, size)
        v[-8:] = (0.6, 0.5, 0.4, 0.3, 1.5, 5.0, 4.0, 3.0)
        s = sc.add_slot("all", v)
        kw.update(albedo_slot=s, albedo_off=size - 8, alpha_slot=s, alpha_off=size - 5, eta_slot=s, eta_off=size - 4)
        light = (s, size - 3)
    else:
        if kind == "full":
            sc.add_slot("filler", np.zeros(12800, np.float32))
        kw.update(albedo_slot=sc.add_slot("albedo", rng.uniform(0.2, 0.8, max(size * size * 3, 65))), albedo_tw=size, albedo_th=size,
                  alpha_slot=sc.add_slot("rough", rng.uniform(0.2, 0.6, max(size * size, 65))), alpha_tw=size, alpha_th=size,
                  eta_slot=sc.add_slot("ior", [1.5]))
        light = (sc.add_slot("Le", [5.0, 4.0, 3.0]), 0)
    w = sc.add_world()
    m = w.add_material(**kw)
    w.add_quad((-4, 0, -4), (0, 0, 8), (8, 0, 0), m)
    w.add_quad((-4, 0, -4), (8, 0, 0), (0, 4, 0), m)
    for _ in range(20):
        w.add_quad(rng.uniform((-3, 0, -3), (3, 2, 2)), rng.normal(size=3) * 0.6, rng.normal(size=3) * 0.6, m)
    w.add_light((-1, 5, -1), (2, 0, 0), (0, 0, 2), *light)
    return sc


def _plan(sc, width, height, spp, depth, **kw):
    import paper_2607_13265_amd as ppt
    views = np.asarray([sg.make_view(0, width, height, spp, (0, 2.5, 6), (0, 0.5, 0), (0, 1, 0), 50.0, sg.SENSOR_NONE, -1, 0, 3)],
                       sg.VIEW_DTYPE)
    plan = ppt.Plan(ppt.Scene(sc.to_blob()), views, depth, **kw)
    plan.set_stats(False)
    d = torch.zeros(plan.image_numel, device="cuda")
    d[::4] = 1.0
    return plan, [torch.from_numpy(p).cuda() for p in sc.params()], d


@pytest.mark.parametrize("noalloc,depth", [(False, 4), (True, 4), (False, 3)])
@pytest.mark.parametrize("kind,size,width,height,spp", [
    ("packed", 65, 31, 33, 1), ("packed", 300, 64, 65, 4), ("packed", 12800, 33, 62, 1), ("packed", 12801, 32, 64, 1),
    ("packed", 12801, 49, 41, 12), ("map", 1, 31, 7, 3), ("map", 5, 64, 48, 12), ("map", 56, 37, 29, 9), ("full", 4, 32, 64, 1),
    ("full", 8, 64, 64, 2), ("full", 8, 64, 65, 2), ("full", 40, 33, 27, 8), ("map", 100, 41, 23, 8),
    # (wavefronts of 32 paths in a walk of depth 3 and 8,193 paths, larger ones from 98,305 on: 33, 63 and 64 paths)
    ("map", 100, 1, 8192, 1), ("map", 100, 8193, 1, 1),
    ("map", 100, 1, 98305, 1), ("map", 100, 293, 11, 60), ("map", 100, 128, 128, 12)])
def test_small_call_gradients_equal_launches_per_bounce(kind, size, width, height, spp, noalloc, depth):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sc = _scene(kind, size)
    plan, params, d = _plan(sc, width, height, spp, depth)

    def run(grads):
        return plan.backward_noalloc(params, 5, d, grads) if noalloc else plan.backward(params, 5, d, grads=grads)

    got = run([torch.full_like(p, 7.0) for p in params])
    plan.set_timing(True)
    ref = run([torch.full_like(p, 7.0) for p in params])
    for name, g, r in zip(sc.slot_names, got, ref):
        g, r = g.double(), r.double()
        assert torch.isfinite(g).all(), name
        assert name == "filler" or float(r.norm()) > 0.0, name
        assert float((g - r).norm()) <= TOL * float(r.norm()), (name, float((g - r).norm()), float(r.norm()))


@pytest.mark.parametrize("kind,size,width,height,spp", [("packed", 100, 128, 128, 12), ("map", 5, 128, 128, 12),
                                                        ("packed", 20000, 128, 128, 4), ("full", 5, 128, 128, 12)])
def test_shared_addresses_cost_no_more_than_launches_per_bounce(kind, size, width, height, spp):
    """Additions to one address pass one after the other: with every vertex adding to the global accumulator such
    calls took 1.6 to 13 times the launches per bounce.  Here both take about the same, or the small call half; the
    limit leaves 30 % for the clock."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    plan, params, d = _plan(_scene(kind, size), width, height, spp, 2)
    grads = [torch.empty_like(p) for p in params]
    took = {False: [], True: []}
    for rep in range(12):
        for timing in (False, True):
            plan.set_timing(timing)
            plan.backward(params, 5, d, grads=grads)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                plan.backward(params, 5, d, grads=grads)
            torch.cuda.synchronize()
            if rep >= 2:
                took[timing].append(time.perf_counter() - t0)
    small, per_bounce = float(np.median(took[False])), float(np.median(took[True]))
    assert small <= 1.3 * per_bounce, (small, per_bounce)
