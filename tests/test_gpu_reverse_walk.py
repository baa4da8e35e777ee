"""The cached backward's reverse walk (adjoint rows carried by the forward pass, one walk back) against
the hybrid replay with one block per path, which evaluates and folds the same vertices by other kernels,
at sizes where the walk's work distribution has edges: wavefronts that span views, chunks of one
wavefront, paths that all end at their first vertex, more angles than the small-slot limit, empty views."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")

# Each path contributes the same chain of about 200 FP32 operations in another order: 200 * 2^-24 = 1.2e-5
# of its share; positive weights on the intensities keep the sums from cancelling.
TOL = 1.2e-5


def _scene(kind, sensor, sizes):
    """Scene and views of the (width, height, spp) list; polarizer angles in one slot."""
    if kind == "tiny":
        sc = sg.config1().scene
        cam = ((0, 1, 6), (0, -0.5, 0), (0, 1, 0), 40.0)
    else:
        sc, _ = sg.scene2()
        cam = (sg.ring_pose(0), (0, 0, 0), (0, 1, 0), 45.0)
    th = sc.add_slot("angles", 0.1 + 0.7 * np.arange(max(len(sizes), 70)) % 3.0)
    views = [sg.make_view(0, w, h, spp, *cam, sensor, th if sensor == sg.SENSOR_POLARIZER else -1,
                          k if sensor == sg.SENSOR_POLARIZER else 0, k) for k, (w, h, spp) in enumerate(sizes)]
    return sc, np.asarray(views, sg.VIEW_DTYPE)


CASES = [
    ("tiny", sg.SENSOR_POLARIZER, [(1, 1, 1)], 3, 0),
    ("tiny", sg.SENSOR_ANALYZER4, [(13, 7, 5)], 4, 64),
    ("tiny", sg.SENSOR_NONE, [(31, 9, 3), (5, 3, 1)], 6, 128),
    ("ring", sg.SENSOR_POLARIZER, [(17, 11, 3)] * 5, 1, 0),
    ("ring", sg.SENSOR_POLARIZER, [(17, 11, 3)] * 5, 2, 192),
    ("ring", sg.SENSOR_POLARIZER, [(3, 2, 1)] * 70, 5, 0),
    ("ring", sg.SENSOR_POLARIZER, [(64, 48, 9), (33, 31, 2)], 7, 0),
    ("ring", sg.SENSOR_ANALYZER4, [(29, 23, 2), (7, 5, 33)], 5, 1000),
    ("ring", sg.SENSOR_NONE, [(40, 30, 4)], 3, 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("kind,sensor,sizes,depth,chunk", CASES)
def test_reverse_walk_equals_hybrid_replay(kind, sensor, sizes, depth, chunk):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_13265_amd as ppt
    sc, views = _scene(kind, sensor, sizes)
    scene = ppt.Scene(sc.to_blob())
    params = [torch.from_numpy(p).cuda() for p in sc.params()]
    walk = ppt.Plan(scene, views, depth, chunk_paths=chunk)
    hybrid = ppt.Plan(scene, views, depth, chunk_paths=chunk, checkpoint_interval=depth)
    rng = np.random.default_rng(depth)
    d = rng.uniform(-0.25, 0.25, (walk.image_numel // 4, 4)).astype(np.float32)
    d[:, 0] = rng.uniform(0.5, 1.5, d.shape[0])
    d = torch.from_numpy(d.ravel()).cuda()
    mask = torch.from_numpy((rng.uniform(size=walk.num_paths) < 0.9).astype(np.uint8)).cuda()
    for m in (None, mask):
        walk.set_path_mask(m)
        hybrid.set_path_mask(m)
        got = walk.backward(params, 17, d, grads=[torch.full_like(p, 7.0) for p in params])
        ref = hybrid.backward(params, 17, d)
        for name, g, r in zip(sc.slot_names, got, ref):
            g, r = g.double(), r.double()
            assert torch.isfinite(g).all(), name
            assert float((g - r).norm()) <= TOL * float(r.norm()), (name, float((g - r).norm()), float(r.norm()))


def test_index_division_by_reciprocal_is_exact():
    # n / d as floor((n + 1/2) (1/d)) in double, for the path and pixel indices below 2^31
    rng = np.random.default_rng(0)
    d = np.unique(np.concatenate([np.arange(1, 70), 2 ** np.arange(1, 31), 2 ** np.arange(2, 31) - 1,
                                  rng.integers(1, 2 ** 31, 2000), [2 ** 31 - 1]])).astype(np.int64)
    inv = 1.0 / d.astype(np.float64)
    top = (2 ** 31 - 1) // d
    for q in (np.zeros_like(d), np.ones_like(d), top // 2, top - 1, top):
        for off in (-1, 0, 1):
            n = np.clip(q * d + off, 0, 2 ** 31 - 1)
            got = np.floor((n.astype(np.float64) + 0.5) * inv).astype(np.int64)
            assert np.array_equal(got, n // d)


def _textured_ground(aw, ah, rw, rh):
    """A blended ground with an aw x ah albedo map and an rw x rh roughness map, and a first slot that can
    fill the workgroup accumulators so that the maps' gradients go to the global one."""
    rng = np.random.default_rng(aw * 1000 + ah)
    sc = sg.Scene()
    sc.add_slot("filler", np.zeros(12800, np.float32))
    s_alb = sc.add_slot("albedo", rng.uniform(0.2, 0.8, aw * ah * 3))
    s_rgh = sc.add_slot("rough", rng.uniform(0.2, 0.6, rw * rh))
    s_ior = sc.add_slot("ior", [1.5])
    s_le = sc.add_slot("Le", [5.0, 4.0, 3.0])
    w = sc.add_world()
    m = w.add_material(type=sg.MAT_BLEND, albedo_slot=s_alb, albedo_tw=aw, albedo_th=ah, alpha_slot=s_rgh,
                       alpha_tw=rw, alpha_th=rh, eta_slot=s_ior, blend=0.5)
    w.add_quad((-4, 0, -4), (0, 0, 8), (8, 0, 0), m)
    w.add_quad((-4, 0, -4), (8, 0, 0), (0, 4, 0), m)
    w.add_light((-1, 5, -1), (2, 0, 0), (0, 0, 2), s_le)
    return sc


@pytest.mark.gpu
@pytest.mark.parametrize("sensor", [sg.SENSOR_POLARIZER, sg.SENSOR_ANALYZER4])
@pytest.mark.parametrize("aw,ah,rw,rh,spp", [(1, 37, 90, 1, 3), (29, 1, 9, 8, 64), (16, 16, 11, 7, 1), (64, 64, 64, 64, 32)])
def test_staged_texture_scatter_equals_workgroup_accumulators(aw, ah, rw, rh, spp, sensor):
    """Texture gradients through the staged scatter into the global accumulator (clamped, one-texel-wide and
    tiny maps; lone lanes, groups and whole wavefronts per texel cell) against the same gradients asked for
    alone, which the workgroup accumulators take in FP32: up to 2^14 additions of one sign per texel, whose
    rounding averages to sqrt(2^14) 2^-24 = 8e-6 of the sum."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_13265_amd as ppt
    sc = _textured_ground(aw, ah, rw, rh)
    th = sc.add_slot("theta", [0.4])
    views = np.asarray([sg.make_view(0, 41, 23, spp, (0, 2.5, 6), (0, 0.5, 0), (0, 1, 0), 50.0, sensor,
                                     th if sensor == sg.SENSOR_POLARIZER else -1, 0, 3)], sg.VIEW_DTYPE)
    plan = ppt.Plan(ppt.Scene(sc.to_blob()), views, 4)
    params = [torch.from_numpy(p).cuda() for p in sc.params()]
    d = torch.zeros(plan.image_numel, device="cuda")
    d[::4] = 1.0
    staged = plan.backward(params, 5, d, want=[True] * len(params))
    assert float(staged[0].abs().max()) == 0.0
    for name in ("albedo", "rough"):
        k = sc.slot(name)
        alone = plan.backward(params, 5, d, want=[i == k for i in range(len(params))])[k].double()
        assert float((staged[k].double() - alone).norm()) <= 8e-6 * float(alone.norm()), name
