"""The launches per bounce (large calls), which small sizes reach under per-kernel timing: the walk's two kernels against
the hybrid replay and against each other's accumulators, traversal without work counters, rank-one and full records,
chunks, and graph replay of a call above the size limit of small ones."""
import numpy as np
import pytest

import scenegen as sg
from parity import rel
from test_gpu_reverse_walk import CASES, TOL, _scene, _textured_ground

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _ppt():
    import paper_2607_13265_amd as ppt
    return ppt


def _params(scene):
    return [torch.from_numpy(p).cuda() for p in scene.params()]


def _batch(n_views=6, res=24, spp=4):
    wl = sg.config3(res=res, spp=spp, n_angles=3, n_poses=2)
    wl.views = wl.views[:n_views]
    return wl


def _plan(scene, views, depth, timing=True, **kw):
    plan = _ppt().Plan(scene, views, depth, **kw)
    plan.set_timing(timing)
    return plan


@pytest.mark.parametrize("kind,sensor,sizes,depth,chunk", CASES)
def test_walk_equals_hybrid_replay(kind, sensor, sizes, depth, chunk):
    sc, views = _scene(kind, sensor, sizes)
    scene = _ppt().Scene(sc.to_blob())
    params = _params(sc)
    walk = _plan(scene, views, depth, chunk_paths=chunk)
    hybrid = _plan(scene, views, depth, chunk_paths=chunk, checkpoint_interval=depth)
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
        t = walk.kernel_times(1)
        assert t["replay"][1] > 0 and (depth == 1 or t["fold"][1] > 0)  # (the walk's two kernels ran)
        for name, g, r in zip(sc.slot_names, got, ref):
            g, r = g.double(), r.double()
            assert torch.isfinite(g).all(), name
            assert float((g - r).norm()) <= TOL * float(r.norm()), (name, float((g - r).norm()), float(r.norm()))


@pytest.mark.parametrize("sensor", [sg.SENSOR_POLARIZER, sg.SENSOR_ANALYZER4])
@pytest.mark.parametrize("aw,ah,rw,rh,spp", [(1, 37, 90, 1, 3), (29, 1, 9, 8, 64), (16, 16, 11, 7, 1), (64, 64, 64, 64, 32)])
def test_staged_and_grouped_scatter_equals_workgroup_accumulators(aw, ah, rw, rh, spp, sensor):
    """Every gradient at once (the maps' through groups of coherent lanes and the staged scatter, their workgroup
    accumulator being full), and each map's alone (in workgroup accumulators), per bounce and as a small call: four
    results of the same additions, up to 2^14 of one sign per texel in FP32 (sqrt(2^14) 2^-24 = 8e-6 of the sum)."""
    sc = _textured_ground(aw, ah, rw, rh)
    th = sc.add_slot("theta", [0.4])
    views = np.asarray([sg.make_view(0, 41, 23, spp, (0, 2.5, 6), (0, 0.5, 0), (0, 1, 0), 50.0, sensor,
                                     th if sensor == sg.SENSOR_POLARIZER else -1, 0, 3)], sg.VIEW_DTYPE)
    plan = _ppt().Plan(_ppt().Scene(sc.to_blob()), views, 4)
    params = _params(sc)
    d = torch.zeros(plan.image_numel, device="cuda")
    d[::4] = 1.0
    for name in ("albedo", "rough"):
        k = sc.slot(name)
        got = []
        for timing in (True, False):
            plan.set_timing(timing)
            got.append(plan.backward(params, 5, d, want=[i == k for i in range(len(params))])[k].double())
            got.append(plan.backward(params, 5, d, want=[True] * len(params))[k].double())
        assert float(got[0].norm()) > 0.0
        for g in got[1:]:
            assert float((g - got[0]).norm()) <= 8e-6 * float(got[0].norm()), name


@pytest.mark.parametrize("sensor", [sg.SENSOR_POLARIZER, sg.SENSOR_NONE])
@pytest.mark.parametrize("kw", [{}, dict(checkpoint_interval=3), dict(pprb_sigma=0.05), dict(tape=True), dict(prb=True)])
def test_traversal_without_work_counters_matches(sensor, kw):
    wl = _batch()
    wl.views["sensor"] = sensor
    params = _params(wl.scene)
    plan = _plan(_ppt().Scene(wl.scene.to_blob()), wl.views, wl.max_depth, chunk_paths=4096, **kw)
    d = torch.ones(plan.image_numel, device="cuda")
    got = []
    for counters in (True, False):
        plan.set_stats(counters)
        got.append((plan.render(params, 13), plan.backward(params, 13, d)))
        if counters:
            assert plan.stats(0)["nodes"] > 0 and plan.stats(1)["nodes"] > 0
    (i0, g0), (i1, g1) = got
    assert float(i0.norm()) > 0.0 and float((i0 - i1).norm()) <= 1e-6 * float(i0.norm())
    for a, b in zip(g0, g1):  # (the same additions in any order: sums of one sign up to the noise of the comparators)
        assert float((a.double() - b.double()).norm()) <= 1e-5 * max(float(a.double().norm()), 1e-30)


def test_rank_one_render_equals_full_render():
    wl = _batch(n_views=4)
    scene = _ppt().Scene(wl.scene.to_blob())
    params = _params(wl.scene)
    extra = wl.views[:1].copy()
    extra["sensor"] = sg.SENSOR_NONE
    extra["view_id"] = 999
    a = _plan(scene, wl.views, wl.max_depth).render(params, 21).double().cpu().numpy()
    b = _plan(scene, np.concatenate([wl.views, extra]), wl.max_depth).render(params, 21).double().cpu().numpy()[:a.size]
    a4, b4 = a.reshape(-1, 4), b.reshape(-1, 4)
    assert np.abs(b4).max() > 0 and np.abs(a4[:, 3]).max() == 0.0 and np.abs(b4[:, 3]).max() == 0.0
    for k in range(3):
        assert np.linalg.norm(a4[:, k] - b4[:, k]) <= 1e-5 * np.linalg.norm(b4[:, k]), k


def test_batched_equals_per_view_and_chunk_invariance():
    wl = _batch()
    scene = _ppt().Scene(wl.scene.to_blob())
    params = _params(wl.scene)
    plan = _plan(scene, wl.views, wl.max_depth)
    img = plan.render(params, 11)
    d = torch.randn(plan.image_numel, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    g = plan.backward(params, 11, d)
    offs = sg.view_offsets(wl.views)
    gsum = [torch.zeros_like(p) for p in params]
    for v in range(len(wl.views)):
        pv = _plan(scene, wl.views[v:v + 1], wl.max_depth)
        o = int(offs[v])
        assert torch.equal(pv.render(params, 11), img[o:o + pv.image_numel])
        for a, b in zip(gsum, pv.backward(params, 11, d[o:o + pv.image_numel].contiguous())):
            a += b
    pc = _plan(scene, wl.views, wl.max_depth, chunk_paths=1000)
    assert pc.launch_info()["n_chunks"] > 1
    assert rel(pc.render(params, 11).cpu().numpy(), img.cpu().numpy()) < 1e-6
    for a, b, c in zip(gsum, g, pc.backward(params, 11, d)):
        assert rel(a.cpu().numpy(), b.cpu().numpy(), floor=1e-12) < 1e-5
        assert rel(c.cpu().numpy(), b.cpu().numpy(), floor=1e-12) < 1e-5


@pytest.mark.parametrize("sensor", [sg.SENSOR_POLARIZER, sg.SENSOR_NONE])
def test_graph_replay_of_a_large_call_matches_eager(sensor):
    wl = _batch(n_views=3, res=144, spp=4)  # 248,832 paths: above the limit of small calls
    wl.views["sensor"] = sensor
    plan = _ppt().Plan(_ppt().Scene(wl.scene.to_blob()), wl.views, wl.max_depth)
    assert plan.num_paths > 3 << 16
    plan.set_stats(False)
    params = _params(wl.scene)
    d = torch.ones(plan.image_numel, device="cuda")
    out = torch.empty(plan.image_numel, device="cuda")
    grads = [torch.empty_like(p) for p in params]
    ws0, ws1 = plan.workspace(0), plan.workspace(1)

    def step():
        plan.render(params, 5, out=out, ws=ws0)
        plan.backward(params, 5, d, grads=grads, ws=ws1)

    step()
    torch.cuda.synchronize()
    ref_img, ref_g = out.clone(), [x.clone() for x in grads]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for r in range(3):
        out.fill_(7.0)
        for x in grads:
            x.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref_img), r
        for a, b in zip(grads, ref_g):
            assert rel(a.cpu().numpy(), b.cpu().numpy(), floor=1e-12) < 1e-5
        _ = plan.render(params, 6)  # eager work between replays
        torch.cuda.synchronize()
