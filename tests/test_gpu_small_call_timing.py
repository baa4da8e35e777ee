"""Per-kernel timing of the launches that an untimed call makes (set_timing(2)): a small call's whole-path launch and its
walk, one of each a chunk, where set_timing(True) times launches per bounce; a large call's launches either way."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small,kw", [(True, {}), (True, dict(chunk_paths=1024)), (True, dict(checkpoint_interval=2)), (False, {})])
def test_timing_of_the_launches_that_run(small, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_13265_amd as ppt
    wl = sg.config1()
    w, h, spp = (37, 29, 3) if small else (256, 256, 4)  # (262,144 paths: above the limit of small calls)
    views = np.asarray([sg.make_view(0, w, h, spp, (0, 1, 6), (0, -0.5, 0), (0, 1, 0), 40.0, sg.SENSOR_NONE, -1, 0, 3)], sg.VIEW_DTYPE)
    plan = ppt.Plan(ppt.Scene(wl.scene.to_blob()), views, 4, **kw)
    params = [torch.from_numpy(p).cuda() for p in wl.scene.params()]
    d = torch.ones(plan.image_numel, device="cuda")
    chunks = plan.launch_info()["n_chunks"]
    times = {}
    for mode in (1, 2):
        plan.set_timing(mode)
        plan.render(params, 5)
        plan.backward(params, 5, d)
        times[mode] = [{f: n for f, (ms, n) in plan.kernel_times(op).items()} for op in (0, 1)]
        assert all(ms >= 0.0 for op in (0, 1) for ms, _ in plan.kernel_times(op).values())
    for op in (0, 1):
        per_bounce, runs = times[1][op], times[2][op]
        assert per_bounce["extend"] == per_bounce["shade"] == per_bounce["compact"] == 4 * chunks
        if small:
            assert runs["extend"] == chunks and runs["shade"] == runs["compact"] == 0
            assert runs["accum"] == (chunks if op == 0 else 0) and runs["replay"] == (0 if op == 0 else chunks)
            assert runs["fold"] == (chunks if op == 1 and kw.get("checkpoint_interval") else 0)
        else:
            assert runs == per_bounce
