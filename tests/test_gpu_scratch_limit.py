"""The allocation-free backward at the end of its fixed scratch: a call whose records and gradient accumulators just
filled it before the queue sizes and work counters had cache lines of their own is still taken, one that did not fit
is still refused."""
import re

import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SCRATCH = 64 << 20
TOL = 1.2e-5  # about 200 FP32 operations of a path's share in another order: 200 * 2^-24


def _scene(stage, filler):
    sc = sg.scene_lightstage(tex=8) if stage else sg.config1().scene
    sc = sc[0] if isinstance(sc, tuple) else sc
    sc.add_slot("filler", np.zeros(filler, np.float32))
    return sc


@pytest.mark.parametrize("mode,stage,kw", [
    ("cached", True, {}), ("hybrid", False, dict(checkpoint_interval=2)), ("rule", False, dict(checkpoint_interval=3, hybrid_rule=(0.5, 1e-3))),
    ("pprb", False, dict(pprb_sigma=0.05)), ("tape", False, dict(tape=True)), ("prb", False, dict(prb=True))])
def test_scratch_limit(mode, stage, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_13265_amd as ppt
    if stage:
        views = sg.lightstage(res=9, spp=1, n_views=1).views
    else:
        views = np.asarray([sg.make_view(0, 13, 7, 2, (0, 1, 6), (0, -0.5, 0), (0, 1, 0), 40.0, sg.SENSOR_NONE, -1, 0, 3)], sg.VIEW_DTYPE)

    def make(filler):
        sc = _scene(stage, filler)
        params = [torch.from_numpy(p).cuda() for p in sc.params()]
        plan = ppt.Plan(ppt.Scene(sc.to_blob()), views, 3, **kw)
        return sc, params, plan, torch.ones(plan.image_numel, device="cuda")

    def need(filler):  # (from the refusal of a far larger call)
        sc, params, plan, d = make(filler)
        with pytest.raises(ppt.PPTError, match="PPT_EUNSUPPORTED") as e:
            plan.backward_noalloc(params, 5, d, [torch.empty_like(p) for p in params])
        return int(re.search(r"\((\d+) bytes needed\)", str(e.value)).group(1))

    big = 9 << 20
    over = need(big) - SCRATCH  # in steps of 256 bytes: 32 values
    # the counters took 256 bytes, and now take 6,912 (twice for the sub-paths of P-RB)
    grown = (2 if mode == "prb" else 1) * (6912 - 256)
    for extra, taken in ((0, True), (256, True), (grown, True), (grown + 256, False)):
        sc, params, plan, d = make(big - (over - extra) // 8)
        got = [torch.full_like(p, 7.0) for p in params]
        if not taken:
            with pytest.raises(ppt.PPTError, match="PPT_EUNSUPPORTED"):
                plan.backward_noalloc(params, 5, d, got)
            continue
        plan.backward_noalloc(params, 5, d, got)
        ref = plan.backward(params, 5, d)
        for name, g, r in zip(sc.slot_names, got, ref):
            g, r = g.double(), r.double()
            assert torch.isfinite(g).all(), name
            assert float((g - r).norm()) <= TOL * float(r.norm()), (extra, name)
