"""The pixel reduction's stores of whole pixels against its additions, which an image that does not lie on 16 bytes
takes for every pixel, for both forms of its scan (three scalars; twelve Stokes words)."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sensor", [sg.SENSOR_NONE, sg.SENSOR_POLARIZER, sg.SENSOR_ANALYZER4])
@pytest.mark.parametrize("spp", [1, 3, 15, 16, 17, 64, 65, 200])
def test_stored_pixels_equal_added_pixels(sensor, spp):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_13265_amd as ppt
    sc = sg.config1().scene
    params = [torch.from_numpy(p).cuda() for p in sc.params()]
    theta = sc.slot("theta") if sensor == sg.SENSOR_POLARIZER else -1
    views = np.asarray([sg.make_view(0, w, h, spp, (0, 1, 6), (0, -0.5, 0), (0, 1, 0), 40.0, sensor, theta, 0, k)
             for k, (w, h) in enumerate([(13, 7), (1, 1), (32, 9)])], sg.VIEW_DTYPE)
    plan = ppt.Plan(ppt.Scene(sc.to_blob()), views, 3)
    stored = plan.render(params, 5, out=torch.full((plan.image_numel,), 7.0, device="cuda"))
    added = plan.render(params, 5, out=torch.full((plan.image_numel + 1,), 7.0, device="cuda")[1:])
    # the same sums; those of a pixel that spans wavefronts are added in any order
    a, b = stored.double(), added.double()
    assert float(b.abs().max()) > 0.0
    assert float((a - b).norm()) <= 4 * 2.0 ** -24 * float(b.norm())
