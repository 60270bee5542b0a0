"""The window reuse of one light's records pair by pair against the row tasks,
which a list of one light takes: the same estimates, for lights that mark few
and many receivers of a candidate, near and far, turned and oblong, in frames
with cut tiles and pixels without a surface."""
import numpy as np
import pytest

import workloads as w
from gpu_util import log

pytestmark = pytest.mark.gpu

# centre, edges (emitting towards the receivers)
LIGHTS = {
    "far": ((0.5, 40.0, 3.0), (1.0, 0.0, 0.5), (-0.5, 0.0, 1.0)),
    "oblong": ((0.0, 6.0, 0.0), (9.0, 0.0, 1.0), (-0.03125, 0.0, 0.28125)),
    "near": ((0.3, 1.6, 0.2), (0.8, 0.3, 0.0), (0.0, 0.0, 0.9)),
    "large": ((0.0, 5.0, 0.0), (24.0, 0.0, 0.0), (0.0, 0.0, 24.0)),
}


# (333 x 197 runs eight waves to a tile, 1367 x 771 four)
@pytest.mark.parametrize("size", [(333, 197), (1367, 771)])
@pytest.mark.parametrize("light", sorted(LIGHTS))
def test_pairs_equal_row_tasks(light, size):
    import torch
    import paper_2607_23122_amd as ocr
    scene = w.boxes_scene(1)
    gb = w.render_gbuffer(scene, w.boxes_camera(*size))
    c, eu, ev = (np.array(v, np.float32) for v in LIGHTS[light])
    lt = w.RectLight(c, eu, ev)
    if np.cross(eu, ev)[1] > 0:  # (emitting upwards)
        lt = w.RectLight(c, ev, eu)
    bvh = ocr.build_bvh(scene.V, scene.F)
    dg = ocr.DeviceGBuffer.from_host(gb)
    occ = ocr.trace_occluders(bvh, dg, "shadow", 1.0, lt, 5, 0)
    for radius in (1, 2, 3):
        log(f"[pairs] {light} {size} window {radius}")
        p = ocr.reuse_params("window", radius, 8, "biased")
        a = ocr.reuse_shadow(bvh, dg, occ, lt, p).cpu().numpy()
        b = ocr.reuse_shadow(bvh, dg, occ, [lt], p).cpu().numpy()
        torch.cuda.synchronize()
        assert (np.abs(a) > 0).mean() > 0.05
        # B is bitwise the same; the unshadowed term of a list is a weighted mean
        # of the one light's (a product and a division: two roundings of a number
        # up to 1)
        assert np.abs(a - b).max() <= 2.0 ** -22
