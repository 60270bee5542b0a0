"""Each of the kernels between which a frame's size, radius and mesh choose, on
the same frames: the same records and bits as the counting walks'."""
import numpy as np
import pytest

import oracle
import workloads as w
from gpu_util import COLLECT, NEAR_FIRST, SHAFT, WALK, bvh_field, log, route

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ocr():
    import paper_2607_23122_amd as m
    return m


def _frame(ocr, scene, size):
    sc, cam, R = (w.terrain_scene(2, 96, 70), w.terrain_camera(*size), 2.0) if scene == "terrain" else \
        (w.boxes_scene(3), w.boxes_camera(*size), 1.0)
    return ocr.build_bvh(sc.V, sc.F), ocr.DeviceGBuffer.from_host(w.render_gbuffer(sc, cam)), R


def test_extent_is_the_lower_quartile(ocr):
    sc = w.boxes_scene(3)
    T = sc.V[sc.F]
    side = (T.max(1) - T.min(1)).max(1)
    bvh = ocr.build_bvh(sc.V, sc.F)
    assert bvh_field(bvh, "extent").value == np.sort(side)[len(side) // 4]
    # one triangle, and triangles without extent (never "short" rays)
    V = np.array([[0, 0, 0], [0, 0, 3], [1, 0, 0]], np.float32)
    assert bvh_field(ocr.build_bvh(V, np.array([[0, 1, 2]], np.uint32)), "extent").value == 3.0
    assert bvh_field(ocr.build_bvh(V, np.array([[0, 0, 0]], np.uint32)), "extent").value == 0.0


@pytest.mark.parametrize("R", [0.5, 2.0, 40.0, 1e6])
@pytest.mark.parametrize("scene,size", [("boxes", (97, 73)), ("terrain", (161, 93))])
def test_ao_trace_routes_equal_counted(ocr, scene, size, R):
    import torch
    bvh, dg, _ = _frame(ocr, scene, size)
    log(f"[routes] trace {scene} {size} R={R}")
    stats = torch.zeros(5, dtype=torch.int64, device="cuda")
    ref = ocr.trace_occluders_counted(bvh, dg, stats, "ao", R, None, 3, 1)
    hit = ref.hit_u32()
    m = hit < oracle.SELF
    assert m.any()
    p = ocr.reuse_params("window", 2, 8, "biased")
    plain = None
    for r in (NEAR_FIRST, COLLECT):
        with route(bvh, **r):
            occ = ocr.trace_occluders(bvh, dg, "ao", R, None, 3, 1)
            img = torch.empty((dg.height, dg.width), device="cuda")
            plan = ocr.Plan([ocr.view_desc(bvh, dg, img, "ao", R, None, 3, 1, p)], ocr.plan_tuning((8, 8), "block8"))
            plan.launch()
            torch.cuda.synchronize()
        assert np.array_equal(occ.hit_u32(), hit)
        for a, b in ((occ.dz, ref.dz), (occ.nz, ref.nz)):
            assert np.array_equal(a.cpu().numpy()[m].view(np.uint32), b.cpu().numpy()[m].view(np.uint32))
        plain = ocr.reuse_ao(None, dg, occ, R, p) if plain is None else plain
        assert torch.equal(img, plain)


# (above 2^17 pixels only the mesh and the radius choose)
@pytest.mark.parametrize("scene,size", [("boxes", (97, 73)), ("terrain", (161, 93)), ("boxes", (640, 360)),
                                        ("terrain", (640, 360))])
@pytest.mark.parametrize("radius", [1, 2, 3, 5])
def test_ao_validation_routes_equal_counted(ocr, scene, size, radius):
    import torch
    bvh, dg, R = _frame(ocr, scene, size)
    log(f"[routes] validate {scene} {size} radius {radius}")
    occ = ocr.trace_occluders(bvh, dg, "ao", R, None, 5, 0)
    cand = (occ.hit_u32() < oracle.SELF).ravel()
    p = ocr.reuse_params("window", radius, 8, "unbiased")
    words = ((4 * radius + 1) ** 2 + 31) // 32
    bits = []
    for r, count in ((SHAFT, False), (WALK, False), ({}, True)):
        ws = torch.zeros(ocr.workspace_bytes(dg.width, dg.height, p), dtype=torch.uint8, device="cuda")
        stats = torch.zeros(5, dtype=torch.int64, device="cuda") if count else None
        with route(bvh, **r):
            ocr.validate_pairs(bvh, dg, occ, "ao", R, None, p, ws, stats=stats)
            torch.cuda.synchronize()
        n = dg.width * dg.height
        bits.append(ws.cpu().numpy()[:4 * n * words].view(np.uint32).reshape(n, words)[cand])
    assert len(bits[0]) and int(stats[4]) > 0
    for b in bits[:2]:
        assert np.array_equal(b, bits[2])
