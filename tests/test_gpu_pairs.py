"""The light effects' pairs found from marks, against what evaluates every
density: the window reuse against the row tasks, which a list of one light
takes, and the validation bits against the work-counting walk; for lights that
mark few and many receivers of a candidate, near and far, turned and oblong, in
frames with cut tiles and pixels without a surface."""
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


def _frame(light, size):
    scene = w.boxes_scene(1)
    gb = w.render_gbuffer(scene, w.boxes_camera(*size))
    c, eu, ev = (np.array(v, np.float32) for v in LIGHTS[light])
    lt = w.RectLight(c, eu, ev)
    if np.cross(eu, ev)[1] > 0:  # (emitting upwards)
        lt = w.RectLight(c, ev, eu)
    return scene, gb, lt


# (333 x 197 runs eight waves to a tile, 1367 x 771 four)
@pytest.mark.parametrize("size", [(333, 197), (1367, 771)])
@pytest.mark.parametrize("light", sorted(LIGHTS))
def test_pairs_equal_row_tasks(light, size):
    import torch
    import paper_2607_23122_amd as ocr
    scene, gb, lt = _frame(light, size)
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


@pytest.mark.parametrize("size", [(61, 37), (333, 197)])
@pytest.mark.parametrize("light", sorted(LIGHTS))
def test_marked_bits_equal_counted(light, size):
    import torch
    import paper_2607_23122_amd as ocr
    scene, gb, lt = _frame(light, size)
    bvh = ocr.build_bvh(scene.V, scene.F)
    dg = ocr.DeviceGBuffer.from_host(gb)
    occ = ocr.trace_occluders(bvh, dg, "shadow", 1.0, lt, 5, 0)
    n = size[0] * size[1]
    for radius in (1, 2, 3):
        log(f"[pairs] bits {light} {size} window {radius}")
        p = ocr.reuse_params("window", radius, 8, "unbiased")
        words = ((4 * radius + 1) ** 2 + 31) // 32
        bits = []
        # one light, a list of it (and of it twice), the counting walk
        for lights, stats in ((lt, None), ([lt], None), ([lt, lt], None), (lt, torch.zeros(5, dtype=torch.int64, device="cuda"))):
            ws = torch.zeros(ocr.workspace_bytes(gb.width, gb.height, p), dtype=torch.uint8, device="cuda")
            ocr.validate_pairs(bvh, dg, occ, "shadow", 1.0, lights, p, ws, stats=stats)
            bits.append(ws.cpu().numpy()[:4 * n * words].view(np.uint32).reshape(n, words))
        cand = (occ.hit_u32() < 0xFFFFFFFE).ravel()
        assert cand.any()
        for b in bits[:-1]:
            assert np.array_equal(b[cand], bits[-1][cand])


# Which body sums a candidate is chosen by its marks alone, so a frame can be sent
# through the row tasks: marks that carry a density of zero (the pairs that even
# without occluders have none) change no sum, and candidates with that many marks
# are left to them.
_EFFECTS = ["shadow", "bilinear", "solid_angle", "solid_angle_bilinear", "direct", "lights"]


def _reuse(ocr, effect, dg, occ, lt, p, ws=None, bvh=None):
    import torch
    out = torch.empty((dg.height, dg.width), device="cuda")
    if effect in ("shadow", "bilinear", "lights"):
        ocr.reuse_shadow(bvh, dg, occ, lt, p, out, ws)
    elif effect.startswith("solid_angle"):
        ocr.reuse_shadow_solid_angle(bvh, dg, occ, lt, p, out, ws)
    else:
        ocr.reuse_direct_illumination(bvh, dg, occ, lt, p, 100.0, 0.8, out, ws)
    return out.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("effect", _EFFECTS)
@pytest.mark.parametrize("light,size", [("near", (61, 37)), ("near", (333, 197)), ("oblong", (333, 197)),
                                        ("large", (333, 197)), ("far", (1367, 771))])
def test_pair_body_equals_row_tasks_to_the_bit(light, size, effect):
    import copy
    import torch
    import paper_2607_23122_amd as ocr
    scene, gb, lt = _frame(light, size)
    if effect.endswith("bilinear"):
        lt = copy.copy(lt)
        lt.pdf = 1
    uniform = copy.copy(lt)
    uniform.pdf = 0
    if effect == "lights":
        second = w.RectLight(lt.center + np.float32([3, 0.5, 1]), lt.edge_u, lt.edge_v)
        lt = uniform = [lt, second]
    bvh = ocr.build_bvh(scene.V, scene.F)
    # no occluder near any segment
    away = ocr.build_bvh(np.array([[0, -900, 0], [1, -900, 0], [0, -900, 1]], np.float32), np.array([[0, 1, 2]], np.uint32))
    dg = ocr.DeviceGBuffer.from_host(gb)
    occ = ocr.trace_occluders(bvh, dg, "shadow", 1.0, lt, 5, 0)
    n = size[0] * size[1]
    cand = (occ.hit_u32() < 0xFFFFFFFE).ravel()
    for radius in (1, 2, 3):
        log(f"[pairs] rows {light} {size} {effect} window {radius}")
        p = ocr.reuse_params("window", radius, 8, "unbiased", validated=True)
        words = ((4 * radius + 1) ** 2 + 31) // 32

        def bits_of(hierarchy):
            ws = torch.zeros(ocr.workspace_bytes(gb.width, gb.height, p), dtype=torch.uint8, device="cuda")
            ocr.validate_pairs(hierarchy, dg, occ, "shadow", 1.0, uniform, p, ws)
            return ws

        true, every = bits_of(bvh), bits_of(away)
        full = (1 << (4 * radius + 1) ** 2) - 1
        mask = np.array([(full >> (32 * i)) & 0xFFFFFFFF for i in range(words)], np.uint32)
        # biased: every mark set, so each candidate takes the row tasks
        biased = ocr.reuse_params("window", radius, 8, "biased", dark_guard=False)
        marked = true.clone()
        marked.view(torch.int32)[:n * words] = torch.from_numpy(np.tile(mask, n).view(np.int32)).cuda()
        assert np.array_equal(_reuse(ocr, effect, dg, occ, lt, biased),
                              _reuse(ocr, effect, dg, occ, lt, p, marked, bvh))
        # unbiased: the pairs without a density marked besides
        b = true.cpu().numpy()[:4 * n * words].view(np.uint32).reshape(n, words)
        e = every.cpu().numpy()[:4 * n * words].view(np.uint32).reshape(n, words)
        both = b | (mask & ~e)
        few = np.unpackbits(b[cand].view(np.uint8), axis=1).sum(1) <= 4 * radius
        log(f"    candidates {int(cand.sum())}, with few pairs {int(few.sum())}, of these moved "
            f"{int((np.unpackbits(both[cand][few].view(np.uint8), axis=1).sum(1) > 4 * radius).sum())}")
        moved = true.clone()
        moved.view(torch.int32)[:n * words] = torch.from_numpy(both.view(np.int32).ravel().copy()).cuda()
        assert np.array_equal(_reuse(ocr, effect, dg, occ, lt, p, true, bvh), _reuse(ocr, effect, dg, occ, lt, p, moved, bvh))
