"""The frame walks against the work-counting ones, which visit the hierarchy
from the root in another order: the same records and validation bits, on
scenes where the walks' tables fill up."""
import numpy as np
import pytest

import oracle
import workloads as w
from gpu_util import log

pytestmark = pytest.mark.gpu


def _soup(n, spread, seed):
    """n random triangles of size ~spread around the origin, and a receiver
    grid plane at y = 0 of 67 x 45 points facing up (prim n, its own triangle)."""
    rng = np.random.default_rng(seed)
    tri = rng.uniform(-1.5, 1.5, (n, 1, 3)) + rng.normal(0, spread, (n, 3, 3))
    tri[:, :, 1] = np.abs(tri[:, :, 1]) + 0.02
    own = np.array([[[-9.0, 0, -9], [-9, 0, 20], [20, 0, -9]]])
    V = np.concatenate([tri, own]).reshape(-1, 3).astype(np.float32)
    F = np.arange(3 * (n + 1), dtype=np.uint32).reshape(-1, 3)
    gb = w.plane_gbuffer(67, 45, 0.05, (-1.6, 0.0, -1.1), prim=n)
    return V, F, gb


@pytest.fixture(scope="module")
def ocr():
    import paper_2607_23122_amd as m
    return m


# one triangle; a node; walks that keep within the column; walks over so many
# overlapping boxes that the leaves are tested early or the column overflows
@pytest.mark.parametrize("n,spread,R", [(1, 0.5, 2.0), (5, 0.5, 2.0), (300, 0.1, 1.0), (4000, 0.5, 3.0), (4000, 3.0, 50.0)])
def test_ao_trace_records_equal_counted(ocr, n, spread, R):
    import torch
    V, F, gb = _soup(n, spread, n)
    bvh = ocr.build_bvh(V, F)
    dg = ocr.DeviceGBuffer.from_host(gb)
    for sample in range(2):
        log(f"[walks] trace n={n} spread={spread} R={R} sample {sample}")
        occ = ocr.trace_occluders(bvh, dg, "ao", R, None, 3, sample)
        stats = torch.zeros(5, dtype=torch.int64, device="cuda")
        ref = ocr.trace_occluders_counted(bvh, dg, stats, "ao", R, None, 3, sample)
        torch.cuda.synchronize()
        hit = occ.hit_u32()
        assert np.array_equal(hit, ref.hit_u32())
        m = hit < oracle.SELF
        assert m.any()
        for a, b in ((occ.dz, ref.dz), (occ.nz, ref.nz)):
            assert np.array_equal(a.cpu().numpy()[m].view(np.uint32), b.cpu().numpy()[m].view(np.uint32))


def _bits(ocr, bvh, dg, gb, occ, R, radius, stats=None):
    import torch
    p = ocr.reuse_params("window", radius, 8, "unbiased")
    ws = torch.zeros(ocr.workspace_bytes(gb.width, gb.height, p), dtype=torch.uint8, device="cuda")
    ocr.validate_pairs(bvh, dg, occ, "ao", R, None, p, ws, stats=stats)
    torch.cuda.synchronize()
    n, words = gb.width * gb.height, ((4 * radius + 1) ** 2 + 31) // 32
    return ws.cpu().numpy()[:4 * n * words].view(np.uint32).reshape(n, words)


# one to all of a list's chunks and runs (radius), the tables of nodes, leaves
# and triangles from one entry to many times their size (n), triangles from
# slivers to larger than the scene (spread), segments from short to long (R)
@pytest.mark.parametrize("n,spread,R,radius", [(1, 0.5, 2.0, 1), (1, 0.5, 2.0, 3), (5, 0.5, 2.0, 2), (300, 0.1, 1.0, 3),
                                               (300, 0.1, 1.0, 8), (4000, 0.5, 3.0, 3), (4000, 0.02, 2.0, 4),
                                               (4000, 3.0, 50.0, 3), (1500, 1.0, 0.05, 3), (300, 0.1, 1.0, 0)])
def test_ao_window_validation_bits_equal_counted(ocr, n, spread, R, radius):
    import torch
    V, F, gb = _soup(n, spread, n)
    bvh = ocr.build_bvh(V, F)
    dg = ocr.DeviceGBuffer.from_host(gb)
    for sample in range(2):
        log(f"[walks] validate n={n} spread={spread} R={R} radius {radius} sample {sample}")
        occ = ocr.trace_occluders(bvh, dg, "ao", R, None, 3, sample)
        stats = torch.zeros(5, dtype=torch.int64, device="cuda")
        got = _bits(ocr, bvh, dg, gb, occ, R, radius)
        ref = _bits(ocr, bvh, dg, gb, occ, R, radius, stats)
        cand = (occ.hit_u32() < oracle.SELF).ravel()
        assert cand.any()
        bad = got[cand] ^ ref[cand]
        segs, free = int(stats[4]), int(np.unpackbits(ref[cand].view(np.uint8)).sum()) - int(cand.sum())
        log(f"    candidates {int(cand.sum())}, segments {segs}, free {free}")
        assert not bad.any(), f"{int(np.unpackbits(bad.view(np.uint8)).sum())} of {segs} pairs differ"


# receivers on many triangles (each its own ignored), background at the frame's
# ends; faces in the plane of the hit point (boxes), triangles without area, and
# ones far larger than any segment, up to vertices whose products overflow
@pytest.mark.parametrize("scene,size,radius", [("boxes", (97, 73), 2), ("boxes", (640, 360), 3), ("odd", (97, 73), 3),
                                               ("terrain", (161, 93), 3), ("terrain", (131, 67), 5)])
def test_frame_validation_bits_equal_counted(ocr, scene, size, radius):
    import torch
    sc, cam, R = (w.terrain_scene(2, 96, 70), w.terrain_camera(*size), 2.0) if scene == "terrain" else \
        (w.boxes_scene(3), w.boxes_camera(*size), 1.0)
    gb = w.render_gbuffer(sc, cam)
    V, F = sc.V, sc.F
    if scene == "odd":
        more = np.array([[0, 0.5, 0], [0, 0.5, 0], [0, 0.5, 0],                      # a point
                         [-1, 0.3, 0], [0, 0.3, 0], [1, 0.3, 0],                     # a line
                         [-3e3, 0.7, -2e3], [4e3, 0.7, -2e3], [0, 0.9, 5e3],         # over the whole scene
                         [-1e12, 1.5, -1e12], [1e12, 1.5, -1e12], [0, 1.5, 2e12]], np.float32)
        F = np.concatenate([F, (len(V) + np.arange(12, dtype=np.uint32)).reshape(-1, 3)])
        V = np.concatenate([V, more])
    bvh = ocr.build_bvh(V, F)
    dg = ocr.DeviceGBuffer.from_host(gb)
    log(f"[walks] validate {scene} {size} radius {radius}")
    occ = ocr.trace_occluders(bvh, dg, "ao", R, None, 5, 0)
    stats = torch.zeros(5, dtype=torch.int64, device="cuda")
    got = _bits(ocr, bvh, dg, gb, occ, R, radius)
    ref = _bits(ocr, bvh, dg, gb, occ, R, radius, stats)
    cand = (occ.hit_u32() < oracle.SELF).ravel()
    assert cand.any() and int(stats[4]) > 0
    assert np.array_equal(got[cand], ref[cand])
