"""The AO window validation by shafts (csrc/shaft.hip) against the counting walk,
which decides every pair by the hierarchy: the same bits, where the shaft's
geometry is hardest on its rounding and its tables."""
import numpy as np
import pytest

import oracle
import workloads as w
from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ocr():
    import paper_2607_23122_amd as m
    return m


def _bits(ocr, bvh, dg, occ, R, radius, stats=None):
    import torch
    p = ocr.reuse_params("window", radius, 8, "unbiased")
    ws = torch.zeros(ocr.workspace_bytes(dg.width, dg.height, p), dtype=torch.uint8, device="cuda")
    ocr.validate_pairs(bvh, dg, occ, "ao", R, None, p, ws, stats=stats)
    torch.cuda.synchronize()
    n, words = dg.width * dg.height, ((4 * radius + 1) ** 2 + 31) // 32
    return ws.cpu().numpy()[:4 * n * words].view(np.uint32).reshape(n, words)


def _compare(ocr, what, V, F, gb, R, radius, blocked=0.0, frame=None):
    """The bits of both, and that at least the share `blocked` of the pairs is."""
    import torch
    bvh, dg = frame or (ocr.build_bvh(V, F), ocr.DeviceGBuffer.from_host(gb))
    log(f"[shaft] {what}: {dg.width}x{dg.height}, R={R}, radius {radius}")
    occ = ocr.trace_occluders(bvh, dg, "ao", R, None, 3, 0)
    stats = torch.zeros(5, dtype=torch.int64, device="cuda")
    got = _bits(ocr, bvh, dg, occ, R, radius)
    ref = _bits(ocr, bvh, dg, occ, R, radius, stats)
    cand = (occ.hit_u32() < oracle.SELF).ravel()
    assert cand.any()
    segs, free = int(stats[4]), int(np.unpackbits(ref[cand].view(np.uint8)).sum()) - int(cand.sum())
    diff = int(np.unpackbits((got[cand] ^ ref[cand]).view(np.uint8)).sum())
    log(f"    candidates {int(cand.sum())}, segments {segs}, free {free}, differ {diff}")
    assert segs - free >= blocked * segs and segs > 0
    assert diff == 0, f"{diff} of {segs} pairs differ"
    return bvh, dg


def _layers(axis, at, gap, tile=0.02):
    """A floor, a ceiling 0.3 above it and, `gap` below the ceiling, a sheet of
    which every other tile is there, all level on `axis`; the origin at (at, at,
    at).  Segments to hit points beside a tile pass it `gap` before their end."""
    nx, nz = 96, 80
    ix, iz = np.meshgrid(np.arange(nx), np.arange(nz), indexing="ij")
    keep = ((ix + iz) & 1) == 0
    x0, z0 = (ix[keep] * tile - 0.4).ravel(), (iz[keep] * tile - 0.4).ravel()
    corners = [np.stack([x0 + dx * tile, np.full_like(x0, 0.3 - gap), z0 + dz * tile], -1)
               for dx, dz in ((0, 0), (1, 0), (1, 1), (0, 1))]
    q = np.stack(corners, 1)
    sheet = np.concatenate([q[:, [0, 1, 2]], q[:, [0, 2, 3]]])
    big = np.array([[-9, 0, -9], [9, 0, -9], [9, 0, 9], [-9, 0, 9]], np.float64)
    top = big + [0, 0.3, 0]
    tri = np.concatenate([sheet, top[[0, 1, 2]][None], top[[0, 2, 3]][None], big[[0, 1, 2]][None]])
    V = tri.reshape(-1, 3)
    gb = w.plane_gbuffer(67, 45, 0.02, prim=len(tri) - 1)
    pos, nrm = gb.pos.astype(np.float64), gb.nrm
    order = ((1, 0, 2), (0, 1, 2), (0, 2, 1))[axis]
    V = (V[:, order] + at).astype(np.float32)
    gb = w.GBuffer((pos[..., order] + at).astype(np.float32), np.ascontiguousarray(nrm[..., order]), gb.prim)
    return V, np.arange(len(V), dtype=np.uint32).reshape(-1, 3), gb


# level sheets close to the hit points, far from the origin: a box's rounding on
# the level axis is as large as the shaft is there
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("at,gap", [(0.0, 0.005), (100.0, 0.002), (100.0, 0.01), (1000.0, 0.01)])
def test_far_level_sheets(ocr, axis, at, gap):
    V, F, gb = _layers(axis, at, gap)
    _compare(ocr, f"sheets on axis {axis} at {at}, gap {gap}", V, F, gb, 1.0, 3, blocked=0.005)


# radii that mean no limit, up to ones whose square is not finite; segments from
# millimetres to kilometres
@pytest.mark.parametrize("scale,R", [(1.0, 1e6), (1.0, 3e19), (1000.0, 1e6), (1000.0, 3e19), (0.01, 3e38)])
def test_radius_without_limit(ocr, scale, R):
    rng = np.random.default_rng(7)
    n = 300
    tri = rng.uniform(-1.5, 1.5, (n, 1, 3)) + rng.normal(0, 0.1, (n, 3, 3))
    tri[:, :, 1] = np.abs(tri[:, :, 1]) + 0.05
    top = np.array([[[-40.0, 3, -40], [40, 3, -40], [0, 3, 60]]])
    own = np.array([[[-9.0, 0, -9], [-9, 0, 20], [20, 0, -9]]])
    V = (np.concatenate([tri, top, own]).reshape(-1, 3) * scale).astype(np.float32)
    gb = w.plane_gbuffer(67, 45, 0.05 * scale, (-1.6 * scale, 0.0, -1.1 * scale), prim=n + 1)
    _compare(ocr, f"scale {scale}", V, np.arange(len(V), dtype=np.uint32).reshape(-1, 3), gb, R, 3, blocked=0.02)
