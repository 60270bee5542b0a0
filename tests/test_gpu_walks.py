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
