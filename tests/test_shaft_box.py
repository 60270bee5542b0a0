"""The box test that gathers a candidate's triangles for the AO window validation
(csrc/shaft_box.hpp), compiled for the host: no box that a segment meets may be
missed, wherever the scene lies, however close to the hit point the box and
however flat both.  The segments are taken in float64 from the FP32 points."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_23122_amd", "csrc")

# every shaft: z, the interval of w, the box; rcp off by `ulp` ulps
SHIM = r"""
#include "shaft_box.hpp"
#include <math.h>
extern "C" void meets(int n, const float *z, const float *lo, const float *hi, const float *bl, const float *bh,
                      int ulp, unsigned char *out) {
    for (int i = 0; i < n; ++i) {
        ocr::Shaft S;
        float cz = 0.0f, W = 0.0f;
        for (int a = 0; a < 3; ++a) {
            S.lo[a] = lo[3 * i + a];
            S.hi[a] = hi[3 * i + a];
            cz = fmaxf(cz, fabsf(z[3 * i + a]));
            W = fmaxf(W, fmaxf(fabsf(S.lo[a]), fabsf(S.hi[a])));
        }
        auto rcp = [&](float v) {
            float r = 1.0f / v;
            return ulp ? nextafterf(r, ulp > 0 ? INFINITY : -INFINITY) : r;
        };
        ocr::shaft_set(S, z + 3 * i, cz + W, W, rcp, [](float v) { return v; });
        out[i] = ocr::shaft_meets(S, bl + 3 * i, bh + 3 * i);
    }
}
"""


@pytest.fixture(scope="module")
def meets(tmp_path_factory):
    d = tmp_path_factory.mktemp("shaft")
    src, so = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas", "-shared", "-fPIC", "-I",
                    CSRC, src, "-o", so], check=True)
    fn = ctypes.CDLL(so).meets

    def call(z, lo, hi, bl, bh, ulp):
        out = np.zeros(len(z), np.uint8)
        args = [np.ascontiguousarray(v, np.float32) for v in (z, lo, hi, bl, bh)]
        fn(len(z), *(v.ctypes.data_as(ctypes.c_void_p) for v in args), ulp, out.ctypes.data_as(ctypes.c_void_p))
        return out.astype(bool)

    return call


# `level`: receivers of one height on the box's flat axis (a floor), or as they come
@pytest.mark.parametrize("level", [True, False])
@pytest.mark.parametrize("coord", [0.0, 10.0, 100.0, 1000.0, 10000.0])
def test_no_box_on_a_segment_is_missed(meets, coord, level):
    rng = np.random.default_rng(int(coord) + level)
    n, f4, f8 = 50000, np.float32, np.float64
    # a receiver and z about 0.5 m from it, by FP32 as the kernels form them
    ok = (coord * rng.uniform(0.9, 1.0, (n, 3)) * rng.choice([-1, 1], (n, 3))).astype(f4)
    oj = (ok + rng.normal(0, 0.2, (n, 3))).astype(f4)
    dz = rng.normal(0, 0.3, (n, 3)).astype(f4)
    axis = rng.integers(0, 3, n)
    row = np.arange(n)
    if level:
        oj[row, axis] = ok[row, axis]
        # nearly level with z as well: w's interval on that axis closes on 0
        dz[row, axis] *= 10.0 ** rng.uniform(-5, 0, n).astype(f4)
    w = ((oj - ok).astype(f4) + dz).astype(f4)
    z = (oj + dz).astype(f4)
    # a sheet across the segment at s from z's end, flat on the axis, 1e-3 m wide
    s = 10.0 ** rng.uniform(-3.9, 0, n)
    at = ok.astype(f8) + (1 - s)[:, None] * w.astype(f8)
    bl, bh = (at - 1e-3).astype(f4), (at + 1e-3).astype(f4)
    plane = at[row, axis].astype(f4)
    bl[row, axis] = bh[row, axis] = plane
    # kept: sheets that the segment crosses in float64 within the box, before its end
    with np.errstate(divide="ignore", invalid="ignore"):
        t = (plane.astype(f8) - ok[row, axis]) / w[row, axis].astype(f8)
    p = ok.astype(f8) + t[:, None] * w.astype(f8)
    inside = ((p >= bl) & (p <= bh))
    inside[row, axis] = True
    real = np.isfinite(t) & (t > 0) & (t < 1 - 1e-4) & inside.all(1)
    assert real.sum() > n // 100
    for ulp in (-1, 0, 1):
        got = meets(z, -w, -w, bl, bh, ulp)
        missed = int((real & ~got).sum())
        assert missed == 0, f"{missed} of {int(real.sum())} sheets missed, reciprocals off by {ulp} ulp"
        # more receivers only widen the shaft
        assert meets(z, -w - f4(0.1), -w + f4(0.05), bl, bh, ulp)[real].all()
    # a test that accepts everything would pass the above: sheets that the segment
    # passes by 10 cm (above what the coordinates' pads come to) are not met
    if coord <= 1000.0:
        off = np.zeros((n, 3), f4)
        off[row, (axis + 1) % 3] = 0.1
        away = meets(z, -w, -w, bl + off, bh + off, 0)
        assert away[real].mean() < 0.5
