"""Voxel walks almost along an axis's planes: only a direction without any
component across them is parallel to them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("across", [0.0, 2e-31, -2e-31, 8e-30, -3e-20, 1e-13, 1e-11, 1e-6])
def test_steep_pencils_cross_the_thin_voxels(S, eng, orc, W, axis, across, precision):
    """a pencil down a stack of voxels so thin that it crosses three of their
    faces, at any steepness; against the oracle's voxel walk, 500 lengths of
    size 1 added per voxel"""
    d = abs(across) / 2 or 1e-31
    start = d * (0.5 if across >= 0.0 else 3.5)
    lo, hi, dims = [-0.5, -0.5, -1.0], [0.5, 0.5, 1.0], [1, 1, 8]
    lo[axis], hi[axis], dims[axis] = 0.0, 4 * d, 4
    p, u = [0.0, 0.0, 0.9], [0.0, 0.0, -1.0]
    p[axis], u[axis] = start, across
    desc = W.absorbing_sphere(mua=0.5)
    desc["prims"] = [{"kind": "box", "c": [0.0, 0.0, 0.0], "half": [1.0] * 3}]
    desc["source"] = {"kind": "pencil", "p": p, "u": u}
    desc = W.with_grid(dict(desc, geometry="voxel", grid={}), dims, lo=lo, hi=hi)
    n = 500
    o, g = orc.run(desc, 3, n, voxel=True), S.run(desc, 3, n, engine=eng, precision=precision)
    assert np.count_nonzero(o["fluence_raw"].sum(axis=(0, 1) if axis == 0 else (0, 2))) == (4 if across else 1)
    assert np.max(np.abs(g["fluence_raw"] - o["fluence_raw"])) <= (1e-12 if precision == "f64" else 1e-5) * n
