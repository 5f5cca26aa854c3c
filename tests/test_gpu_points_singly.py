"""Point queries of scenes with one primitive per region, whose large calls
take one evaluation after the other."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["sphere", "slab"])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_large_calls_equal_small_ones(S, eng, W, name, precision):
    """the same points in one call of 2^17 + 5 and in calls of 5000: the same
    evaluations, so equal to rounding -- distances of size 1, normals from
    differences over a step of 1e-7"""
    desc = W.WORKLOADS[name](8)
    lo, hi = np.array(desc["grid"]["lo"]), np.array(desc["grid"]["hi"])
    pts = np.random.default_rng(4).uniform(lo - 0.05, hi + 0.05, (131077, 3))
    d0, own0, nrm0 = S.distance(desc, pts, engine=eng, precision=precision, normals=True)
    for first in (0, 65536, 131077 - 5000):
        part = slice(first, first + 5000)
        d, own, nrm = S.distance(desc, pts[part], engine=eng, precision=precision, normals=True)
        assert np.max(np.abs(d - d0[part])) <= (1e-14 if precision == "f64" else 1e-6)
        far = np.abs(d).min(axis=1) > 1e-5
        assert np.array_equal(own[far], own0[part][far])
        assert np.max(np.abs(nrm - nrm0[part])) <= 1e-8
    assert np.all(np.abs(np.linalg.norm(nrm0, axis=2) - 1.0) <= 1e-12)
