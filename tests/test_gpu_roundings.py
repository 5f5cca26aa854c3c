"""One distance, several inlinings: the acceleration grid's compact capsule
records and the brute-force union take the same operations, so where the
grid's value is a distance it is the same number, to the bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("n_caps", [1, 40, 2000])
def test_capsule_distances_through_the_grid_are_the_same_bits(S, W, n_caps, precision):
    desc = W.vessel_scene(6, n_caps=n_caps, n_grid=8)
    caps = [desc["prims"][i] for i in desc["regions"][1]["prims"]]
    lo = np.min([np.minimum(p["a"], p["b"]) - p["r"] for p in caps], axis=0)
    hi = np.max([np.maximum(p["a"], p["b"]) + p["r"] for p in caps], axis=0)
    margin = np.max((hi - lo) / np.array(desc["accel_cells"]))
    # by the walls of the capsules, inside and out
    g = np.random.default_rng(3)
    pick = g.integers(0, len(caps), 20000)
    a, b, r = (np.array([caps[i][k] for i in pick]) for k in ("a", "b", "r"))
    v = g.normal(size=(len(pick), 3))
    pts = a + g.random((len(pick), 1)) * (b - a) + (r * g.uniform(0.0, 2.0, len(pick)))[:, None] * v / np.linalg.norm(v, axis=1)[:, None]
    eng = S.Engine(0)
    d, own = S.distance(desc, pts, engine=eng, precision=precision)
    e, own_e = S.distance(desc, pts, engine=eng, precision=precision, accelerated=True)
    near = d[:, 1] < margin * (1 - 1e-5)
    assert np.mean(near) > 0.5
    assert np.array_equal(d[near, 1], e[near, 1])
    assert np.array_equal(own, own_e)
    eng.close()
