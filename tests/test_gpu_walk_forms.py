"""GPU parity with the oracle at the sizes where the walk's division of work
changes: packet counts around one lane, one wave and one packet per wave of
the launch, and scenes whose regions fill one or two rounds of the interface
step's eight lanes per packet."""
import copy

import numpy as np
import pytest

from gpu_helpers import compare_traces, extent_of, identity_residual

pytestmark = pytest.mark.gpu

WAVES_F64 = 3072  # waves of a full FP64 launch (256 CUs, 3 per SIMD): where a wave starts to take 2 packets


def layered_ball(W, n_regions):
    """n_regions nested regions of alternating indices (spheres and boxes by
    turns, every third one a pair of spheres) around a point source"""
    prims, regions = [], []
    for i in range(n_regions):
        r = 1.0 - 0.8 * i / n_regions
        c = [0.01 * i, -0.005 * i, 0.0]
        if i % 3 == 1:
            prims.append({"kind": "box", "c": c, "half": [r * 0.6] * 3})
        else:
            prims.append({"kind": "sphere", "c": c, "r": r})
        ids = [len(prims) - 1]
        if i % 3 == 2:
            prims.append({"kind": "sphere", "c": [c[0] + 0.05, c[1], 0.02], "r": 0.9 * r})
            ids.append(len(prims) - 1)
        regions.append({"prims": ids, "op": "union", "k": 0.0, "mua": 0.2 + 0.1 * (i % 4), "mus": 5.0 + i,
                        "g": 0.5, "n": 1.3 + 0.05 * (i % 5)})
    sc = copy.deepcopy(W.absorbing_sphere())
    sc.update(prims=prims, regions=regions, grid={"lo": [-1.1] * 3, "hi": [1.1] * 3, "dims": [12] * 3})
    return sc


@pytest.mark.parametrize("n_regions", [1, 7, 8, 9, 16])
def test_interface_steps_over_the_rounds_of_regions(S, eng, orc, W, n_regions):
    desc = layered_ball(W, n_regions)
    n = 96
    mut = [rg["mua"] + rg["mus"] for rg in desc["regions"]]
    o = [orc.trace(desc, 3, pid, 40) for pid in range(n)]
    g = S.trace(desc, 3, list(range(n)), 40, engine=eng, precision="f64")
    frac, worst, bad = compare_traces(o, g, extent_of(S, desc), 1e-6, cap=40, mut=mut)
    assert frac >= 0.98, (frac, worst, bad[:5])  # at most one grazing near-tie of 96
    r, t = S.run(desc, 3, 2000, engine=eng, precision="f64"), orc.run(desc, 3, 2000)
    assert abs(identity_residual(r)) <= 1e-9 * 2000
    assert abs(r["absorbed"].sum() - t["absorbed"].sum()) <= 1.0 + 1e-9 * 2000  # one packet's weight
    assert abs(r["interfaces"] - t["interfaces"]) <= max(2, 2e-3 * t["interfaces"])


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, WAVES_F64 - 1, WAVES_F64, WAVES_F64 + 1, 2 * WAVES_F64 + 1])
def test_packet_counts_around_the_lanes_of_a_launch(S, eng, orc, W, n):
    desc = W.sphere_scene(20)
    g = S.run(desc, 5, n, first=7, engine=eng, precision="f64")
    o = orc.run(desc, 5, n, first=7)
    assert g["launched"] == n and g["escapes"] + g["kills"] + g["stalls"] == n
    assert abs(g["absorbed"].sum() - o["absorbed"].sum()) <= 1e-9 * o["absorbed"].sum()
    # the same packets in two launches, whose waves hold other numbers of
    # them: equal to the order of FP64 sums (some 1e2 terms per voxel)
    h = [S.run(desc, 5, m, first=f, engine=eng, precision="f64") for f, m in ((7, n // 2), (7 + n // 2, n - n // 2))]
    F = sum(x["fluence_raw"] for x in h)
    assert np.max(np.abs(g["fluence_raw"] - F)) <= 1e-12 * F.max()
    for k in ("events", "steps", "interactions", "voxel_pieces", "escapes"):
        assert g[k] == sum(x[k] for x in h), k


@pytest.mark.parametrize("surface_min", [1, 8, 9, 64])
def test_gathered_interface_steps_leave_the_walk_unchanged(S, eng, W, surface_min):
    desc = layered_ball(W, 9)
    e = S.Engine(0, surface_min=surface_min, precision="f64")
    a, b = S.run(desc, 9, 5000, engine=eng, precision="f64"), S.run(desc, 9, 5000, engine=e, precision="f64")
    for k in ("events", "steps", "interfaces", "reflections", "refractions", "advances", "escapes"):
        assert a[k] == b[k], k
    assert np.max(np.abs(a["fluence_raw"] - b["fluence_raw"])) <= 1e-12 * a["fluence_raw"].max()
    e.close()


@pytest.mark.parametrize("cells", [(1, 1, 1), (1, 2, 3), (16, 16, 8), (127, 17, 1), (2048 // 64, 64, 1), (33, 35, 37),
                                   (256, 256, 3)])
@pytest.mark.parametrize("n_caps", [1, 3, 300])
def test_grid_builds_at_the_edges_of_the_scan_tiles(S, eng, W, cells, n_caps):
    """the accelerated distance is the brute-force one below the margin and a
    lower bound of it, not below the margin, elsewhere (reading of the grid);
    tolerance: FP64 rounding of coordinates of size 0.2 (1e-15) and the
    bound's own relative 2^-20"""
    desc = W.vessel_scene(3, n_caps=n_caps, n_grid=8)
    desc["accel_cells"] = list(cells)
    if n_caps == 1:  # a union of one capsule and a small box: no capsule records
        desc["prims"].append({"kind": "box", "c": [0.05, 0.05, 0.05], "half": [0.004] * 3})
        desc["regions"][1]["prims"] = [1, 2]
    prims = [desc["prims"][i] for i in desc["regions"][1]["prims"]]
    lo = np.min([np.minimum(p["a"], p["b"]) - p["r"] if "r" in p else np.subtract(p["c"], p["half"]) for p in prims], axis=0)
    hi = np.max([np.maximum(p["a"], p["b"]) + p["r"] if "r" in p else np.add(p["c"], p["half"]) for p in prims], axis=0)
    margin = np.max((hi - lo) / np.array(cells))
    pts = np.random.default_rng(1).uniform(-0.02, 0.22, (4000, 3))
    d, own = S.distance(desc, pts, engine=eng)
    a, own_a = S.distance(desc, pts, engine=eng, accelerated=True)
    d, a = d[:, 1], a[:, 1]
    near = d < margin
    assert np.all(np.abs(a[near] - d[near]) <= 1e-14)
    assert np.all(a <= d + 1e-14)
    inside = np.all((pts > lo - margin) & (pts < hi + margin), axis=1)
    far = ~near & inside
    assert np.all(a[far] >= margin * (1 - 1e-12))
    assert np.array_equal(own, own_a)


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 3), (33, 7, 2), (5, 64, 31), (127, 129, 128)])
def test_tally_over_grids_and_layouts(S, eng, orc, W, dims):
    """straight absorbed paths through odd grids that the ball overlaps in
    part; at the finest one a wave's pieces overflow its staging area.  FP64
    against the oracle to rounding (positions of size 1, a few hundred
    additions per voxel); FP32 bricks against FP32 linear storage: the same
    pieces in another order."""
    desc = W.absorbing_sphere(mua=0.8)
    desc["grid"] = {"lo": [-1.2, -0.9, -1.0], "hi": [0.95, 1.1, 1.05], "dims": list(dims)}
    n = 1000
    o = orc.run(desc, 21, n)
    layouts = [S.Engine(0, tally_layout=k) for k in (0, 1)]
    scale = o["fluence_raw"].max()
    for e in layouts:
        g = S.run(desc, 21, n, engine=e, precision="f64")
        assert np.max(np.abs(g["fluence_raw"] - o["fluence_raw"])) <= 1e-12 * scale
    a, b = [S.run(desc, 21, n, engine=e, precision="f32") for e in layouts]
    assert a["voxel_pieces"] == b["voxel_pieces"]
    assert np.max(np.abs(a["fluence_raw"] - b["fluence_raw"])) <= 1e-12 * scale
    assert abs(a["fluence_raw"].sum() - o["fluence_raw"].sum()) <= 1e-4 * o["fluence_raw"].sum()
    for e in layouts:
        e.close()


@pytest.mark.parametrize("relax", [1.0, 1.7])
@pytest.mark.parametrize("placed", [False, True])
def test_accelerated_unions_in_every_kernel(S, eng, orc, W, relax, placed):
    """vessels through the grid, plain and over-relaxed (another kernel), with
    and without a placed member (another again), against the oracle"""
    plain = W.vessel_scene(2, n_caps=60, n_grid=8)
    if placed:
        p = plain["prims"][plain["regions"][1]["prims"][0]]
        p["transform"] = {"R": W.rotation([0.0, 0.0, 1.0], 0.0), "t": [0.0, 0.0, 0.0], "s": 1.0}
    desc = dict(plain, relax=relax)
    n = 200
    mut = [rg["mua"] + rg["mus"] for rg in desc["regions"]]
    o = [orc.trace(plain, 13, pid, 40) for pid in range(n)]
    g = S.trace(desc, 13, list(range(n)), 40, engine=eng, precision="f64")
    frac, worst, bad = compare_traces(o, g, extent_of(S, desc), 1e-6, cap=40, mut=mut)
    assert frac >= 0.98, (frac, worst, bad[:5])  # grazing near-ties
    k, t = S.run(desc, 13, 3000, engine=eng, precision="f64"), S.run(plain, 13, 3000, engine=eng, precision="f64")
    assert abs(identity_residual(k)) <= 1e-9 * 3000
    assert abs(k["interactions"] - t["interactions"]) <= 2e-3 * t["interactions"]


@pytest.mark.parametrize("name", ["vessels", "gallery", "cylinder"])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_point_queries_at_the_edges_of_their_kernels(S, eng, W, name, precision):
    """the same points asked for in calls of every size where the division of
    the work changes (waves of 64, a workgroup of 256, a point per lane from
    2^17 on): the same evaluations, so equal to rounding -- distances of size
    1, normals from differences over a step of 1e-5 or so"""
    desc = W.vessel_scene(1, n_caps=20, n_grid=8) if name == "vessels" else W.WORKLOADS[name](8)
    lo, hi = np.array(desc["grid"]["lo"]), np.array(desc["grid"]["hi"])
    pts = np.random.default_rng(4).uniform(lo - 0.05, hi + 0.05, (131072, 3))
    d0, own0, nrm0 = S.distance(desc, pts, engine=eng, precision=precision, normals=True)
    for n in (1, 63, 64, 65, 255, 257, 5000, 131071):
        d, own, nrm = S.distance(desc, pts[:n], engine=eng, precision=precision, normals=True)
        assert np.max(np.abs(d - d0[:n])) <= (1e-14 if precision == "f64" else 1e-6)
        far = np.abs(d0[:n]).min(axis=1) > 1e-5
        assert np.array_equal(own[far], own0[:n][far])
        both = np.isfinite(nrm) & np.isfinite(nrm0[:n])
        assert np.mean(both) > 0.99 and np.max(np.abs(nrm - nrm0[:n])[both]) <= 1e-8
        e, own_e = S.distance(desc, pts[:n], engine=eng, precision=precision)
        assert np.max(np.abs(e - d)) <= (1e-14 if precision == "f64" else 1e-6)


def test_fp32_lengths_are_correctly_rounded(S, eng, W):
    """the FP32 distance of a sphere about the origin, on an axis, is
    sqrt(x x) - r with one rounding each: float32 arithmetic, bit by bit"""
    desc = W.absorbing_sphere(r=1.0)
    x = np.concatenate([np.geomspace(1e-12, 1e12, 30000), np.random.default_rng(2).uniform(0.5, 2.0, 30000)])
    x = x.astype(np.float32)
    pts = np.zeros((x.size, 3))
    for axis in range(3):
        pts[:] = 0.0
        pts[:, axis] = x
        d, _ = S.distance(desc, pts, engine=eng, precision="f32")
        assert np.array_equal(d[:, 0].astype(np.float32), np.sqrt(x * x) - np.float32(1.0))


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("u", [[0.0, 0.0, -1.0], [0.0, -1.0, 0.0], [1.0, 0.0, 0.0], [0.0, -0.6, 0.8]])
def test_tally_of_rays_along_voxel_planes(S, eng, orc, W, u, precision):
    """pencil beams parallel to axes, in a grid's outer faces, in planes
    between voxels, inside and outside: against the oracle, exactly placed
    (steps of 1/8: no rounding in FP32 either) up to the absorbed lengths"""
    for x in (-0.5, -0.25, 0.125, 0.5, 0.625):
        desc = W.absorbing_sphere(mua=0.5)
        desc["prims"] = [{"kind": "box", "c": [0.0, 0.0, 0.0], "half": [1.0] * 3}]
        p = [x, -x, x]
        for i in range(3):
            if u[i] != 0.0:
                p[i] = 0.0
        desc["source"] = {"kind": "pencil", "p": p, "u": u}
        desc["grid"] = {"lo": [-0.5] * 3, "hi": [0.5] * 3, "dims": [4, 8, 4]}
        n = 500
        o, g = orc.run(desc, 3, n), S.run(desc, 3, n, engine=eng, precision=precision)
        eps = 1e-12 if precision == "f64" else 1e-5  # of lengths of size 1, n of them
        assert np.max(np.abs(g["fluence_raw"] - o["fluence_raw"])) <= eps * n, (x, u)


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 1, 2), (17, 33, 5), (64, 64, 64)])
def test_voxel_moves_over_grid_sizes(S, eng, orc, W, dims):
    """the voxelised model from one voxel up: traces and counts against the
    oracle's voxel walk, and the same packets in two launches"""
    desc = dict(W.cylinder_scene(8), geometry="voxel")
    desc["grid"] = dict(desc["grid"], dims=list(dims))
    n = 128
    mut = [rg["mua"] + rg["mus"] for rg in desc["regions"]]
    o = [orc.trace(desc, 17, pid, 40, voxel=True) for pid in range(n)]
    g = S.trace(desc, 17, list(range(n)), 40, engine=eng, precision="f64")
    frac, worst, bad = compare_traces(o, g, extent_of(S, desc), 1e-6, cap=40, mut=mut)
    assert frac >= 0.98, (frac, worst, bad[:5])
    for precision in ("f64", "f32"):
        a = S.run(desc, 17, 3001, engine=eng, precision=precision)
        h = [S.run(desc, 17, m, first=f, engine=eng, precision=precision) for f, m in ((0, 1), (1, 3000))]
        for k in ("events", "steps", "interactions", "voxel_pieces", "escapes"):
            assert a[k] == sum(x[k] for x in h), k
        F = sum(x["fluence_raw"] for x in h)
        assert np.max(np.abs(a["fluence_raw"] - F)) <= 1e-12 * F.max()
        assert abs(identity_residual(a)) <= 1e-9 * 3001
