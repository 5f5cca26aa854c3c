"""Packet counts around one packet per wave of an FP32 launch, in the plain
kernel and in the staged-capsule kernel with its workgroups of 16 waves: where
a launch's packets are spread over more lanes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

WAVES = 4096  # waves of a full FP32 launch (256 CUs, 4 per SIMD; 16 per staged workgroup)


@pytest.mark.parametrize("scene", ["plain", "staged"])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, WAVES - 1, WAVES, WAVES + 1, 2 * WAVES + 1, 64 * WAVES + 3])
def test_fp32_packet_counts_around_the_lanes_of_a_launch(S, W, scene, n):
    """the same packets in one launch, in two, whose waves hold other numbers
    of them, and (staged) without the table: equal counts, and sums equal to
    their order (some 1e2 terms per voxel)"""
    desc = W.sphere_scene(16) if scene == "plain" else W.vessel_scene(8, n_caps=40, n_grid=16)
    eng = S.Engine(0)
    g = S.run(desc, 5, n, first=7, engine=eng, precision="f32")
    assert g["launched"] == n and g["escapes"] + g["kills"] + g["stalls"] == n
    parts = [[S.run(desc, 5, m, first=f, engine=eng, precision="f32") for f, m in ((7, n // 2), (7 + n // 2, n - n // 2)) if m]]
    if scene == "staged":
        other = S.Engine(0, no_stage=1)
        parts.append([S.run(desc, 5, n, first=7, engine=other, precision="f32")])
        other.close()
    for h in parts:
        F = sum(x["fluence_raw"] for x in h)
        assert np.max(np.abs(g["fluence_raw"] - F)) <= 1e-12 * F.max()
        for k in ("events", "steps", "interactions", "interfaces", "voxel_pieces", "escapes"):
            assert g[k] == sum(x[k] for x in h), k
    eng.close()


@pytest.mark.parametrize("relax", [1.0, 1.7])
@pytest.mark.parametrize("placed", [False, True])
def test_fp32_accelerated_unions_in_every_kernel(S, W, relax, placed):
    """vessels through the grid in FP32: staged, over-relaxed and with a placed
    member, each another kernel; against the plain kernel's interactions (3000
    packets of about 40 each: 4 standard errors of their sum)"""
    plain = W.vessel_scene(2, n_caps=60, n_grid=8)
    desc = dict(plain, relax=relax, prims=[dict(p) for p in plain["prims"]])
    if placed:
        desc["prims"][plain["regions"][1]["prims"][0]]["transform"] = {"R": W.rotation([0.0, 0.0, 1.0], 0.0),
                                                                      "t": [0.0, 0.0, 0.0], "s": 1.0}
    n = 3000
    one, eng = S.Engine(0, no_stage=1), S.Engine(0)
    t, k = S.run(plain, 13, n, engine=one, precision="f32"), S.run(desc, 13, n, engine=eng, precision="f32")
    assert k["launched"] == n and k["escapes"] + k["kills"] + k["stalls"] == n
    weight = k["absorbed"].sum() + k["escaped_face"].sum() + k["roulette_loss"] - k["roulette_gain"] + k["stalled"]
    assert abs(weight - n) <= 1e-9 * n
    if relax == 1.0 and not placed:
        assert k["interactions"] == t["interactions"] and k["steps"] == t["steps"]
    assert abs(k["interactions"] - t["interactions"]) <= 4 * 40 * np.sqrt(2 * n)
    one.close()
    eng.close()
