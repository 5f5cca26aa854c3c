"""What a request is charged against the server's budget covers the device
bytes that its admission allocates (dry runs: no device needed)."""
import copy
import os
import subprocess
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def S():
    from paper_2112_08035_amd import build_lib, smcrt
    if build_lib.is_stale():
        build_lib.build()
    smcrt.lib()
    return smcrt


@pytest.fixture(scope="module")
def record_bytes(tmp_path_factory):
    """sizes of the records of layout.h: Prim (both precisions), StepRec (both)"""
    d = tmp_path_factory.mktemp("sizes")
    (d / "sizes.cpp").write_text('#include <stdio.h>\n#include "layout.h"\nusing namespace smcrt;\n'
                                 'int main() { printf("%zu %zu %zu\\n", sizeof(PrimD) + sizeof(PrimF), '
                                 'sizeof(StepRec<double>) + sizeof(StepRec<float>), sizeof(WalkArgs)); }\n')
    inc = os.path.join(ROOT, "paper_2112_08035_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", inc, "-o", str(d / "sizes"), str(d / "sizes.cpp")], check=True)
    return [int(x) for x in subprocess.run([str(d / "sizes")], capture_output=True, text=True, check=True).stdout.split()]


def _charged(S, desc, **opts):
    """bytes_in_use while the request is the only one admitted"""
    sv = S.Server(device=-1, hbm_budget_bytes=1 << 30, **opts)
    try:
        rid = sv.submit(S.Scene(desc), 1, 1 << 50)[0]
        end = time.time() + 20
        while sv.poll(rid)[0] != "RUNNING" and time.time() < end:
            time.sleep(0.001)
        used = sv.stats()["bytes_in_use"]
        sv.cancel(rid)
        return used
    finally:
        sv.close()


def _balls(W, n):
    sc = copy.deepcopy(W.absorbing_sphere())
    sc["prims"] += [{"kind": "sphere", "c": [0.0, 0.0, 1e-3 * i], "r": 0.01} for i in range(n - 1)]
    sc["regions"][0]["prims"] = list(range(n))
    return sc


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_every_table_of_a_scene_is_charged(S, W, record_bytes, precision):
    prim, step, job = record_bytes
    one, many = (_charged(S, _balls(W, n), precision=precision) for n in (1, 3001))
    assert many - one >= 3000 * (prim + step) - 256
    assert one >= prim + step + job


@pytest.mark.parametrize("geometry", ["sdf", "voxel"])
def test_grids_of_a_scene_are_charged(S, W, record_bytes, geometry):
    """the accelerated region's capsules have one evaluation record in all,
    but compact records and the grid's counts, cursors and offsets"""
    prim, step, job = record_bytes
    desc = dict(W.vessel_scene(3, n_caps=400, n_grid=20), geometry=geometry, accel_cells=[30, 31, 32])
    held = 401 * prim + 2 * step + 400 * 8 * 12 + 3 * 4 * (30 * 31 * 32 + 1) + 8 * 20 ** 3 + job
    if geometry == "voxel":
        held += 20 ** 3
    assert _charged(S, desc) >= held
