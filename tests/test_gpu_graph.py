"""Captured launches whose scenes change between replays in what the captured
kernels hold as arguments, while every table and buffer keeps its size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(got, want, tol=1e-11):
    for k in ("launched", "interactions", "interfaces", "steps", "voxel_pieces"):
        assert got[k] == want[k], k
    f, g = got["fluence_raw"], want["fluence_raw"]
    assert np.max(np.abs(f - g)) <= tol * g.max()  # the order of FP64 sums


def test_replays_follow_the_dims_of_the_grid(S, W):
    """two scenes whose cubic voxels make grids of permuted dims, by turns in
    one output buffer: each equals its eager run"""
    import torch
    dims = [(8, 16, 32), (32, 8, 16)]
    scenes = [S.Scene(W.with_grid(W.sphere_scene(8), d, lo=[-n / 16 for n in d], hi=[n / 16 for n in d])) for d in dims]
    g_eng, e_eng = S.Engine(0, use_graph=1), S.Engine(0)
    outs = [S.Outputs(sc) for sc in scenes]
    outs[1].fluence = outs[0].fluence
    for seed in range(6):
        k = seed & 1
        S.launch(g_eng, scenes[k], seed, 4000, outputs=outs[k].zero_())
        torch.cuda.synchronize()
        got = outs[k].host()
        _check(got, S.run(scenes[k], seed, 4000, engine=e_eng))
    g_eng.close()
    e_eng.close()


def test_replays_follow_the_scenes_of_a_batch(S, W):
    """a batch of two vessel networks (equal table sizes, lists of other
    capacities) and one voxelised scene, in another order each time"""
    import torch
    nets = [S.Scene(W.vessel_scene(s, n_caps=100, n_grid=16)) for s in (4, 5)]
    vox = [S.Scene(dict(W.cylinder_scene(16), geometry="voxel")), S.Scene(dict(W.sphere_scene(16), geometry="voxel"))]
    g_eng, e_eng = S.Engine(0, precision="f64", use_graph=1), S.Engine(0, precision="f64")
    orders = [[nets[0], nets[1], vox[0]], [nets[1], nets[0], vox[0]], [nets[1], nets[0], vox[0]],
              [nets[0], vox[0], nets[0]], [nets[0], nets[0], vox[0]], [vox[0], vox[1], vox[0]], [vox[0], vox[1], vox[1]]]
    for rep, scenes in enumerate(orders):
        outs = [S.Outputs(sc) for sc in scenes]
        S.launch_batch(g_eng, scenes, [rep, rep + 9, rep + 17], [3000] * 3, outputs=outs)
        torch.cuda.synchronize()
        got = [o.host() for o in outs]
        want = S.launch_batch(e_eng, scenes, [rep, rep + 9, rep + 17], [3000] * 3)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            _check(a, b.host())
    g_eng.close()
    e_eng.close()
