"""A served epoch ends within some steps of its deadline."""
import copy

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_epochs_end_within_some_steps_of_their_deadline(S, W, precision):
    """packets that take some 1600 steps past a row of 300 spheres, each step
    well over 2 us, in epochs of 100 us: with the clock read every 16 steps
    an epoch holds at most 50 steps up to the deadline and 31 beyond it"""
    import torch
    n_balls, n = 300, 640
    desc = copy.deepcopy(W.absorbing_sphere(mua=1e-9))
    balls = [{"kind": "sphere", "c": [0.01, 0.0, -1.0 + (2 * i + 1) / n_balls], "r": 0.009} for i in range(n_balls)]
    desc["prims"] = [{"kind": "box", "c": [0.0, 0.0, 0.0], "half": [0.05, 0.05, 1.0]}] + balls
    desc["regions"] = [desc["regions"][0], dict(desc["regions"][0], prims=list(range(1, n_balls + 1)))]
    desc["source"] = {"kind": "pencil", "p": [0.0, 0.0, 0.99], "u": [0.0, 0.0, -1.0]}
    sv = S.Server(0, hbm_budget_bytes=1 << 30, epoch_us=100, precision=precision)
    rid, out = sv.submit(desc, 1, n)
    sv.wait(rid, 60.0)
    epochs = sv.stats()["epochs"]
    torch.cuda.synchronize()
    steps = out.host()["steps"] / n
    sv.close()
    print(f"{precision}: {steps:.0f} steps a packet in {epochs} epochs")
    assert steps > 1000
    assert steps / epochs <= 96
