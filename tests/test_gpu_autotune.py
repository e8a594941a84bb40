"""The autotuner on a batch whose slots hold fewer particles than they have room for."""
import numpy as np
import pytest
import torch

from gpu_util import assert_grads, assert_state, env_slices, make_env, oracle_rollout, random_cotangents, to_np
from paper_2412_12089_amd import scenes

pytestmark = pytest.mark.gpu


def test_autotune_with_slots_below_capacity():
    """Results are compared over the live particles. (The end state used to be copied with all 24 x capacity floats
    into a buffer of 24 x live ones.)"""
    from paper_2412_12089_amd.batch import Batch
    cap = [make_env(scenes.NEOHOOKEAN, N=4000, n=48, seed=51 + i) for i in range(2)]
    live = [make_env(scenes.NEOHOOKEAN, N=1500, n=32, seed=53), make_env(scenes.COROTATED, N=700, n=48, seed=54, F_dev=0.02)]
    S = 4
    b = Batch(cap, max_substeps=S, ckpt_every=2)
    for i, spec in enumerate(live):
        b.configure_env(i, spec)
        b.set_particles(*(torch.from_numpy(getattr(spec, k)) for k in ("x", "v", "C", "F")), env=i)
    before = [to_np(t) for t in b.get_particles()]
    print("[autotune] 1500 and 700 particles in slots of 4000", flush=True)
    b.autotune(2000)
    for a, c in zip(before, b.get_particles()):
        assert np.array_equal(a, to_np(c))
    b.forward(S, record=True)
    st = [to_np(t) for t in b.get_particles()]
    cots = random_cotangents(live, seed=55)
    cat = lambda k: torch.from_numpy(np.concatenate([c[k] for c in cots], axis=0))
    gr = [to_np(t) for t in b.backward(cat(0), cat(1), cat(2), cat(3))[:4]]
    assert b.sync(raise_on_error=False) == 0
    b.close()
    for i, (spec, sl) in enumerate(zip(live, env_slices(live))):
        o = oracle_rollout(spec, S, cots[i])
        assert_state([a[sl] for a in st], o["state"], spec.x, f"env {i}", S=S)
        assert_grads([g[sl] for g in gr], o["grads"], f"env {i}")
