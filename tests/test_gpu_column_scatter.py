"""The column scatter (P2G and G2P adjoint of the batched mode) where its blocks change shape: one particle,
a full block and one particle more, many particles per cell (four lanes share a task), a tile row longer than
the LDS box (slabs), particles leaving their tile rows between sorts, and blocks that fall back to the grid."""
import numpy as np
import pytest
import torch

from gpu_util import assert_grads, assert_state, make_env, oracle_rollout, random_cotangents, to_np
from paper_2412_12089_amd import scenes

pytestmark = pytest.mark.gpu

CASES = {  # particles, lower corner, sides, velocity scale
    "one": (1, (0.4, 0.4, 0.4), (0.02, 0.02, 0.02), 0.5),
    "block": (256, (0.4, 0.4, 0.4), (0.12, 0.12, 0.12), 0.5),
    "block-and-one": (257, (0.4, 0.4, 0.4), (0.12, 0.12, 0.12), 0.5),
    "dense": (1500, (0.41, 0.41, 0.41), (0.06, 0.06, 0.1), 0.5),
    "one-column": (400, (0.405, 0.405, 0.15), (0.015, 0.015, 0.7), 0.5),
    "slabs": (350, (0.42, 0.42, 0.12), (0.08, 0.08, 0.76), 0.5),
    "crossing": (900, (0.35, 0.35, 0.35), (0.2, 0.2, 0.2), 60.0),
    "sparse": (300, (0.12, 0.12, 0.12), (0.76, 0.76, 0.76), 0.5),
}


@pytest.mark.parametrize("box", [0, 1], ids=["large-box", "small-box"])
@pytest.mark.parametrize("name", list(CASES))
def test_column_scatter_matches_oracle(name, box):
    from paper_2412_12089_amd import _capi as C
    from paper_2412_12089_amd.batch import Batch
    N, lo, sides, vs = CASES[name]
    rng = np.random.Generator(np.random.PCG64(7))
    spec = make_env(scenes.NEOHOOKEAN, N=N, n=48, seed=5, dt=5e-5, v_scale=vs, F_dev=0.01)
    spec.x = scenes._f32(np.array(lo) + rng.uniform(0, 1, size=(N, 3)) * np.array(sides))
    spec.Vp = float(np.prod(sides)) / N
    S, K = 5, 4
    cot = random_cotangents([spec], seed=9)[0]
    print(f"[column scatter] {name}: {N} particles, box option {box}", flush=True)
    b = Batch([spec], max_substeps=S, ckpt_every=K)
    b.set_option(C.OPT_BOX, box)
    b.set_particles_from_specs()
    b.forward(S, record=True)
    st = [to_np(t) for t in b.get_particles()]
    gr = [to_np(t) for t in b.backward(*(torch.from_numpy(c) for c in cot))[:4]]
    assert b.sync(raise_on_error=False) == 0
    b.close()
    o = oracle_rollout(spec, S, cot)
    assert_state(st, o["state"], spec.x, name, S=S)
    assert_grads(gr, o["grads"], name)
