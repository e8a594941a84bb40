"""The column scatter's block shapes of test_gpu_column_scatter.py in the unfused schedule and with materials that
keep an eigen-decomposition in the payload rows."""
import numpy as np
import pytest
import torch

from gpu_util import assert_grads, assert_state, make_env, oracle_rollout, random_cotangents, to_np
from paper_2412_12089_amd import scenes
from test_gpu_column_scatter import CASES

pytestmark = pytest.mark.gpu

MATERIALS = {"corotated": dict(material=scenes.COROTATED, nu=0.25),
             "von-mises": dict(material=scenes.VONMISES, nu=0.2, sigma_y=50.0)}


@pytest.mark.parametrize("fuse", [0, 1], ids=["unfused", "fused"])
@pytest.mark.parametrize("mat", list(MATERIALS))
@pytest.mark.parametrize("name", ["one", "block-and-one", "dense", "slabs", "sparse"])
def test_column_scatter_materials_and_schedules(name, mat, fuse):
    from paper_2412_12089_amd import _capi as C
    from paper_2412_12089_amd.batch import Batch
    N, lo, sides, vs = CASES[name]
    rng = np.random.Generator(np.random.PCG64(7))
    spec = make_env(N=N, n=48, seed=5, dt=5e-5, v_scale=vs, F_dev=0.01, **MATERIALS[mat])
    spec.x = scenes._f32(np.array(lo) + rng.uniform(0, 1, size=(N, 3)) * np.array(sides))
    spec.Vp = float(np.prod(sides)) / N
    S, K = 5, 4
    cot = random_cotangents([spec], seed=9)[0]
    print(f"[column scatter] {name}, {mat}, fuse {fuse}", flush=True)
    b = Batch([spec], max_substeps=S, ckpt_every=K)
    b.set_option(C.OPT_FUSE, fuse)
    b.set_option(C.OPT_FUSE_ADJ, fuse)
    b.set_particles_from_specs()
    b.forward(S, record=True)
    st = [to_np(t) for t in b.get_particles()]
    gr = [to_np(t) for t in b.backward(*(torch.from_numpy(c) for c in cot))[:4]]
    assert b.sync(raise_on_error=False) == 0
    b.close()
    o = oracle_rollout(spec, S, cot)
    assert_state(st, o["state"], spec.x, name, S=S)
    assert_grads(gr, o["grads"], name)
