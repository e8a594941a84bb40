"""The kernel options of the batched mode run what they name."""
import numpy as np
import pytest
import torch

from gpu_util import assert_grads, assert_state, make_env, oracle_rollout, random_cotangents, to_np
from paper_2412_12089_amd import scenes

pytestmark = pytest.mark.gpu

STATE_AND_GRADS = ("x", "v", "C", "F", "dx", "dv", "dC", "dF")


def run(envs, S, K, cots, mode="batched", options=()):
    from paper_2412_12089_amd import _capi as C
    from paper_2412_12089_amd.batch import Batch
    print(f"[schedules] {mode} {dict(options)}", flush=True)
    b = Batch(envs, max_substeps=S, ckpt_every=K, mode=mode)
    for name, value in options:
        b.set_option(getattr(C, "OPT_" + name), value)
    b.set_particles_from_specs()
    b.forward(S, record=True)
    out = [to_np(t) for t in b.get_particles()]
    cat = lambda k: torch.from_numpy(np.concatenate([c[k] for c in cots], axis=0))
    out += [to_np(t) for t in b.backward(cat(0), cat(1), cat(2), cat(3))]
    assert b.sync(raise_on_error=False) == 0
    b.close()
    return out


@pytest.mark.parametrize("material", [scenes.COROTATED, scenes.VONMISES, scenes.FLUID_TAIT])
def test_options_at_zero_run_the_plain_kernels(material):
    """Particles whose stencils share no node: no sum depends on an order, so the same kernels give the same bits."""
    spec = make_env(material, N=64, n=48, seed=41, F_dev=0.01, sigma_y=5.0)
    rng = np.random.Generator(np.random.PCG64(42))
    at = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3)
    spec.x = scenes._f32((6.0 + 9.0 * at + rng.uniform(0.0, 4.0, size=(64, 3))) / 48.0)
    cots = random_cotangents([spec], seed=43)
    plain = run([spec], 3, 2, cots, mode="plain")
    zero = run([spec], 3, 2, cots, options=[(k, 0) for k in ("P2G", "G2P", "G2P_ADJ", "P2G_ADJ", "FUSE", "FUSE_ADJ")])
    for name, a, b in zip(STATE_AND_GRADS, plain, zero):
        assert np.array_equal(a, b), (name, np.abs(a - b).max())


@pytest.mark.parametrize("N", [1, 2, 3, 5, 255, 257])
@pytest.mark.parametrize("mode", ["plain", "batched"])
def test_global_scatters_at_partial_quads(mode, N):
    """The scatters with global atomics take particles in fours: counts that leave a quad partly filled, in plain mode
    and in the batched mode's fallback (particles over the whole interior cross too many tile rows for a box)."""
    spec = make_env(scenes.NEOHOOKEAN, N=N, n=48, seed=44, lo=0.12, side=0.76, F_dev=0.01, dt=5e-5)
    cot = random_cotangents([spec], seed=45)
    out = run([spec], 4, 2, cot, mode=mode)
    o = oracle_rollout(spec, 4, cot[0])
    assert_state(out[:4], o["state"], spec.x, f"{mode} {N}", S=4)
    assert_grads(out[4:8], o["grads"], f"{mode} {N}")
