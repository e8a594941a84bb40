"""The kernel options of the batched mode run what they name, and the unfused schedule, which the defaults do not
run in a segment's middle substeps, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import (assert_grads, assert_state, env_slices, make_env, oracle_rollout, random_cotangents, relerr,
                      to_np)
from oracle import mpm_oracle as O
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


SCHEDULES = {
    "unfused": (("FUSE", 0), ("FUSE_ADJ", 0)),
    "unfused-small-box-list": (("FUSE", 0), ("FUSE_ADJ", 0), ("BOX", 1), ("GRID_LIST", 1)),
    "unfused-generic-xcd": (("FUSE", 0), ("FUSE_ADJ", 0), ("SPECIALIZE", 0), ("XCD", 1)),
    "forward-unfused": (("FUSE", 0),),
    "adjoint-unfused": (("FUSE_ADJ", 0),),
}


@pytest.mark.parametrize("name", list(SCHEDULES))
def test_unfused_schedules_match_oracle(name):
    envs = [make_env(scenes.VONMISES, N=1800, seed=61, F_dev=(0.01, 0.0003), nu=0.2, sigma_y=5.0),
            make_env(scenes.COROTATED, N=1300, n=48, seed=62, F_dev=0.02),
            make_env(scenes.FLUID_PAPER, N=700, seed=63),
            make_env(scenes.FLUID_TAIT, N=600, n=32, seed=64, lo=0.12, side=0.76, v_scale=0.3)]
    S, K = 6, 4
    cots = random_cotangents(envs, seed=65)
    out = run(envs, S, K, cots, options=SCHEDULES[name])
    for i, (e, sl) in enumerate(zip(envs, env_slices(envs))):
        o = oracle_rollout(e, S, cots[i])
        assert_state([a[sl] for a in out[:4]], o["state"], e.x, f"{name} env {i}", S=S)
        assert_grads([a[sl] for a in out[4:8]], o["grads"], f"{name} env {i}")


def test_unfused_schedule_with_a_driven_collider():
    """A turned box driven by velocities and angular speeds, with a free env beside it: states, cotangents and the
    gradients of both actions, the start center and the start angle (the inputs and bars of test_gpu_parity.py's
    spin actions, which run the other schedules)."""
    from paper_2412_12089_amd import _capi as C
    from paper_2412_12089_amd.batch import Batch
    box = scenes.BoxCollider(center=(0.6, 0.46, 0.46), half=(0.04, 0.12, 0.2), velocity=(-0.4, 0.0, 0.0), alpha=64.0,
                             mu_b=0.3, axis=(0.0, 0.6, 0.8), angle=0.4, omega=6.0)
    spec = make_env(scenes.FLUID_TAIT, N=3000, seed=162, collider=box, v_scale=0.2)
    other = make_env(scenes.NEOHOOKEAN, N=1000, seed=163)
    S, K, N = 10, 4, spec.n_particles
    rng = np.random.default_rng(164)
    vel = (np.array(box.velocity) + 0.3 * rng.standard_normal((S, 3))).astype(np.float32)
    om = (box.omega + 4.0 * rng.standard_normal(S)).astype(np.float32)
    cots = random_cotangents([spec, other], seed=165)
    cat = lambda k: torch.from_numpy(np.concatenate([c[k] for c in cots], axis=0))
    print("[schedules] unfused, driven collider", flush=True)
    b = Batch([spec, other], max_substeps=S, ckpt_every=K)
    b.set_option(C.OPT_FUSE, 0)
    b.set_option(C.OPT_FUSE_ADJ, 0)
    b.set_particles_from_specs()
    b.set_collider_motion(0, vel, om)
    b.forward(S, record=True)
    st = [to_np(t) for t in b.get_particles(env=0)]
    gr = [to_np(t)[:N] for t in b.backward(cat(0), cat(1), cat(2), cat(3))[:4]]
    dvel, dc0, dom, dang = b.collider_grad(0, S, spin=True)
    assert b.sync(raise_on_error=False) == 0
    b.close()
    env, prm, st0 = O.env_from_spec(spec)
    velt, omt = torch.from_numpy(vel).double(), torch.from_numpy(om).double()
    end, _ = O.rollout(env, prm, st0, S, vel=velt, omega=omt)
    c = tuple(torch.from_numpy(a).double() for a in cots[0])
    g, _, gvel, gc0, gom, gang = O.rollout_vjp(env, prm, st0, S, c, vel=velt, omega=omt)
    assert_state(st, [t.numpy() for t in end], spec.x, "driven, unfused", S=S)
    assert_grads(gr, [t.numpy() for t in g], "driven, unfused")
    e = [relerr(dvel, gvel.numpy()), relerr(dc0, gc0.numpy()), relerr(dom, gom.numpy()), abs(dang - float(gang)) / abs(float(gang))]
    print(f"[schedules] dL/d(vel, c0, omega, angle0) off by {e}", flush=True)
    assert np.abs(gom.numpy()).max() > 0 and abs(float(gang)) > 0
    assert max(e) < 1e-3
