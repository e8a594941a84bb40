"""The FEM kernels on meshes where their split changes: one element, more than 256 nodes with one, two and four
elements per thread, and an element count near the largest with more than 64 KiB of LDS.

Bars: velocities and the cotangents of the state and the activations as in the other FEM tests. These bars are up
to 1.4 m long and move by a third of a millimetre, so a displacement is held to what storing a position of
that size in FP32 after every substep allows (half an ulp each time) and to the velocities' bar. The parameters'
cotangents are sums that cancel to any degree on such meshes; the other FEM tests check them."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_2412_12089_amd import fem_scenes as FS
from gpu_util import particle_maxerr, relerr
from test_gpu_fem import PER_NODE, TOL_GRAD, TOL_STATE, announce, oracle_env, run_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

H = 0.02


def block(a, b, c):
    return FS.cube_lattice_mesh([(i, j, k) for i in range(a) for j in range(b) for k in range(c)], H)


def union(*parts):
    X, tets, off, n = [], [], 0.0, 0
    for Xp, tp in parts:
        X.append(Xp - Xp.min(0) + [off, 0.0, 0.0])
        tets.append(tp + n)
        off, n = off + np.ptp(Xp[:, 0]) + H, n + len(Xp)
    return np.concatenate(X), np.concatenate(tets).astype(np.int32)


def one_tet():
    return H * np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]]), np.array([[0, 1, 2, 3]], dtype=np.int32)


MESHES = {  # mesh, nodes, elements
    "one": (one_tet, 4, 1),
    "nodes-256": (lambda: block(1, 1, 63), 256, 378),
    "islands": (lambda: union(*[one_tet()] * 65), 260, 65),
    "bar": (lambda: block(1, 1, 80), 324, 480),
    "long": (lambda: block(2, 2, 30), 279, 720),
    "lds-68k": (lambda: union(block(4, 5, 5), block(1, 1, 70)), 464, 1020),
}


@pytest.mark.parametrize("name", list(MESHES))
def test_meshes_match_oracle(name):
    make, n, T = MESHES[name]
    Xm, tets = make()
    assert (Xm.shape[0], tets.shape[0]) == (n, T)
    rng = np.random.default_rng(n + T)
    E, S = 2, 6
    X = np.stack([Xm + [0.1 * e, 0.0, 0.01 * e] for e in range(E)]).astype(np.float32)
    x0 = (X * np.array([1.02, 0.99, 1.0])).astype(np.float32)
    x0[:, :, 2] -= 0.0005
    v0 = (0.2 * rng.standard_normal((E, n, 3))).astype(np.float32)
    prm = np.tile([800.0, 1200.0, 1.0, 0.5, 200.0, 0.05, 0.05, 0.0], (E, 1))
    act = rng.uniform(-0.2, 0.2, size=(S, E, T)).astype(np.float32)
    w = FS.FemWorkload(name, tets, X, x0, v0, prm, act, 1e-4, S)
    announce(f"{name}: E {E} n {n} T {T} S {S}")
    gpu, gx, gv = run_gpu(w, seed=7)
    for e in range(E):
        o, og = oracle_env(w, e, gx, gv)
        x, v, dx, dv, da = (g[e] for g in gpu[:4] + [gpu[4].transpose(1, 0, 2)])
        ulp = np.spacing(np.abs(x).max().astype(np.float32)).astype(np.float64)
        far = np.abs(x - o[0]).max()
        bar = S * (0.5 * ulp + w.dt * PER_NODE * TOL_STATE * np.abs(o[1]).max())
        errs = dict(v=relerr(v, o[1]), v_n=particle_maxerr(v, o[1]) / PER_NODE)
        grads = dict(dx=relerr(dx, og[0]), dv=relerr(dv, og[1]), dact=relerr(da, og[2]))
        announce(f"{name} env {e}: x off by {far:.2e} of {bar:.2e} " +
                 " ".join(f"{k} {r:.2e}" for k, r in (errs | grads).items()))
        assert far < bar
        assert max(errs.values()) < TOL_STATE and max(grads.values()) < TOL_GRAD
