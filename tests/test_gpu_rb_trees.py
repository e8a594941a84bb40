"""The rigid-body kernels on trees where their walks change shape: one link, forests (several roots, one depth
level), stars, and chains one link below, at and above the depths where root paths take one more round of pointer
doubling and mass-matrix rows one more quad of entries. Bars of the other rigid-body tests: the condition number
of these mass matrices (about 1e4) times the FP32 rounding is 6e-4 of an acceleration, and a substep adds a
twentieth of a joint's speed at most."""
import pytest

from conftest import gpu_available
from paper_2412_12089_amd import rb_scenes as RS
from test_gpu_rb import announce, check, oracle, run_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

SHAPES = {  # links, parent of link i > 0
    "single": (1, None),
    "forest": (6, lambda i: -1),
    "forest-of-chains": (12, lambda i: -1 if i % 4 == 0 else i - 1),
    "star": (16, lambda i: 0),
    "wide-star": (33, lambda i: 0),
    "chain-2": (2, lambda i: i - 1),
    "chain-3": (3, lambda i: i - 1),
    "chain-4": (4, lambda i: i - 1),
    "chain-5": (5, lambda i: i - 1),
    "chain-8": (8, lambda i: i - 1),
    "chain-9": (9, lambda i: i - 1),
    "chain-17": (17, lambda i: i - 1),
    "binary": (31, lambda i: (i - 1) // 2),
}


@pytest.mark.parametrize("shape", list(SHAPES))
def test_tree_shapes_match_oracle(shape):
    n, parent = SHAPES[shape]
    w = RS.tree_batch(seed=n, n_links=n, n_envs=3, substeps=3)
    for i in range(1, n):
        w.links[i].parent = parent(i)
    announce(f"{shape}: E {w.n_envs} N {n} S {w.substeps}")
    gpu, gq, gqd = run_gpu(w, seed=n)
    o, og = oracle(w, gq, gqd)
    check(shape, w, gpu, o, og)
