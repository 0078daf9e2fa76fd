"""A vertex's blocks divided among eight, four, two or one wave, by the number
of vertices: vertices from the start and the end of the call against the FP64
checker with the FP32 bounds of the parity tests.
"""
import numpy as np
import pytest
import torch

from test_gpu_parity import check_frames, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rrt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_07272_amd as m
    return m


@pytest.mark.parametrize("n,V,nnz", [(64, 1280, 100), (64, 1281, 100), (64, 2561, 600), (128, 640, 100),
                                     (128, 641, 600), (256, 640, 60), (256, 2600, 60)])
@pytest.mark.parametrize("compensated", [False, True])
def test_blocks_among_waves(rrt, n, V, nnz, compensated):
    from oracle.relight import relight
    from scenes.scene import random_rotations
    g = np.random.default_rng(n + V)
    cells = 6 * n * n
    li = np.sort(g.choice(cells, 700, replace=False)).astype(np.int32)
    lv = g.normal(size=700).astype(np.float32)
    # all entries on two faces, a quarter of them in the levels above the blocks
    hi = np.where(g.random((V, nnz)) < 0.25, n // 32, n)
    ti = (g.integers(1, 3, (V, nnz)) * n * n + g.integers(0, hi) * n + g.integers(0, hi)).astype(np.int32)
    # (a repeated index counts once: the checker takes distinct entries)
    tv = g.normal(size=(V, nnz)).astype(np.float32)
    ti.sort(1)
    tv[:, 1:][ti[:, 1:] == ti[:, :-1]] = 0.0
    rot = random_rotations(n, V)
    out = rrt.relight(n, dev(li), dev(lv), dev(rot), dev(ti), dev(tv), compensated=compensated)
    for v in (0, 1, 2, V // 2, V - 2, V - 1):
        idx, first = np.unique(ti[v], return_index=True)
        ref = relight(li, lv, n, rot[v:v + 1], None, idx[None], tv[v:v + 1, first], return_scale=True)
        check_frames(out[:, v:v + 1].cpu().numpy(), ref, rel_l2=False)
