"""Source-index exactness of the relight gather at the map sizes where its
index arithmetic changes (fewer than 16 fraction bits from n = 256 on, the
smallest and the largest maps), including quarters of a block that lie in one
source face, quarters that cross faces, ties between faces, directions of a
scaled rotation and matrices whose entries exceed one.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rrt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_07272_amd as m
    return m


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n", [8, 16, 32, 256, 512, 1024])
def test_gather_index_exact(rrt, n):
    """Every row holds one finest-level coefficient, so a radiance is
    (+-a +-b +-c +-d) / 2 of four gathered texels of an integer-valued map
    whose neighbouring texels all differ: a wrong texel moves it by at least
    1/2, while the reconstruction of values below 61 from at most ten
    binary32 levels stays far below 0.1."""
    from oracle.haar import haar_forward
    from oracle.sphere import quantise_rotation, rotate_pixels
    from scenes.scene import random_rotations
    f, i, j = np.meshgrid(np.arange(6), np.arange(n), np.arange(n), indexing="ij")
    tex = ((7 * i + 13 * j + 29 * f) % 61).astype(np.float64)
    light = haar_forward(tex).ravel().astype(np.float32)
    light_idx = np.arange(6 * n * n, dtype=np.int32)
    g = np.random.default_rng(n)
    h, V = n // 2, 6000
    r, c = g.integers(0, h, V), g.integers(0, h, V)
    edge = g.random(V) < 0.3           # more of the blocks along the faces' borders
    r = np.where(edge, g.choice([0, h - 1], V), r)
    quad = g.integers(0, 3, V)
    rows = (g.integers(0, 6, V) * n * n + (r + h * (quad != 0)) * n + c + h * (quad != 1)).astype(np.int32)
    c_, s_ = np.cos(np.pi / 4), np.sin(np.pi / 4)
    tilt = np.array([[c_, -s_, 0], [s_, c_, 0], [0, 0, 1]])
    R0 = random_rotations(900 + n, 2)
    for R in [R0[0], R0[1], tilt, np.array([[0, -1, 0], [1, 0, 0], [0, 0, 1.0]]), 0.5 * R0[0],
              np.diag([1.0, 1.25, 0.75])]:
        R = np.asarray(R, np.float32)
        out = rrt.relight(n, dev(light_idx), dev(light), dev(np.tile(R, (V, 1, 1))),
                          dev(rows.reshape(V, 1)), dev(np.ones((V, 1), np.float32)))
        want = haar_forward(rotate_pixels(tex, quantise_rotation(R, n))).ravel()[rows]
        err = np.abs(out.cpu().numpy()[0] - want)
        assert err.max() < 0.1, (n, R, int((err >= 0.1).sum()), float(err.max()))
