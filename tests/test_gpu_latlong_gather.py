"""Source-index exactness of the longitude-latitude rule at every map size:
the boundary estimates (next to the poles above all), the comparisons made
again with the rounded rho, the smallest maps, and (cos b, sin b) pairs that
are not of a rotation.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("H", [4, 8, 16, 32, 64, 256, 512])
def test_latlong_index_exact(H):
    """Rows of one finest-level coefficient on an integer-valued map whose
    neighbouring texels differ: a wrong texel moves a radiance by at least
    1/2; the reconstruction of values below 61 stays far below 0.1."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_07272_amd as rrt
    from oracle.haar import haar_forward
    from oracle.latlong import rotate
    s, i, j = np.meshgrid(np.arange(2), np.arange(H), np.arange(H), indexing="ij")
    tex = ((7 * i + 13 * j + 29 * s) % 61).astype(np.float64)
    light = haar_forward(tex).ravel().astype(np.float32)
    g = np.random.default_rng(H)
    h, V = H // 2, 5000
    r, c = g.integers(0, h, V), g.integers(0, h, V)
    r = np.where(g.random(V) < 0.3, g.choice([0, h - 1], V), r)      # more next to the poles
    quad = g.integers(0, 3, V)
    rows = (g.integers(0, 2, V) * H * H + (r + h * (quad != 0)) * H + c + h * (quad != 1)).astype(np.int32)
    pairs = [(1.0, 0.0), (-1.0, 0.0), (0.0, 1.0), (np.cos(1e-4), np.sin(1e-4)),
             (np.cos(np.pi / H), np.sin(np.pi / H)), (0.6, 0.8), (0.7, 0.1), (1.5, -0.2)]
    pairs += [(np.cos(b), np.sin(b)) for b in np.arccos(g.uniform(-1, 1, 4))]
    for cb, sb in pairs:
        e = np.array([cb, sb], np.float32)
        sh = g.integers(-3 * H, 3 * H, 2).astype(np.int32)
        out = rrt.relight_latlong(H, dev(np.arange(2 * H * H, dtype=np.int32)), dev(light),
                                  dev(np.tile(e, (V, 1))), dev(np.tile(sh, (V, 1))),
                                  dev(rows.reshape(V, 1)), dev(np.ones((V, 1), np.float32)))
        want = haar_forward(rotate(tex, e[0], e[1], sh[0], sh[1])).ravel()[rows]
        err = np.abs(out.cpu().numpy() - want)
        assert err.max() < 0.1, (H, e, sh, int((err >= 0.1).sum()), float(err.max()))


@pytest.mark.parametrize("H", [4, 64, 512])
def test_latlong_pairs_of_any_length(H):
    """(cos b, sin b) pairs that are no rotation's, from 1e-6 off the unit
    circle to zero and to both sides of 2^20, take the texels of the rule."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_07272_amd as rrt
    from oracle.haar import haar_forward
    from oracle.latlong import rotate
    s, i, j = np.meshgrid(np.arange(2), np.arange(H), np.arange(H), indexing="ij")
    tex = ((7 * i + 13 * j + 29 * s) % 61).astype(np.float64)
    light = haar_forward(tex).ravel().astype(np.float32)
    g = np.random.default_rng(H)
    h, V = H // 2, 3000
    quad = g.integers(0, 3, V)
    rows = (g.integers(0, 2, V) * H * H + (g.integers(0, h, V) + h * (quad != 0)) * H +
            g.integers(0, h, V) + h * (quad != 1)).astype(np.int32)
    for k, length in enumerate([1 + 2e-6, 1 - 3e-4, 1.01, 0.5, 3.0, 1e-3, 0.0, 2.0**20, 2.0**21, 1e-30]):
        b = g.uniform(0, 2 * np.pi)
        e = np.array([length, 0.0] if k % 3 == 0 else [length * np.cos(b), length * np.sin(b)], np.float32)
        sh = g.integers(-3 * H, 3 * H, 2).astype(np.int32)
        out = rrt.relight_latlong(H, dev(np.arange(2 * H * H, dtype=np.int32)), dev(light),
                                  dev(np.tile(e, (V, 1))), dev(np.tile(sh, (V, 1))),
                                  dev(rows.reshape(V, 1)), dev(np.ones((V, 1), np.float32)))
        want = haar_forward(rotate(tex, e[0], e[1], sh[0], sh[1])).ravel()[rows]
        assert np.abs(out.cpu().numpy() - want).max() < 0.1, (H, e, sh)
