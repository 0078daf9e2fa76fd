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


def rows_over(n, squares, V, nnz, g):
    """Rows over all squares, a quarter of the entries in the levels above the blocks."""
    hi = np.where(g.random((V, nnz)) < 0.25, max(n // 32, 2), n)
    ti = g.integers(0, squares, (V, nnz)) * n * n + g.integers(0, hi) * n + g.integers(0, hi)
    ti.sort(1)
    tv = g.normal(size=(V, nnz)).astype(np.float32)
    tv[:, 1:][ti[:, 1:] == ti[:, :-1]] = 0.0
    return ti.astype(np.int32), tv


def assert_same(got, want):
    """The division among waves only moves sums in FP64, by a few 2^-53 of
    their terms, so a binary32 result changes where it lies that close to the
    middle of two values: one place, for fewer than one value in a thousand."""
    got, want = got.cpu().numpy().ravel(), want.cpu().numpy().ravel()
    assert np.all(np.abs(got - want) <= np.spacing(np.abs(want)))
    assert np.count_nonzero(got != want) <= got.size // 1000


@pytest.mark.parametrize("n", [64, 128, 256])
@pytest.mark.parametrize("kind", ["double", "compensated", "triple", "chain", "latlong"])
def test_vertex_alone(rrt, n, kind):
    """A vertex relit with 39, 699, 1,299, 2,599 and 5,199 others has the same
    value: eight, four, two and one wave each."""
    from scenes.scene import random_rotations
    g, V, squares = np.random.default_rng(n), 5200, 2 if kind == "latlong" else 6
    cells = squares * n * n
    li = np.sort(g.choice(cells, 700, replace=False)).astype(np.int32)
    lv = g.normal(size=700).astype(np.float32)
    ti, tv = rows_over(n, squares, V, 60, g)
    light = (n, dev(li), dev(lv))
    if kind == "latlong":
        b = np.arccos(g.uniform(-1, 1, V))
        rows = [np.stack([np.cos(b), np.sin(b)], 1).astype(np.float32),
                g.integers(0, 2 * n, (V, 2)).astype(np.int32), ti, tv]
        call, more = rrt.relight_latlong, {}
    else:
        rows, call, more = [random_rotations(n, V), ti, tv], rrt.relight, {}
        if kind == "triple":
            more = {"brdf": dev(np.abs(g.normal(size=(1, 6, n, n))).astype(np.float32))}
        elif kind != "double":
            more = {"compensated": kind == "compensated", "chain_rule": kind == "chain"}
    rows = [dev(x) for x in rows]
    if kind == "triple":
        more["material"] = torch.zeros(V, dtype=torch.int32, device="cuda")
    out = []
    for count in (40, 700, 1300, 2600, V):
        part = dict(more, material=more["material"][:count]) if kind == "triple" else more
        out.append(call(*light, *(x[:count] for x in rows), **part).reshape(-1)[:40].clone())
    for other in out[1:]:
        assert_same(other, out[0])


@pytest.mark.parametrize("n,nnz", [(64, 60), (128, 600)])
@pytest.mark.parametrize("F", [16, 17, 32, 33, 64, 65])
def test_frame_alone(rrt, n, nnz, F):
    """40 vertices in 16 to 65 frames (the parts of the frames times the
    vertices on both sides of 640, 1,280 and 2,560) have the values of calls
    with one frame, and those of the FP64 oracle."""
    from oracle.relight import relight
    from scenes.scene import random_rotations
    g, V = np.random.default_rng(n), 40
    li = np.sort(g.choice(6 * n * n, 700, replace=False)).astype(np.int32)
    lv = g.normal(size=700).astype(np.float32)
    ti, tv = rows_over(n, 6, V, nnz, g)
    rot, frot = random_rotations(n, V), random_rotations(n + 1, F)
    args = (n, dev(li), dev(lv), dev(rot), dev(ti), dev(tv))
    out = rrt.relight(*args, frame_rot=dev(frot))
    for f in range(0, F, 5):
        assert_same(out[f], rrt.relight(*args, frame_rot=dev(frot[f:f + 1]))[0])
    for v in (0, V - 1):
        idx, first = np.unique(ti[v], return_index=True)
        ref = relight(li, lv, n, rot[v:v + 1], frot, idx[None], tv[v:v + 1, first], frames=[0, F - 1],
                      return_scale=True)
        check_frames(out[[0, F - 1], v:v + 1].cpu().numpy(), ref, rel_l2=False)
