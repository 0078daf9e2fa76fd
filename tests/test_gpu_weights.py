"""Levels above the blocks as weights of the blocks: rows in any order, with
entries past the listed 512, repeated entries and entries that cancel over
part of a face, against the FP64 checker with the FP32 bounds of the parity
tests; and a triple product whose factor is zero on whole blocks, on single
texels of them, or nowhere.
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


def lighting(n, g, k=800):
    cells = 6 * n * n
    return (np.sort(g.choice(cells, k, replace=False)).astype(np.int32),
            g.normal(size=k).astype(np.float32))


@pytest.mark.parametrize("n,nnz,V", [(64, 700, 4), (128, 700, 3), (256, 40, 4), (512, 600, 1)])
@pytest.mark.parametrize("compensated", [False, True])
def test_coarse_entries_anywhere(rrt, n, nnz, V, compensated):
    """Coarse entries at the end of a shuffled row (past the list for 600 and
    more); rows 1.. hold a face's scaling and vertical top coefficient with equal
    values, whose weights cancel over half of the face."""
    from oracle.relight import relight
    from scenes.scene import random_rotations
    g = np.random.default_rng(n + nnz)
    li, lv = lighting(n, g)
    rows, vals = [], []
    for v in range(V):
        face = g.integers(0, 6, nnz)
        fine = g.random(nnz) < 0.8
        r = np.where(fine, g.integers(0, n, nnz), g.integers(0, max(n // 32, 2), nnz))
        c = np.where(fine, g.integers(0, n, nnz), g.integers(0, max(n // 32, 2), nnz))
        at = np.unique(face * n * n + r * n + c)
        at = np.concatenate([at, np.full(nnz - at.size, -1)])     # -1: no entry
        val = g.normal(size=nnz)
        order = np.argsort((r < n // 32) & (c < n // 32) if at.size != nnz else at % (n * n) < n)
        at, val = at[order], val[order]
        if v:
            at[:], val[:] = -1, 0.0
            at[:3] = [2 * n * n, 2 * n * n + n, 2 * n * n + 5 * n + 7]
            val[:3] = [0.75, 0.75 * (-1) ** v, 0.5]
        rows.append(at)
        vals.append(val)
    ti, tv = np.stack(rows).astype(np.int32), np.stack(vals).astype(np.float32)
    rot = random_rotations(n, V)
    out = rrt.relight(n, dev(li), dev(lv), dev(rot), dev(ti), dev(tv), compensated=compensated)
    # the checker takes one row of valid entries at a time
    for v in range(V):
        ok = ti[v] >= 0
        ref = relight(li, lv, n, rot[v:v + 1], None, ti[v:v + 1, ok], tv[v:v + 1, ok], return_scale=True)
        check_frames(out[:, v:v + 1].cpu().numpy(), ref, rel_l2=False)


def test_repeated_entries(rrt):
    """An index that a row holds three times counts three times, in the fine
    and in the coarse levels: the same as once with the sum of the values."""
    from scenes.scene import random_rotations
    n, g = 128, np.random.default_rng(3)
    li, lv = lighting(n, g)
    rot = random_rotations(5, 2)
    once = np.array([[7, 2 * n * n + 2, 2 * n * n + 90 * n + 17]] * 2, np.int32)
    val = np.array([[1.0, -0.5, 0.25], [0.5, 2.0, 1.0]], np.float32)
    a = rrt.relight(n, dev(li), dev(lv), dev(rot), dev(once), dev(4 * val))
    b = rrt.relight(n, dev(li), dev(lv), dev(rot), dev(np.concatenate([once] * 3, 1)),
                    dev(np.concatenate([val, val, 2 * val], 1)))
    assert torch.allclose(a, b, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("kind", ["half", "texel", "nowhere"])
def test_triple_zero_factors(rrt, kind):
    """With complete visibility rows the triple product is the double product
    with the texel product of the two factors (FP64 checker)."""
    from oracle.haar import haar_forward, haar_inverse
    from oracle.relight import relight
    from scenes.scene import random_rotations
    n, V, g = 64, 3, np.random.default_rng(11)
    li, lv = lighting(n, g)
    rot = random_rotations(9, V)
    brdf = np.abs(g.normal(size=(2, 6, n, n))).astype(np.float32)
    if kind == "half":
        brdf[:, :, n // 2:, :] = 0.0
        brdf[1, 3] = -0.0
    elif kind == "texel":                      # one texel of a block left
        brdf[:, :, 32:, 32:] = 0.0
        brdf[:, :, 63, 40] = 1.5
    mat = np.array([0, 1, 0], np.int32)
    nnz = 300
    ti = np.sort(np.stack([g.choice(6 * n * n, nnz, replace=False) for _ in range(V)]), 1).astype(np.int32)
    tv = g.normal(size=ti.shape).astype(np.float32)
    out = rrt.relight(n, dev(li), dev(lv), dev(rot), dev(ti), dev(tv), brdf=dev(brdf), material=dev(mat))
    dense = np.zeros((V, 6 * n * n))
    for v in range(V):
        dense[v, ti[v]] = tv[v]
        texels = haar_inverse(dense[v].reshape(6, n, n)) * brdf[mat[v]].astype(np.float64)
        dense[v] = haar_forward(texels).ravel()
    ref = relight(li, lv, n, rot, None, None, dense, return_scale=True)
    check_frames(out.cpu().numpy(), ref, rel_l2=False)


@pytest.mark.parametrize("n", [32, 64, 128])
def test_triple_with_ones(rrt, n):
    """A triple product whose factor is one everywhere is the double product,
    each within its FP32 bound of the same sum (a block without entries inside
    is summed in another order, so not bit for bit)."""
    from oracle.relight import relight
    from scenes.scene import random_rotations
    V, g = 6, np.random.default_rng(n)
    li, lv = lighting(n, g)
    rot = random_rotations(n, V)
    wide = g.integers(0, max(n // 16, 2), (V, 40, 2))
    ti = np.stack([np.unique(np.concatenate([
        (g.integers(0, 6, 40) * n + wide[v, :, 0]) * n + wide[v, :, 1],
        g.choice(6 * n * n, 200, replace=False)]))[:200] for v in range(V)]).astype(np.int32)
    tv = g.normal(size=ti.shape).astype(np.float32)
    args = (n, dev(li), dev(lv), dev(rot), dev(ti), dev(tv))
    double = rrt.relight(*args).cpu().numpy()
    triple = rrt.relight(*args, brdf=torch.ones(1, 6, n, n, device="cuda"),
                         material=torch.zeros(V, dtype=torch.int32, device="cuda")).cpu().numpy()
    ref, s = relight(li, lv, n, rot, None, ti, tv, return_scale=True)
    check_frames(double, (ref, s), rel_l2=False)
    assert np.all(np.abs(triple - double) <= 2 * (1e-5 * np.abs(ref) + 2e-7 * s))
