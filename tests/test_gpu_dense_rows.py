"""Dense rows (every coefficient in order, found by its position) and frames
divided among waves, against the FP64 checker with the FP32 bounds of the
parity tests: |got - ref| <= 1e-5 |ref| + 2e-7 s.
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


def scene(n, V, F, seed):
    from scenes.scene import random_rotations
    g = np.random.default_rng(seed)
    cells = 6 * n * n
    k = min(cells, 500)
    li = np.sort(g.choice(cells, k, replace=False)).astype(np.int32)
    lv = g.normal(size=k).astype(np.float32)
    rows = g.normal(size=(V, cells)).astype(np.float32)
    return (li, lv, random_rotations(seed, V), random_rotations(seed + 1, F) if F > 1 else None, rows)


@pytest.mark.parametrize("n,V,F,form", [(2, 5, 1, "f32"), (4, 3, 3, "s16"), (8, 2, 1, "bf16"),
                                        (16, 3, 2, "s11"), (32, 2, 1, "f32"), (64, 2, 3, "f32"),
                                        (64, 2, 1, "s11"), (128, 1, 2, "e4m3"), (512, 1, 1, "f32")])
@pytest.mark.parametrize("compensated", [False, True])
def test_dense_rows(rrt, n, V, F, form, compensated):
    from oracle.relight import relight
    li, lv, rot, frot, rows = scene(n, V, F, 40 + n)
    val, scale = dev(rows), None
    if form == "bf16":
        val = rrt.convert(val, "bf16")
        rows = val.float().cpu().numpy()
    elif form != "f32":
        # the same codes as sparse rows of all indices are read back as values
        val, scale = rrt.convert(val, form)
    out = rrt.relight(n, dev(li), dev(lv), dev(rot), None, val, block_scale=scale,
                      frame_rot=None if frot is None else dev(frot), compensated=compensated)
    if form in ("f32", "bf16"):
        check_frames(out.cpu().numpy(), relight(li, lv, n, rot, frot, None, rows, return_scale=True),
                     rel_l2=False)
    else:
        idx = torch.arange(6 * n * n, dtype=torch.int32, device="cuda").repeat(V, 1)
        want = rrt.relight(n, dev(li), dev(lv), dev(rot), idx, val, block_scale=scale,
                           frame_rot=None if frot is None else dev(frot), compensated=compensated)
        _, s = relight(li, lv, n, rot, frot, None, rows, return_scale=True)
        got, want = out.cpu().numpy(), want.cpu().numpy()
        # two evaluations of the same sum, each within its bound; the decoded
        # rows' scale is within a form's relative step (1/8) of the rows' own
        assert np.all(np.abs(got - want) <= 2 * (1e-5 * np.abs(want) + 2.25e-7 * s))


@pytest.mark.parametrize("V,F", [(1, 7), (3, 70), (700, 5)])
def test_frames_divided(rrt, V, F):
    """Every frame of every vertex is the single-frame call's result with that
    frame's rotation: the frames' division changes no value."""
    n = 32
    g = np.random.default_rng(V)
    li, lv, rot, frot, _ = scene(n, V, F, 7 * V)
    idx = np.sort(np.stack([g.choice(6 * n * n, 90, replace=False) for _ in range(V)]), 1).astype(np.int32)
    val = g.normal(size=idx.shape).astype(np.float32)
    args = (n, dev(li), dev(lv), dev(rot), dev(idx), dev(val))
    out = rrt.relight(*args, frame_rot=dev(frot))
    for f in range(0, F, max(1, F // 9)):
        one = rrt.relight(*args, frame_rot=dev(frot[f:f + 1]))
        assert torch.equal(out[f], one[0])


@pytest.mark.parametrize("H", [4, 32, 128])
def test_latlong_dense_rows(rrt, H):
    from oracle.latlong import relight_latlong
    g = np.random.default_rng(H)
    cells, V = 2 * H * H, 2
    li = np.sort(g.choice(cells, min(cells, 300), replace=False)).astype(np.int32)
    lv = g.normal(size=li.size).astype(np.float32)
    b = np.arccos(g.uniform(-1, 1, V))
    elev = np.stack([np.cos(b), np.sin(b)], 1).astype(np.float32)
    shift = g.integers(0, 2 * H, (V, 2)).astype(np.int32)
    rows = g.normal(size=(V, cells)).astype(np.float32)
    out = rrt.relight_latlong(H, dev(li), dev(lv), dev(elev), dev(shift), None, dev(rows))
    check_frames(out.cpu().numpy()[None], relight_latlong(li, lv, H, elev, shift, None, rows,
                                                          return_scale=True), rel_l2=False)


@pytest.mark.parametrize("n,V", [(4, 5120), (4, 5121), (16, 5121)])
@pytest.mark.parametrize("compensated", [False, True])
def test_faces_among_waves(rrt, n, V, compensated):
    """Up to 5,120 waves a vertex's faces are divided among six waves, above
    one wave takes them all."""
    from oracle.relight import relight
    li, lv, rot, _, rows = scene(n, V, 1, n + V)
    out = rrt.relight(n, dev(li), dev(lv), dev(rot), None, dev(rows), compensated=compensated)
    for at in (slice(0, 40), slice(V - 40, V)):
        ref = relight(li, lv, n, rot[at], None, None, rows[at], return_scale=True)
        check_frames(out[:, at].cpu().numpy(), ref, rel_l2=False)
