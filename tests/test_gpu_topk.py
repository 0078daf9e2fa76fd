"""Selection at the sizes and contents where its way changes: the workgroup
sizes, lengths past the position bits, unaligned rows, more equal keys than
the candidate list holds, thresholds among the zeros, and k = len.  Positions
and values are compared bit for bit with the checker's.
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


def rows_of(kind, rows, length, g):
    x = g.normal(size=(rows, length)).astype(np.float32)
    if kind == "sparse":                    # most values zero, of either sign
        x[g.random(x.shape) < 0.97] = 0.0
        x[:, 1::2] *= np.float32(-1.0)
    elif kind == "constant":
        x = np.where(g.random(x.shape) < 0.5, -1.5, 1.5).astype(np.float32)
    elif kind == "near":                    # one top-bits bin, ties among its keys
        x = (np.float32(1.0) + g.integers(0, 50, x.shape).astype(np.float32) * np.float32(2.0 ** -23))
    elif kind == "few":                     # a few hundred different keys, many times
        x = (g.integers(1, 300, x.shape).astype(np.float32) * np.float32(2.0 ** -20)) * np.sign(x)
    elif kind == "extreme":
        x[:, 0::5] = np.inf
        x[:, 1::5] = -np.finfo(np.float32).max
        x[:, 2::5] = np.float32(1e-45)      # the smallest subnormal
    return x


@pytest.mark.parametrize("rows,length,k,kind", [
    (9, 8192, 100, "normal"), (9, 8193, 100, "normal"), (20, 98304, 256, "sparse"),
    (11, 98304, 5000, "sparse"), (10, 12288, 700, "constant"), (10, 12289, 3000, "near"),
    (2, 131072, 1024, "normal"), (2, 131076, 1024, "near"), (1, 393216, 2048, "sparse"),
    (1, 393217, 2048, "sparse"), (9, 393220, 300, "normal"), (3, 1536, 300, "extreme"),
    (12, 9000, 4000, "extreme"), (70, 384, 383, "normal"), (70, 384, 384, "normal"),
    (200, 1536, 600, "sparse"), (12, 1536, 1200, "few"), (12, 98304, 20000, "few"),
    (4, 31, 30, "near"), (1, 98304, 98304, "normal"), (1, 98304, 98303, "sparse"),
])
def test_topk_ways(rrt, rows, length, k, kind):
    from oracle.select import topk_abs
    x = rows_of(kind, rows, length, np.random.default_rng(rows + length + k))
    idx, val = (t.cpu().numpy() for t in rrt.topk(torch.from_numpy(x).cuda(), k))
    for r in range(rows):
        want = topk_abs(x[r], k)
        assert np.array_equal(idx[r], want), (r, int((idx[r] != want).sum()))
        assert np.array_equal(val[r].view(np.uint32), x[r][want].view(np.uint32))


def room(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib * 2**30:
        pytest.skip(f"needs {gib} GiB of device memory")


def test_topk_all_past_a_launch(rrt):
    """k = len of more values than one launch has threads (2^32)."""
    room(70)
    rows, length = (1 << 26) + 3, 64
    x = torch.empty((rows, length), device="cuda").uniform_()
    idx, val = rrt.topk(x, length)
    assert torch.equal(val, x)
    del val, x
    assert bool((idx == torch.arange(length, dtype=torch.int32, device="cuda")).all())


def test_topk_rows_past_a_launch(rrt):
    """As many rows as 1,024 threads each are 2^32."""
    room(160)
    rows, length = 1 << 22, 8193
    x = torch.zeros((rows, length), device="cuda")
    at = (torch.arange(rows, device="cuda") * 7919 % length).view(-1, 1)
    x.scatter_(1, at, -2.0)
    idx, val = rrt.topk(x, 1)
    del x
    assert torch.equal(idx.long(), at)
    assert bool((val == -2.0).all())
