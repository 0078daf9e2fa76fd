"""Source map of a sparse lighting: the one-launch way equals the staged way
(scatter, inverse Haar transform) bit for bit, on both sides of the rule that
chooses between them, with repeated calls into the same workspace and with
entries outside the map.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rrt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_07272_amd as m
    return m


def strips(pix):
    """Row-major squares [6, n, n] -> strips of eight columns, row by row."""
    n = pix.shape[-1]
    if n < 8:
        return pix.reshape(-1)
    return pix.view(6, n, n // 8, 8).transpose(1, 2).reshape(-1)


@pytest.mark.parametrize("n,k", [(2, 24), (4, 17), (8, 100), (32, 6144), (64, 16384), (64, 16385),
                                 (128, 1), (128, 1024), (256, 10922), (256, 10923), (1024, 600)])
@pytest.mark.parametrize("half", [False, True])
def test_prepared_map(rrt, n, k, half):
    cells = 6 * n * n
    g = torch.Generator(device="cuda").manual_seed(n + k)
    ws = torch.full((8 * cells + 4096,), 0x7f, dtype=torch.uint8, device="cuda")
    for _ in range(2):                  # another lighting into the same workspace
        at = torch.randperm(cells, generator=g, device="cuda")[:k].sort().values.int()
        val = torch.randn(k, generator=g, device="cuda")
        val = val.half() if half else val
        dense = torch.zeros(cells, device="cuda")
        dense[at.long()] = val.float()
        want = strips(rrt.haar_inverse(dense.view(6, n, n)))
        if k > 2:
            at[0], at[1] = -1, cells    # outside the map: skipped
            dense[torch.arange(cells, device="cuda")] = 0.0
            dense[at[2:].long()] = val[2:].float()
            want = strips(rrt.haar_inverse(dense.view(6, n, n)))
        rrt.prepare_lighting(n, at.contiguous(), val.contiguous(), workspace=ws)
        off = (4 * cells + 255) // 256 * 256
        got = ws[off:off + 4 * cells].view(torch.float32)
        assert torch.equal(got.view(torch.int32), want.contiguous().view(torch.int32))


@pytest.mark.parametrize("n,k", [(64, 1500), (128, 1400), (256, 1500), (64, 16500)])
@pytest.mark.parametrize("half", [False, True])
def test_repeated_index(rrt, n, k, half):
    """Every square has one index three times, far apart in the list, with
    three values: the square is the inverse transform with one of them (the
    same in all of its tiles), bit for bit."""
    cells, g = 6 * n * n, torch.Generator(device="cuda").manual_seed(n + k)
    ws = torch.full((8 * cells + 4096,), 0x7f, dtype=torch.uint8, device="cuda")
    # scaling, the widest levels, the one above 32 x 32 tiles, a fine one
    twin = [0, 1, n + 1, 1, (n // 64) * n, (n - 3) * n + n // 2 + 5]
    at = torch.randperm(cells, generator=g, device="cuda")[:k].sort().values.int()
    for f, pos in enumerate(twin):
        at[at == f * n * n + pos] = -1
        for j in range(3):
            at[70 * (3 * f + j) + 5 * f] = f * n * n + pos
    for _ in range(4):
        val = 3 * torch.randn(k, generator=g, device="cuda")
        val = val.half() if half else val
        rrt.prepare_lighting(n, at, val, workspace=ws)
        off = (4 * cells + 255) // 256 * 256
        got = ws[off:off + 4 * cells].view(torch.int32).view(6, -1)
        once = at >= 0
        for f, pos in enumerate(twin):
            once &= at != f * n * n + pos
        dense = torch.zeros(cells, device="cuda")
        dense[at[once].long()] = val[once].float()
        same = torch.zeros(6, 3, dtype=torch.bool, device="cuda")
        for j in range(3):
            for f, pos in enumerate(twin):
                dense[f * n * n + pos] = val[70 * (3 * f + j) + 5 * f].float()
            want = strips(rrt.haar_inverse(dense.view(6, n, n))).contiguous().view(torch.int32).view(6, -1)
            same[:, j] = (got == want).all(1)
        assert bool(same.any(1).all()), same
