"""Decoder gradients and loss at the batch sizes where their split changes:
one row range written straight out, several ranges, a last range of few rows,
more rows than the partial sums have ranges for; and the loss on arrays that
do not start on 16 bytes.
"""
import numpy as np
import pytest
import torch

from oracle import mlp as ref
from test_gpu_mlp import _bf16, _net, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rrt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_07272_amd as m
    return m


@pytest.mark.parametrize("B", [1, 127, 129, 511, 1025, 4097, 9000])
def test_gradients_row_ranges(rrt, B):
    """The output layer's bias gradient is the column sum of the bfloat16
    gradient rows: at most B binary32 roundings of the sum of magnitudes.
    The others carry the bfloat16 activations between layers (3e-2)."""
    Wq, bq, w_dev, b_dev = _net(5)
    g = np.random.default_rng(B)
    x = _bf16(ref.encode(g.uniform(-1, 1, size=(B, 6))))
    dout = g.normal(size=(B, ref.OUT)).astype(np.float32)
    ws = rrt.mlp_workspace(B, "cuda")
    rrt.mlp_forward(w_dev, b_dev, x.cuda(), workspace=ws)
    first = [t.cpu().numpy() for t in rrt.mlp_backward(w_dev, x.cuda(), torch.from_numpy(dout).cuda(), ws)]
    again = [t.cpu().numpy() for t in rrt.mlp_backward(w_dev, x.cuda(), torch.from_numpy(dout).cuda(), ws)]
    assert all(np.array_equal(a, b) for a, b in zip(first, again))   # the forward's values are kept
    dw, db = first
    rounded = _bf16(dout).float().numpy().astype(np.float64)
    err = np.abs(db[-ref.OUT:] - rounded.sum(0))
    assert np.all(err <= B * 2.0 ** -24 * np.abs(rounded).sum(0))
    _, cache = ref.forward(Wq, bq, x.float().numpy().astype(np.float64))
    dWs, dbs = ref.backward(Wq, cache, dout.astype(np.float64))
    wo = bo = 0
    for l, (o, i) in enumerate(ref.shapes()):
        assert _rel(dw[wo:wo + o * i].reshape(o, i), dWs[l]) <= 3e-2, l
        assert _rel(db[bo:bo + o], dbs[l]) <= 3e-2, l
        wo += o * i
        bo += o


@pytest.mark.parametrize("B", [1, 63, 65, 4096, 4500, 9000])
def test_bias_gradient_order(rrt, B):
    """The output layer's bias gradient is the binary32 sum of ranges of 64
    rows, added in order, at most 64 ranges at a time: the same bits."""
    _, _, w_dev, b_dev = _net(5)
    g = np.random.default_rng(B)
    x = _bf16(ref.encode(g.uniform(-1, 1, size=(B, 6)))).cuda()
    dout = g.normal(size=(B, ref.OUT)).astype(np.float32)
    ws = rrt.mlp_workspace(B, "cuda")
    rrt.mlp_forward(w_dev, b_dev, x, workspace=ws)
    _, db = rrt.mlp_backward(w_dev, x, torch.from_numpy(dout).cuda(), ws)
    dz = np.zeros((-(-B // 64) * 64, ref.OUT), np.float32)
    dz[:B] = _bf16(dout).float().numpy()
    dz = dz.reshape(-1, 64, ref.OUT)
    ranges = np.zeros((len(dz), ref.OUT), np.float32)
    for r in range(64):
        ranges += dz[:, r]
    total = None
    for c0 in range(0, len(dz), 64):
        s = np.zeros(ref.OUT, np.float32)
        for part in ranges[c0:c0 + 64]:
            s = s + part
        total = s if total is None else total + s
    assert np.array_equal(db[-ref.OUT:].cpu().numpy(), total)


@pytest.mark.parametrize("count,offset", [(1, 0), (7, 0), (4096, 1), (300003, 0), (300004, 3)])
def test_loss_alignment(rrt, count, offset):
    """dout is one subtraction, an exact doubling and one division (two
    roundings); the loss is summed in 64 bits over rounded differences."""
    g = torch.Generator(device="cuda").manual_seed(count)
    a, b = (torch.randn(count + offset, generator=g, device="cuda")[offset:] for _ in range(2))
    d = torch.empty(count + offset, device="cuda")[offset:]
    dout, loss = rrt.mse(a, b, dout=d)
    want = 2.0 * (a.double() - b.double()) / count
    assert torch.all((dout.double() - want).abs() <= 2.0 ** -22 * want.abs() + 1e-30)
    ref_loss = ((a.double() - b.double()) ** 2).mean().item()
    assert abs(loss.item() - ref_loss) <= 2.0 ** -22 * ref_loss
