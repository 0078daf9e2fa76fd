"""The training step's layers in tiles of 32 rows: batches around a tile, and
results and gradients in arrays that do not start on 16 bytes.
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


@pytest.mark.parametrize("B", [1, 31, 32, 33, 4095])
def test_row_tiles(rrt, B):
    """Forward within 2e-2 and gradients within 3e-2 relative L2 of the FP64
    network (bfloat16 between layers); a batch's rows do not depend on the
    rows beside them, nor the results on where the arrays start."""
    Wq, bq, w_dev, b_dev = _net(6)
    g = np.random.default_rng(B)
    x = _bf16(ref.encode(g.uniform(-1, 1, size=(B + 40, 6)))).cuda()
    dout = torch.from_numpy(g.normal(size=(B, ref.OUT)).astype(np.float32)).cuda()
    ws = rrt.mlp_workspace(B + 40, "cuda")
    longer = rrt.mlp_forward(w_dev, b_dev, x, workspace=ws)
    ws = rrt.mlp_workspace(B, "cuda")
    out = rrt.mlp_forward(w_dev, b_dev, x[:B], workspace=ws)
    assert torch.equal(out, longer[:B])
    grads = rrt.mlp_backward(w_dev, x[:B], dout, ws)
    off = torch.empty(B * ref.OUT + 1, device="cuda")[1:].view(B, ref.OUT)
    ws2 = rrt.mlp_workspace(B, "cuda")
    assert torch.equal(rrt.mlp_forward(w_dev, b_dev, x[:B], out=off, workspace=ws2), out)
    off.copy_(dout)
    again = rrt.mlp_backward(w_dev, x[:B], off, ws2)
    assert all(torch.equal(p, q) for p, q in zip(grads, again))
    xf = x[:B].float().cpu().numpy().astype(np.float64)
    y, cache = ref.forward(Wq, bq, xf)
    assert _rel(out.cpu().numpy(), y) <= 2e-2
    dWs, dbs = ref.backward(Wq, cache, dout.cpu().numpy().astype(np.float64))
    assert _rel(grads[0].cpu().numpy(), np.concatenate([d.ravel() for d in dWs])) <= 3e-2
    assert _rel(grads[1].cpu().numpy(), np.concatenate(dbs)) <= 3e-2


@pytest.mark.parametrize("B,at", [(33, 0), (4096, 0), (4096, 1024), (20000, 3072)])
def test_x_inside_out(rrt, B, at):
    """The encoded batch may lie in the array that the result is written to
    (`at`: 16-byte units from its start)."""
    _, _, w_dev, b_dev = _net(6)
    g = np.random.default_rng(B)
    x = _bf16(ref.encode(g.uniform(-1, 1, size=(B, 6)))).cuda()
    want = rrt.mlp_forward(w_dev, b_dev, x)
    out = torch.empty((B, ref.OUT), device="cuda")
    inside = out.view(-1).view(torch.bfloat16)[8 * at:8 * at + x.numel()].view(x.shape)
    inside.copy_(x)
    assert torch.equal(rrt.mlp_forward(w_dev, b_dev, inside, out=out), want)
