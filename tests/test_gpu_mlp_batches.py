"""Training steps at the batch sizes where the kernels split differently,
against the network oracle: a single row, below, at and above the 32 rows of a
tile and of a gradient slice, slices that are not 32 rows (33 and 100 rows),
batches that are and are not multiples of 8 (transposed or strided weight
gradients), split weight gradients (1,024 rows), and the last batch of the
small tiles and the first beyond.  Tolerances are those of the network tests.
The forward pass after the steps uses the weights' BF16 copies, plain and
transposed: it must equal that of a network given the same weights."""
import numpy as np
import pytest

from oracle import mlp as M
from paper_2203_14071_amd import rlf
from tests import gpu_common as G
from tests.test_gpu_mlp import _bf16_tensor, _init, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8, 31, 32, 33, 64, 100, 500, 1024, 1025, 3072, 3080])
def test_step_at_batch_edges(n):
    torch = G.torch_cuda()
    ctx = rlf.Context(0)
    p = _init(n)
    rng = np.random.default_rng(n + 1)
    x = M.bf16(rng.standard_normal((n, M.N_IN)) * 0.2)
    t = (rng.standard_normal((n, 3)) * 0.3).astype(np.float32)
    net = rlf.Mlp(ctx, max_batch=n)
    net.set_state(M.pack(p))
    loss = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    xd, td = _bf16_tensor(x), torch.from_numpy(t).to("cuda:0")
    net.train_step(xd, td, 1e-3, loss)
    ctx.sync()
    y, cache = M.forward(x, p)
    assert loss.item() == pytest.approx(M.loss(y, t.astype(np.float64)), rel=1e-4)
    g, gg = M.backward(p, cache, t.astype(np.float64)), M.unpack(net.get_state()["grad"])
    for k, _ in M.SHAPES:
        assert _rel(gg[k], g[k]) < 2e-3, (k, _rel(gg[k], g[k]))
    net.train_step(xd, td, 1e-3, loss)
    ctx.sync()
    other = rlf.Mlp(ctx, max_batch=n)
    other.set_state(net.get_state()["params"])
    out = [torch.empty((n, 6), dtype=torch.float32, device="cuda:0") for _ in range(2)]
    net.forward(xd, out[0])
    other.forward(xd, out[1])
    ctx.sync()
    assert torch.equal(out[0], out[1])
    net.free()
    other.free()
    ctx.close()
