"""The backward entry points that write the parameter gradients in the I/O element type round the same
float32 sums once: bit for bit what the float32 entry points give, cast by torch.  Sizes: every form of the
second pass (one segment: four groups of lanes per wave; a few: two; many: one), feature blocks with a ragged
end, empty segments and batches without rows (zeros)."""
import numpy as np
import pytest
import torch

from paper_2605_17923_amd import lnmod

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _randn(g, *shape, dt):
    return torch.randn(*shape, generator=g, device="cuda").to(dt)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("lens,D", [([700], 1536), ([513, 2], 8), ([40, 0, 77, 1, 300, 9, 64], 2568),
                                    ([5] * 130, 1032), ([0, 0], 64)])
def test_reduced_gradients_are_the_float32_sums_rounded_once(lens, D, dtype):
    dt, n, T = DT[dtype], len(lens), sum(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    x, u, dy, dh = (_randn(g, T, D, dt=dt) for _ in range(4))
    gate, shift, scale = (_randn(g, n, D, dt=dt) for _ in range(3))
    _, mean, rstd = lnmod.forward_varlen(x, shift, scale, cu)
    a = lnmod.backward_varlen(dy, x, scale, cu, mean, rstd)
    b = lnmod._backward_varlen(dy, x, scale, cu, mean, rstd, 1e-6, io_grads=True)
    h, _, gm, gr = lnmod.gated_forward(x, u, gate, shift, scale, cu)
    c = lnmod.gated_backward(dy, dh, h, u, gate, scale, gm, gr, cu)
    d = lnmod._gated_backward(dy, dh, h, u, gate, scale, gm, gr, cu, 1e-6, io_grads=True)
    rq, rk = lnmod.qknorm_forward(x, u, shift[0], scale[0])[2:]
    e = lnmod.qknorm_backward(dy, dh, x, u, shift[0], scale[0], rq, rk)
    f = lnmod._qknorm_backward(dy, dh, x, u, shift[0], scale[0], rq, rk, 1e-6, io_grads=True)
    torch.cuda.synchronize()
    for want, got in ((a, b), (c, d), (e, f)):
        for w, t in zip(want, got):
            assert t.dtype == dt and torch.equal(t, w.to(dt))
