"""The second pass of the backwards where its grid, its lanes and its stores have edges, against plain torch float64: more
segments than its grid has blocks along them (65 535), one segment with few and with many slots, row ends inside a block of
features, and weight gradients of the query/key normalisation at any float's address.

Tolerance: float32 sums of up to 5003 products, off by the order of their additions: 1e-5 of the 2-norm, as in the other
parity tests."""
import pytest
import torch

from paper_2605_17923_amd import lnmod

pytestmark = pytest.mark.gpu

EPS = 1e-6
TOL = 1e-5


def _rand(g, *shape, dt=torch.float32):
    return torch.randn(*shape, generator=g, device="cuda").to(dt)


def _close(name, got, want, tol=TOL):
    err = float((got.double() - want).norm() / want.norm().clamp_min(1e-30))
    assert err <= tol, "%s: relative error %.2e" % (name, err)


def _xhat(x):
    v = x.double()
    c = v - v.mean(-1, keepdim=True)
    return c * (c.square().mean(-1, keepdim=True) + EPS).rsqrt()


@pytest.mark.parametrize("D", [64, 136])
@pytest.mark.parametrize("packed", [False, True])
def test_more_segments_than_blocks(D, packed):
    n = 70003
    g = torch.Generator(device="cuda")
    g.manual_seed(D)
    lens = torch.randint(0, 4, (n,), generator=g, device="cuda") if packed else torch.full((n,), 1, device="cuda")
    lens[-1] = 3 if packed else 1
    cu = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), lens.cumsum(0)]).to(torch.int32)
    T = int(cu[-1])
    print("second pass, segments", n, "rows", T, "D", D, packed, flush=True)
    x, dy, scale, shift = _rand(g, T, D), _rand(g, T, D), _rand(g, n, D), _rand(g, n, D)
    if packed:
        _, mean, rstd = lnmod.forward_varlen(x, shift, scale, cu, EPS)
        dx, dshift, dscale = lnmod.backward_varlen(dy, x, scale, cu, mean, rstd, EPS)
    else:
        _, mean, rstd = lnmod.forward(x.view(n, 1, D), shift, scale, EPS)
        dx, dshift, dscale = lnmod.backward(dy.view(n, 1, D), x.view(n, 1, D), scale, mean, rstd, EPS)
    owner = torch.repeat_interleave(torch.arange(n, device="cuda"), lens)
    zero = torch.zeros(n, D, dtype=torch.float64, device="cuda")
    want_shift = zero.index_add(0, owner, dy.double())
    want_scale = zero.index_add(0, owner, dy.double() * _xhat(x))
    for part in (slice(0, 65535), slice(65535, 65536), slice(65536, n)):
        _close("dshift", dshift[part], want_shift[part])
        _close("dscale", dscale[part], want_scale[part])
    empty = lens == 0
    assert not packed or int(empty.sum()) > 10000
    assert not dshift[empty].any() and not dscale[empty].any()


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [8, 72, 264, 1536, 5128, 8192])
@pytest.mark.parametrize("rows", [1, 2, 5, 17, 130, 700, 5003])
def test_one_segment(D, rows, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(D + rows)
    print("second pass, one segment", D, rows, dt, flush=True)
    x, dy, u, dh = (_rand(g, 1, rows, D, dt=dt) for _ in range(4))
    scale, shift, gate = (_rand(g, 1, D, dt=dt) for _ in range(3))
    cu = torch.tensor([0, rows], dtype=torch.int32, device="cuda")
    _, mean, rstd = lnmod.forward(x, shift, scale, EPS)
    want_shift, want_scale = dy.double().sum(1), (dy.double() * _xhat(x)).sum(1)
    for stats in ((mean, rstd), (None, None)):
        _, dshift, dscale = lnmod.backward(dy, x, scale, *stats, EPS)
        _close("dshift", dshift, want_shift)
        _close("dscale", dscale, want_scale)
        # the same sample as a packed batch of one segment goes through the segment table: the same bits
        flat = [None if t is None else t.view(rows) for t in stats]
        _, pshift, pscale = lnmod.backward_varlen(dy[0], x[0], scale, cu, *flat, EPS)
        assert torch.equal(pshift, dshift) and torch.equal(pscale, dscale)
    h, _, mean, rstd = lnmod.gated_forward(x, u, gate, shift, scale, None, EPS)
    _, _, dgate, dshift, dscale = lnmod.gated_backward(dy, dh, h, u, gate, scale, mean, rstd, None, EPS)
    _close("gated dshift", dshift, dy.double().sum(1))
    xhat = (h.double() - mean.double().view(1, rows, 1)) * rstd.double().view(1, rows, 1)
    _close("gated dscale", dscale, (dy.double() * xhat).sum(1))


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [8, 104, 128, 200, 1536, 5120])
@pytest.mark.parametrize("rows", [1, 3, 601, 4100])
def test_weight_gradients_at_any_floats_address(D, rows, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(D * 7 + rows)
    print("second pass, weight gradients", D, rows, dt, flush=True)
    q, k, dqo, dko = (_rand(g, rows, D, dt=dt) for _ in range(4))
    wq, wk = (_rand(g, D, dt=dt) for _ in range(2))
    _, _, rq, rk = lnmod.qknorm_forward(q, k, wq, wk, EPS)
    dq, dk = torch.empty_like(q), torch.empty_like(k)
    ws = torch.empty(lnmod.lnmod_qknorm_backward_workspace_bytes(rows, D), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for off in (0, 1, 2, 3):
        # words around both gradients show a store that reaches beyond them
        buf = torch.full((2 * D + 12,), 77.0, device="cuda")
        dwq, dwk = buf[off + 1:off + 1 + D], buf[off + D + 4:off + 2 * D + 4]
        st = lnmod.lnmod_qknorm_backward(dqo, dko, q, k, wq, wk, rows, D, EPS, stream, rq, rk, dq, dk, dwq, dwk, ws, ws.numel(),
                                         0 if dt == torch.bfloat16 else 1)
        assert st == 0
        for name, dy, x, r, dw in (("dwq", dqo, q, rq, dwq), ("dwk", dko, k, rk, dwk)):
            _close(name, dw, (dy.double() * x.double() * r.double()[:, None]).sum(0))
        keep = torch.ones_like(buf, dtype=torch.bool)
        keep[off + 1:off + 1 + D] = False
        keep[off + D + 4:off + 2 * D + 4] = False
        assert (buf[keep] == 77.0).all()
