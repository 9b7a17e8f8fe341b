"""Every entry of the launch-shape tables, of every family, against plain torch float64 on the same inputs: one width
per 256 features, once with rows that are not whole 128-byte lines (one chunk short of the multiple of 256) and once
with rows that are (64 features short), on launches beyond the short ones (more than 72 MB of x) and on short ones
(2 MB and 20 MB), three samples of unequal alignment to the blocks' steps.  The per-token backward in its three forms:
with dshift, without it, and with the statistics formed again.  Then the forward on many short segments, whose shape
depends on the width, the size of the launch and the rows per segment.

Tolerances: bf16 results are rounded once (2^-9 relative, 1.7e-3 in the 2-norm; 4e-3 allowed); fp32 results and
the float32 sums over 60 to 200 000 rows are off by the order of their additions (1e-5 of the 2-norm)."""
import pytest
import torch

from paper_2605_17923_amd import lnmod

pytestmark = pytest.mark.gpu

EPS = 1e-6


def _close(name, got, want, tol):
    err = float((got.double() - want).norm() / want.norm())
    assert err <= tol, "%s: relative error %.2e" % (name, err)


def _ln(x, dy, scale, rms=False):
    """(xhat, rstd, dx) of one sample in float64; scale is what multiplies xhat."""
    c = x if rms else x - x.mean(-1, keepdim=True)
    rstd = (c.square().mean(-1, keepdim=True) + EPS).rsqrt()
    xhat, g = c * rstd, dy * scale
    dx = g - xhat * (g * xhat).mean(-1, keepdim=True)
    return xhat, rstd, (dx if rms else dx - g.mean(-1, keepdim=True)) * rstd


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("aligned", [False, True], ids=["unaligned", "aligned"])
@pytest.mark.parametrize("i", range(1, 33))
def test_every_long_entry_against_float64(i, aligned, dtype):
    _every_operator(i, aligned, dtype, 74e6)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("aligned", [False, True], ids=["unaligned", "aligned"])
@pytest.mark.parametrize("i", range(1, 33))
def test_every_short_entry_against_float64(i, aligned, dtype):
    _every_operator(i, aligned, dtype, 2e6)
    _every_operator(i, aligned, dtype, 20e6)


def _every_operator(i, aligned, dtype, nbytes):
    dt, e = (torch.bfloat16, 2) if dtype == "bf16" else (torch.float32, 4)
    D = 256 * i - (64 if aligned else 16 // e)
    B = 3
    S = int(nbytes / e / D / B) + 1
    tol = 4e-3 if e == 2 else 1e-5
    g = torch.Generator(device="cuda")
    g.manual_seed(i)

    def rand(*s):
        return torch.randn(*s, generator=g, device="cuda").to(dt)

    x, u, dy, dh = (rand(B, S, D) + (0.5 if k == 0 else 0.0) for k in range(4))
    gate, shift, scale = (rand(B, D) * 0.3 for _ in range(3))
    y, mean, rstd = lnmod.forward(x, shift, scale, EPS)
    dx, dsh, dsc = lnmod.backward(dy, x, scale, mean, rstd, EPS)
    rx, rsh, rsc = lnmod.backward(dy, x, scale, None, None, EPS)
    h, yh, gm, gr = lnmod.gated_forward(x, u, gate, shift, scale, eps=EPS)
    gdx, gdu, dg, gsh, gsc = lnmod.gated_backward(dy, dh, h, u, gate, scale, gm, gr, eps=EPS)
    qn, kn, rq, rk = lnmod.qknorm_forward(x, u, shift[0], scale[0], EPS)
    dq, dk, dwq, dwk = lnmod.qknorm_backward(dy, dh, x, u, shift[0], scale[0], rq, rk, EPS)
    tsc, tsh = rand(B, S, D) * 0.3, rand(B, S, D) * 0.3
    ty, tm, tr = lnmod.forward(x, tsh, tsc, EPS)
    tdx, tdsh, tdsc = lnmod.backward(dy, x, tsc, tm, tr, EPS)
    tdx2, tdsh2, tdsc2 = lnmod.backward(dy, x, tsc, None, None, EPS)
    ndx, ndsc = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    code = lnmod.LNMOD_BF16 if e == 2 else lnmod.LNMOD_F32
    stream = torch.cuda.current_stream().cuda_stream
    assert lnmod.lnmod_backward_token(dy, x, tsc, B, S, D, EPS, stream, tm, tr, ndx, ndsc, code) == lnmod.LNMOD_OK
    # the same waves and chunks per lane as with dshift, so the same sums of a row
    assert torch.equal(ndx, tdx) and torch.equal(ndsc, tdsc)
    for b in range(B):
        xd, ud, dyd, dhd = (t[b].double() for t in (x, u, dy, dh))
        A = 1.0 + scale[b].double()
        xhat, rs, want = _ln(xd, dyd, A)
        _close("y", y[b], xhat * A + shift[b].double(), tol)
        _close("rstd", rstd[b], rs[:, 0], 1e-5)
        for name, t, s, c in (("saved", dx, dsh, dsc), ("recomputed", rx, rsh, rsc)):
            _close("dx " + name, t[b], want, tol)
            _close("dshift " + name, s[b], dyd.sum(0), 1e-5)
            _close("dscale " + name, c[b], (dyd * xhat).sum(0), 1e-5)
        TA = 1.0 + tsc[b].double()
        _close("per-token y", ty[b], xhat * TA + tsh[b].double(), tol)
        want = _ln(xd, dyd, TA)[2]
        _close("per-token dx", tdx[b], want, tol)
        _close("per-token dx recomputed", tdx2[b], want, tol)
        _close("per-token dscale", tdsc[b], dyd * xhat, tol)
        _close("per-token dscale recomputed", tdsc2[b], dyd * xhat, tol)
        assert torch.equal(tdsh[b], dy[b]) and torch.equal(tdsh2[b], dy[b])
        hd = h[b].double()
        _close("h", h[b], xd + gate[b].double() * ud, tol)
        hhat, _, want = _ln(hd, dyd, A)
        want = want + dhd
        _close("gated y", yh[b], hhat * A + shift[b].double(), tol)
        _close("gated dx", gdx[b], want, tol)
        _close("gated du", gdu[b], want * gate[b].double(), tol)
        _close("dgate", dg[b], (want * ud).sum(0), 1e-5)
        _close("gated dscale", gsc[b], (dyd * hhat).sum(0), 1e-5)
        _close("gated dshift", gsh[b], dyd.sum(0), 1e-5)
    for name, t, w, d, out, grad, dw in (("q", x, shift[0], dy, qn, dq, dwq), ("k", u, scale[0], dh, kn, dk, dwk)):
        td, wd, dd = t.double().reshape(-1, D), w.double(), d.double().reshape(-1, D)
        that, _, want = _ln(td, dd, wd, rms=True)
        _close(name, out.reshape(-1, D), that * wd, tol)
        _close("d" + name, grad.reshape(-1, D), want, tol)
        _close("dw" + name, dw, (dd * that).sum(0), 1e-5)


@pytest.mark.parametrize("megabytes", [3, 30, 100, 210])
@pytest.mark.parametrize("D", [256, 440, 712, 768, 1000, 1024, 1232, 1280, 1400, 1408, 1536, 2560, 5312])
def test_forward_on_many_short_segments(D, megabytes):
    g = torch.Generator(device="cuda")
    g.manual_seed(D + megabytes)
    T = int(megabytes * 1e6 / 2 / D)
    x = torch.randn(T, D, generator=g, device="cuda", dtype=torch.bfloat16) + 0.5
    for mean in (40, 150, 300, 700):
        n = T // mean + 1
        cuts = torch.randint(0, T + 1, (n - 1,), generator=g, device="cuda").sort().values       # empty ones among them
        cu = torch.cat([cuts.new_zeros(1), cuts, cuts.new_full((1,), T)]).to(torch.int32)
        shift, scale = (torch.randn(n, D, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
        y, mu, rstd = lnmod.forward_varlen(x, shift, scale, cu, EPS)
        seg = torch.repeat_interleave(torch.arange(n, device="cuda"), (cu[1:] - cu[:-1]).long(), output_size=T)
        err = ref = 0.0
        for r in range(0, T, 1 << 16):
            v = x[r:r + (1 << 16)].double()
            c = v - v.mean(-1, keepdim=True)
            rs = (c.square().mean(-1, keepdim=True) + EPS).rsqrt()
            m = seg[r:r + (1 << 16)]
            want = c * rs * (1.0 + scale[m].double()) + shift[m].double()
            d = y[r:r + (1 << 16)].double() - want
            err, ref = err + float(d.square().sum()), ref + float(want.square().sum())
            # every row by itself too: a row with another segment's modulation would hide in the whole
            assert float((d.norm(dim=-1) / want.norm(dim=-1)).max()) <= 4e-3
            _close("rstd", rstd[r:r + (1 << 16)], rs[:, 0], 1e-5)
        assert (err / ref) ** 0.5 <= 4e-3
