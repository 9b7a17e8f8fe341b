"""The launch shapes that the size rules name, each run once at a width, size and segment count on its side of the lines, and
once beyond them: plain operator (both element types, with and without statistics), gated operator, query/key normalisation,
against plain torch float64.

Tolerances as in the other size-class tests: bf16 results are rounded once (2^-9 relative, 1.7e-3 in the 2-norm; 4e-3
allowed), float32 results and float32 sums over up to 80 000 rows are off by the order of their additions (1e-5)."""
import pytest
import torch

from paper_2605_17923_amd import lnmod

pytestmark = pytest.mark.gpu

EPS = 1e-6
TYPES = {"bf16": (torch.bfloat16, 4e-3), "f32": (torch.float32, 1e-5)}


def _close(name, got, want, tol):
    err = float((got.double() - want).norm() / want.norm())
    assert err <= tol, "%s: relative error %.2e" % (name, err)


def _make(D, mb, dtype, seed):
    dt = TYPES[dtype][0]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return int(mb * 1e6) // (D * dt.itemsize), lambda *s: torch.randn(*s, generator=g, device="cuda").to(dt)


def _lengths(rows, segments):
    """`segments` lengths that add up to rows, no two alike, one of a single row where there are three or more."""
    if segments == 1:
        return [rows]
    base = rows // segments
    lens = [max(1, base + (i - segments // 2) * (base // (2 * segments))) for i in range(segments)]
    if segments >= 3:
        lens[1] = 1
    lens[-1] += rows - sum(lens)
    assert min(lens) >= 1 and sum(lens) == rows
    return lens


def _cuts(lens):
    cu = torch.tensor([0] + lens, dtype=torch.int32, device="cuda").cumsum(0).to(torch.int32)
    at = 0
    rows = []
    for n in lens:
        rows.append(slice(at, at + n))
        at += n
    return cu, rows


def _norm(v):
    c = v - v.mean(-1, keepdim=True)
    rs = (c.square().mean(-1, keepdim=True) + EPS).rsqrt()
    return c * rs, rs


def _ln_backward(d, scale, h, rs):
    gr = d * (1.0 + scale)
    return (gr - gr.mean(-1, keepdim=True) - h * (gr * h).mean(-1, keepdim=True)) * rs


@pytest.mark.parametrize("D,mb,dtype,segments", [
    # forward
    (1152, 30, "bf16", 1), (1152, 30, "bf16", 3), (4096, 30, "bf16", 4), (4096, 30, "bf16", 5), (3584, 40, "bf16", 2),
    (3584, 60, "bf16", 2), (5904, 20, "bf16", 1), (5904, 28, "bf16", 2), (5904, 28, "bf16", 1), (800, 100, "bf16", 1),
    (896, 100, "bf16", 2), (880, 100, "bf16", 2), (1640, 100, "bf16", 3), (1728, 100, "bf16", 3), (4400, 100, "bf16", 12),
    (4400, 100, "bf16", 13), (5120, 100, "bf16", 1), (5120, 170, "bf16", 3), (3072, 15, "bf16", 2), (3072, 40, "bf16", 1),
    (3072, 100, "bf16", 2), (2824, 100, "bf16", 3), (4088, 100, "bf16", 2), (5112, 100, "bf16", 2), (1536, 9, "bf16", 8),
    (1536, 15, "bf16", 40), (1536, 40, "bf16", 60), (2560, 11, "f32", 2), (2560, 40, "f32", 3), (6144, 40, "f32", 1),
    (6144, 40, "f32", 6), (6144, 30, "f32", 5),
    # backward, with and without statistics
    (1152, 0.9, "bf16", 1), (1152, 0.9, "bf16", 3), (1152, 10, "bf16", 5), (5120, 3, "bf16", 1), (5120, 10, "bf16", 3),
    (1000, 22, "bf16", 1), (1000, 40, "bf16", 2), (1000, 100, "bf16", 2), (1000, 160, "bf16", 5), (2264, 30, "bf16", 2),
    (2264, 50, "bf16", 2), (1400, 100, "bf16", 4), (1400, 100, "bf16", 5), (1344, 100, "bf16", 2), (3400, 100, "bf16", 3),
    (636, 100, "f32", 9), (712, 100, "f32", 4), (712, 100, "f32", 5),
    (2048, 0.8, "bf16", 1), (2048, 0.8, "bf16", 2), (1768, 0.9, "bf16", 1), (2560, 0.9, "bf16", 2), (2560, 1.5, "bf16", 1),
    (2264, 0.9, "bf16", 1), (2264, 3, "bf16", 1), (2264, 6, "bf16", 3), (3072, 1.5, "bf16", 1), (3072, 3, "bf16", 2),
    (3072, 13, "bf16", 4), (3072, 13, "bf16", 5), (2600, 13, "bf16", 2), (3384, 1, "bf16", 2), (3384, 13, "bf16", 12),
    (3584, 18, "bf16", 8), (3584, 18, "bf16", 9), (5264, 10, "bf16", 4), (5264, 10, "bf16", 5), (5888, 4, "bf16", 1),
    (5888, 10, "bf16", 3), (640, 40, "bf16", 1), (640, 40, "bf16", 2), (640, 60, "bf16", 1), (1768, 30, "bf16", 3),
    (1768, 60, "bf16", 3), (2048, 100, "bf16", 3), (2048, 100, "bf16", 65), (1000, 76, "bf16", 2), (4016, 76, "bf16", 2),
])
def test_plain(D, mb, dtype, segments):
    rows, rand = _make(D, mb, dtype, D + segments)
    dt, tol = TYPES[dtype]
    lens = _lengths(rows, segments)
    cu, cuts = _cuts(lens)
    print("size rule", D, mb, dtype, rows, segments, flush=True)
    x, dy, shift, scale = rand(rows, D), rand(rows, D), rand(segments, D), rand(segments, D)
    if segments == 1:
        y, mean, rstd = lnmod.forward(x[None], shift, scale, EPS)
        both = [lnmod.backward(dy[None], x[None], scale, *st, EPS) for st in ((mean, rstd), (None, None))]
        y, both = y[0], [(a[0], b, c) for a, b, c in both]
    else:
        y, mean, rstd = lnmod.forward_varlen(x, shift, scale, cu, EPS)
        both = [lnmod.backward_varlen(dy, x, scale, cu, *st, EPS) for st in ((mean, rstd), (None, None))]
    for m, r in enumerate(cuts):
        d, a = dy[r].double(), scale[m].double()
        h, rs = _norm(x[r].double())
        _close("y", y[r], h * (1.0 + a) + shift[m].double(), tol)
        dx = _ln_backward(d, a, h, rs)
        for dxg, dsh, dsc in both:
            _close("dx", dxg[r], dx, tol)
            _close("dshift", dsh[m], d.sum(0), 1e-5)
            _close("dscale", dsc[m], (d * h).sum(0), 1e-5)


@pytest.mark.parametrize("D,mb,segments", [
    (696, 3, 2), (696, 10, 1), (696, 40, 3), (696, 100, 4), (696, 100, 5), (1000, 100, 2), (1000, 210, 2), (1000, 210, 5),
    (1000, 1, 2), (1912, 100, 2), (1912, 1, 1), (2560, 1, 2), (2560, 14, 3), (3584, 40, 8), (3584, 40, 9), (2656, 10, 2),
    (2656, 40, 3)])
def test_gated(D, mb, segments):
    rows, rand = _make(D, mb, "bf16", D * 3 + segments)
    lens = _lengths(rows, segments)
    cu, cuts = _cuts(lens)
    print("size rule, gated", D, mb, rows, segments, flush=True)
    x, u, dy, dh = (rand(rows, D) for _ in range(4))
    gate, shift, scale = (rand(segments, D) for _ in range(3))
    h, y, mean, rstd = lnmod.gated_forward(x, u, gate, shift, scale, cu, EPS)
    dx, du, dgate, dshift, dscale = lnmod.gated_backward(dy, dh, h, u, gate, scale, mean, rstd, cu, EPS)
    for m, r in enumerate(cuts):
        gt, sc, d = gate[m].double(), scale[m].double(), dy[r].double()
        _close("h", h[r], x[r].double() + gt * u[r].double(), 4e-3)
        n, rs = _norm(h[r].double())                 # everything after the residual is of the kept values
        _close("y", y[r], n * (1.0 + sc) + shift[m].double(), 4e-3)
        dxw = _ln_backward(d, sc, n, rs) + dh[r].double()
        _close("dx", dx[r], dxw, 4e-3)
        _close("du", du[r], gt * dxw, 4e-3)
        _close("dgate", dgate[m], (u[r].double() * dxw).sum(0), 1e-5)
        _close("dshift", dshift[m], d.sum(0), 1e-5)
        _close("dscale", dscale[m], (d * n).sum(0), 1e-5)


@pytest.mark.parametrize("D,mb,dtype", [
    (1152, 3, "bf16"), (1152, 14, "bf16"), (2560, 3, "bf16"), (2560, 10, "bf16"), (3072, 3, "bf16"), (3072, 10, "bf16"),
    (4096, 40, "bf16"), (3584, 1, "bf16"), (3584, 10, "bf16"), (1152, 40, "f32"), (2048, 3, "f32"), (2048, 10, "f32"),
    (2048, 30, "f32"), (2048, 40, "f32"), (2200, 6, "f32"), (2200, 8, "f32"), (2200, 20, "f32"), (3072, 3, "f32"),
    (3072, 20, "f32"), (6144, 30, "f32"), (6144, 40, "f32"), (3584, 9, "f32"), (3584, 30, "f32"), (3584, 160, "f32"),
    (1536, 3.5, "f32"), (1536, 12, "f32"), (1536, 40, "f32")])
def test_query_key_norm(D, mb, dtype):
    rows, rand = _make(D, mb, dtype, D * 5 + int(mb))
    tol = TYPES[dtype][1]
    print("size rule, query/key norm", D, mb, dtype, rows, flush=True)
    q, k, dq, dk = (rand(rows, D) for _ in range(4))
    wq, wk = rand(D), rand(D)
    qn, kn, rq, rk = lnmod.qknorm_forward(q, k, wq, wk, EPS)
    got = lnmod.qknorm_backward(dq, dk, q, k, wq, wk, rq, rk, EPS)
    for t, w, d, y, dx, dw in ((q, wq, dq, qn, got[0], got[2]), (k, wk, dk, kn, got[1], got[3])):
        v, w, d = t.double(), w.double(), d.double()
        rs = (v.square().mean(-1, keepdim=True) + EPS).rsqrt()
        h = v * rs
        g = d * w
        _close("y", y, h * w, tol)
        _close("dx", dx, (g - h * (g * h).mean(-1, keepdim=True)) * rs, tol)
        _close("dw", dw, (d * h).sum(0), 1e-5)
