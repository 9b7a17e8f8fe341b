"""The launch shapes of the size classes at widths that are whole multiples of 256 features (the tests of the long launches
run one chunk below them): forward, backward and the backward that forms the statistics again, against plain torch float64,
three equal samples and five ragged segments, one of them a single row.

Tolerances: bf16 results are rounded once (2^-9 relative, 1.7e-3 in the 2-norm; 4e-3 allowed); the float32 sums over up to
26 000 rows are off by the order of their additions (1e-5 of the 2-norm)."""
import pytest
import torch

from paper_2605_17923_amd import lnmod

pytestmark = pytest.mark.gpu

EPS = 1e-6


def _close(name, got, want, tol):
    err = float((got.double() - want).norm() / want.norm())
    assert err <= tol, "%s: relative error %.2e" % (name, err)


@pytest.mark.parametrize("mb", [14, 40, 100, 160])
@pytest.mark.parametrize("D", [1536, 2048, 2560, 3072, 3584, 4096, 5120, 6144])
def test_every_class_against_float64(D, mb):
    g = torch.Generator(device="cuda")
    g.manual_seed(D + mb)

    def rand(*s):
        return torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)

    rows = int(mb * 1e6 / 2 / D)
    S = rows // 3 + 1
    cut = [0, rows // 7, rows // 7 + 1, rows // 2 + 3, rows - 5, rows]
    for lens in ([S] * 3, [b - a for a, b in zip(cut, cut[1:])]):
        n, T = len(lens), sum(lens)
        print("size class", D, mb, lens, flush=True)
        x, dy, shift, scale = rand(T, D), rand(T, D), rand(n, D), rand(n, D)
        cu = torch.tensor([sum(lens[:i]) for i in range(n + 1)], dtype=torch.int32, device="cuda")
        if n == 3:
            y, mean, rstd = lnmod.forward(x.view(n, S, D), shift, scale, EPS)
            got = lnmod.backward(dy.view(n, S, D), x.view(n, S, D), scale, mean, rstd, EPS)
            again = lnmod.backward(dy.view(n, S, D), x.view(n, S, D), scale, None, None, EPS)
        else:
            y, mean, rstd = lnmod.forward_varlen(x, shift, scale, cu, EPS)
            got = lnmod.backward_varlen(dy, x, scale, cu, mean, rstd, EPS)
            again = lnmod.backward_varlen(dy, x, scale, cu, None, None, EPS)
        at = 0
        for m, rows_m in enumerate(lens):
            r = slice(at, at + rows_m)
            at += rows_m
            v, d, a = x[r].double(), dy[r].double(), 1.0 + scale[m].double()
            c = v - v.mean(-1, keepdim=True)
            rs = (c.square().mean(-1, keepdim=True) + EPS).rsqrt()
            h, gr = c * rs, d * a
            _close("y", y.reshape(T, D)[r], h * a + shift[m].double(), 4e-3)
            dx = (gr - gr.mean(-1, keepdim=True) - h * (gr * h).mean(-1, keepdim=True)) * rs
            for dxg, dsh, dsc in (got, again):
                _close("dx", dxg.reshape(T, D)[r], dx, 4e-3)
                _close("dshift", dsh[m], d.sum(0), 1e-5)
                _close("dscale", dsc[m], (d * h).sum(0), 1e-5)
