"""The C++ host path of the autograd functions and of the plain forward against the Python path it stands in
for: the same outputs and gradients bit for bit, the same errors, and everything that is not the plain case
(hooks apart, which both paths serve) handed back to the Python path."""
import pytest
import torch

from paper_2605_17923_amd import functional as F
from paper_2605_17923_amd import lnmod

pytestmark = pytest.mark.gpu


def _leaves(dtype, *shapes):
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    return [torch.randn(*s, generator=g, device="cuda").to(dtype).requires_grad_() for s in shapes]


def _case(op, dtype):
    """(the native call, the Python class's call, leaves)"""
    if op in ("sample", "token", "recompute"):
        mod = (2, 37, 264) if op == "token" else (2, 264)
        ts = _leaves(dtype, (2, 37, 264), mod, mod)
        a = (None, 1e-6, op != "recompute")
        return lambda x, sh, sc: F.ln_modulate(x, sh, sc, 1e-6, None, a[2]), lambda *t: F._LnModulate.apply(*t, *a), ts
    cu = torch.tensor([0, 0, 30, 31, 74], dtype=torch.int32, device="cuda")
    if op == "packed":
        ts = _leaves(dtype, (74, 264), (4, 264), (4, 264))
        return lambda x, sh, sc: F.ln_modulate(x, sh, sc, cu_seqlens=cu), lambda *t: F._LnModulate.apply(*t, cu, 1e-6, True), ts
    if op in ("gated", "gated packed"):
        c, rows, n = (cu, (74, 264), 4) if op == "gated packed" else (None, (2, 37, 264), 2)
        ts = _leaves(dtype, rows, rows, (n, 264), (n, 264), (n, 264))
        return lambda *t: F.gated_ln_modulate(*t, cu_seqlens=c), lambda *t: F._GatedLnModulate.apply(*t, c, 1e-6), ts
    ts = _leaves(dtype, (3, 5, 264), (3, 5, 264), (264,), (264,))
    return lambda *t: F.qk_norm(*t), lambda *t: F._QkNorm.apply(*t, 1e-6), ts


def _results(call, ts, out_grads=True):
    outs = call(*ts)
    outs = outs if isinstance(outs, tuple) else (outs,)
    loss = sum((o.float() * (i + 1.5)).sum() for i, o in enumerate(outs[:None if out_grads else 1]))
    return [o.detach() for o in outs] + list(torch.autograd.grad(loss, ts, allow_unused=True)), outs


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("op", ["sample", "token", "recompute", "packed", "gated", "gated packed", "qk"])
def test_same_results_as_the_python_path(op, dtype):
    native, python, ts = _case(op, dtype)
    for both in (True, False):                        # False: one of two outputs has no gradient
        a, outs = _results(native, ts, both)
        b, ref = _results(python, ts, both)
        assert type(outs[0].grad_fn) is not type(ref[0].grad_fn)
        assert len(a) == len(b)
        for u, v in zip(a, b):
            assert (u is None) == (v is None)
            assert u is None or (u.dtype == v.dtype and u.shape == v.shape and torch.equal(u, v))
    with torch.autograd.graph.save_on_cpu():          # saved tensors go through the hooks
        c, _ = _results(native, ts)
    for u, v in zip(c, _results(python, ts)[0]):
        assert torch.equal(u, v)
    with torch.no_grad():
        out = native(*ts)
        assert not (out[0] if isinstance(out, tuple) else out).requires_grad


@pytest.mark.parametrize("op", ["sample", "token", "recompute", "packed", "gated", "gated packed", "qk"])
def test_nodes_show_the_saved_tensors(op):
    """y.grad_fn.saved_tensors: what the Python path's node shows, also through hooks; gone after the backward."""
    native, python, ts = _case(op, torch.bfloat16)

    def node(call):
        out = call(*ts)
        return (out[0] if isinstance(out, tuple) else out).grad_fn, out

    (a, out), (b, ref) = node(native), node(python)
    assert type(a) is not type(b) and len(a.next_functions) == len(b.next_functions) and a.name()
    assert len(a.saved_tensors) == len(b.saved_tensors) >= 5
    for u, v in zip(a.saved_tensors, b.saved_tensors):
        assert (u is None) == (v is None)
        assert u is None or (u.shape == v.shape and torch.equal(u, v))
    with torch.autograd.graph.save_on_cpu():
        held, kept = node(native)
    for u, v in zip(held.saved_tensors, b.saved_tensors):
        assert u is None or torch.equal(u, v)
    del ref, kept                                      # (a node without its output has nothing saved any more)
    seen = []
    a.register_hook(lambda *g: seen.append(len(g)))
    sum(o.float().sum() for o in (out if isinstance(out, tuple) else (out,))).backward()
    assert seen == [2]
    with pytest.raises(RuntimeError):
        a.saved_tensors


def test_plain_forward_matches_the_python_path():
    x, sh, sc = (t.detach() for t in _leaves(torch.bfloat16, (2, 37, 264), (2, 264), (2, 264)))
    for u, v in zip(lnmod.forward(x, sh, sc), lnmod.forward(x, sh, sc, stream=torch.cuda.current_stream())):
        assert u.shape == v.shape and u.dtype == v.dtype and torch.equal(u, v)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        got = lnmod.forward(x, sh, sc)
    s.synchronize()
    assert torch.equal(got[0], lnmod.forward(x, sh, sc)[0])


def test_errors_are_those_of_the_python_path():
    x, sh, sc = _leaves(torch.bfloat16, (2, 8, 64), (2, 64), (2, 64))
    for bad in ((x, sh[:1], sc), (x, sh, sc.float()), (x.transpose(0, 1), sh, sc), (x, sh, None), (x.cpu(), sh, sc)):
        with pytest.raises((ValueError, AttributeError)):
            F.ln_modulate(*bad)
    wide = _leaves(torch.bfloat16, (1, 2, 12), (1, 12), (1, 12))      # not a multiple of 16 bytes
    with pytest.raises(lnmod.LnmodError) as e:
        F.ln_modulate(*wide)
    assert e.value.status == lnmod.LNMOD_EUNSUPPORTED
    y = F.ln_modulate(x, sh, sc)
    flat = torch.zeros(2 * 8 * 64 + 1, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(lnmod.LnmodError) as e:        # a gradient that is dense but not 16-byte aligned
        torch.autograd.grad(y, (x,), flat[1:].view(2, 8, 64))
    assert e.value.status == lnmod.LNMOD_EALIGN


def test_transforms_are_refused_as_before():
    x, sh, sc = (t.detach() for t in _leaves(torch.float32, (3, 2, 8, 64), (3, 2, 64), (3, 2, 64)))
    with pytest.raises(RuntimeError):
        torch.func.vmap(F.ln_modulate)(x, sh, sc)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: F.ln_modulate(t, sh[0], sc[0]).sum())(x[0])
    with torch.autograd.forward_ad.dual_level(), pytest.raises(RuntimeError):
        F.ln_modulate(torch.autograd.forward_ad.make_dual(x[0], x[0]), sh[0], sc[0])


@pytest.mark.parametrize("stats", [True, False])
def test_per_token_shift_gradient_is_a_tensor_of_its_own(stats):
    """dshift equals dy; a leaf's .grad must not share memory with a gradient that others still hold."""
    x, sh, sc = _leaves(torch.bfloat16, (2, 37, 264), (2, 37, 264), (2, 37, 264))
    y = F.ln_modulate(x, sh, sc, save_stats=stats)
    y.retain_grad()
    other = torch.zeros_like(y).requires_grad_()
    dy = torch.randn_like(y)
    keep = dy.clone()
    (y + other).backward(dy)
    assert torch.equal(sh.grad, keep)
    sh.grad.mul_(2)
    for t in (dy, y.grad, other.grad):
        assert torch.equal(t, keep)
    # a recorded backward keeps its copy: no half-connected second derivative
    y = F.ln_modulate(x, sh, sc, save_stats=stats)
    g = torch.randn_like(y).requires_grad_()
    for t in torch.autograd.grad(y, (x, sh, sc), g, create_graph=True):
        assert not t.requires_grad
    # an expanded gradient
    (got,) = torch.autograd.grad(F.ln_modulate(x, sh, sc, save_stats=stats).sum(), (sh,))
    assert torch.equal(got, torch.ones_like(sh)) and got.is_contiguous()


@pytest.mark.parametrize("stats", [True, False])
def test_per_token_shift_gradient_shares_no_memory_behind_a_view(stats):
    """A view of y gives the operator a fresh dy over memory that is the caller's."""
    def leaves():
        return _leaves(torch.bfloat16, (2, 37, 264), (2, 37, 264), (2, 37, 264))

    dz = torch.randn(74, 264, device="cuda", dtype=torch.bfloat16)
    keep = dz.clone()
    for look in (lambda y: y.view(-1, 264), lambda y: y.flatten(0, 1), lambda y: y.reshape(74, 264)):
        x, sh, sc = leaves()
        look(F.ln_modulate(x, sh, sc, save_stats=stats)).backward(dz)
        assert sh.grad.untyped_storage().data_ptr() != dz.untyped_storage().data_ptr()
        look(F.ln_modulate(x, sh, sc, save_stats=stats)).backward(dz)         # accumulates into sh.grad
        assert torch.equal(dz, keep) and torch.equal(sh.grad, keep.view_as(sh) * 2)
    # two operators that receive views of one gradient: each leaf has a .grad of its own
    (x1, s1, c1), (x2, s2, c2) = leaves(), leaves()
    both = F.ln_modulate(x1, s1, c1, save_stats=stats).view(-1, 264) + F.ln_modulate(x2, s2, c2, save_stats=stats).view(-1, 264)
    both.backward(dz)
    for t in (s1, s2):
        t.grad.mul_(0.5)
    for t in (s1, s2):
        assert torch.equal(t.grad, keep.view_as(t) * 0.5)
    # the caller's own dy, refilled after the call
    x, sh, sc = leaves()
    dy = dz.view(2, 37, 264)
    got = torch.autograd.grad(F.ln_modulate(x, sh, sc, save_stats=stats), (x, sh, sc), dy)
    dy.zero_()
    assert torch.equal(got[1], keep.view_as(sh))
    got[1].fill_(7)
    assert not dy.any()
