"""The native calls of the autograd front end against its Python classes: same bits, same saved tensors, same
refusals.  The classes call the same entry points, so equality is exact."""
import numpy as np
import pytest


def _calls():
    import torch
    from paper_2309_16669_amd import autograd as ag
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    bf = torch.bfloat16
    rn = lambda *s, dt=bf: torch.randn(*s, generator=g, device="cuda").to(dt)
    f32 = lambda n: rn(n, dt=torch.float32)
    return {
        "attention": (ag.attention, ag._Attention, [rn(2, 70, 3, 64) for _ in range(3)], (0.125, False)),
        "attention_f16_causal": (ag.attention, ag._Attention, [rn(1, 200, 2, 80, dt=torch.float16) for _ in range(3)], (0.1, True)),
        "attention_strided": (ag.attention, ag._Attention, [rn(2, 3, 70, 64).transpose(1, 2) for _ in range(3)], (0.125, False)),
        "qkvpacked": (ag.attention_qkvpacked, ag._AttentionPacked, [rn(2, 70, 3, 2, 64)], (0.125, True)),
        "layer_norm": (ag.layer_norm, ag._LayerNorm, [rn(2, 5, 768), f32(768), f32(768)], (1e-6,)),
        "layer_norm_strided": (ag.layer_norm, ag._LayerNorm, [rn(40, 64).t(), f32(80)[::2], f32(40)], (1e-5,)),
        "bias_gelu": (ag.bias_gelu, ag._BiasGelu, [rn(3, 7, 1024), f32(1024)], ()),
        "bias_gelu_linear": (ag.bias_gelu_linear, ag._BiasGeluLinear, [rn(9, 256), f32(256), rn(64, 256), rn(64)], ()),
        "bias_gelu_linear_no_bias": (ag.bias_gelu_linear, ag._BiasGeluLinear, [rn(9, 256), f32(256), rn(64, 256)], ()),
    }


NAMES = ["attention", "attention_f16_causal", "attention_strided", "qkvpacked", "layer_norm", "layer_norm_strided", "bias_gelu",
         "bias_gelu_linear", "bias_gelu_linear_no_bias"]


def _pass(f, args, rest, grad=None, saved=None):
    import torch
    leaves = [a.detach().requires_grad_() for a in args]
    pack = lambda t: ((saved.append((tuple(t.shape), t.dtype)) if saved is not None else None), t)[1]
    with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t):
        y = f(*leaves, *rest)
    grad = torch.ones_like(y) if grad is None else grad(y)
    return [y.detach(), *torch.autograd.grad(y, leaves, grad)]


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_same_bits_and_saved_tensors_as_the_classes(name):
    import torch
    front, cls, args, rest = _calls()[name]
    apply = lambda *a: cls.apply(*(a if name != "bias_gelu_linear_no_bias" else (*a, None)))
    wide = lambda y: torch.linspace(-1, 1, y.shape[-1], device="cuda").to(y.dtype).expand(y.shape)   # a gradient that is a view
    for grad in (None, wide):
        s1, s2 = [], []
        a, b = _pass(front, args, rest, grad, s1), _pass(apply, args, rest, grad, s2)
        assert s1 == s2 and len(a) == len(b)
        for t, u in zip(a, b):
            assert t.shape == u.shape and t.dtype == u.dtype and torch.equal(t, u)
    with torch.no_grad():
        assert torch.equal(front(*args, *rest), a[0]) and not front(*args, *rest).requires_grad


@pytest.mark.gpu
def test_plain_calls_are_taken_and_others_are_declined():
    import torch
    from paper_2309_16669_amd import autograd as ag
    native = ag.native_calls()
    front, cls, args, rest = _calls()["layer_norm"]
    assert native.layer_norm(*args, 1e-5) is not None

    class Sub(torch.Tensor):
        pass
    x, gamma, beta = args
    declined = [(x.as_subclass(Sub), gamma, beta), (x.float(), gamma, beta), (x, gamma.double(), beta), (x, gamma[:-8], beta),
                (x.cpu(), gamma, beta), (x[:0], gamma, beta)]
    for bad in declined:
        assert native.layer_norm(*bad, 1e-5) is None
    q, k, v = _calls()["attention"][2]
    assert native.attention(q, k, v, 0.125, False) is not None
    for bad in ((q.float(), k, v), (q, k[:, :-1], v), (q, k.half(), v), (q[0], k[0], v[0])):
        assert native.attention(*bad, 0.125, False) is None
    # refused before, refused now: function transforms and forward-mode tangents
    for f in (lambda: torch.func.vmap(ag.layer_norm, in_dims=(0, None, None))(x, gamma, beta),
              lambda: torch.func.jvp(lambda t: ag.layer_norm(t, gamma, beta), (x,), (x,))):
        with pytest.raises(Exception):
            f()


@pytest.mark.gpu
def test_errors_of_the_library_keep_their_type_in_both_directions():
    import torch
    import paper_2309_16669_amd as av
    from paper_2309_16669_amd import autograd as ag
    bad = [torch.randn(1, 40, 2, 48, device="cuda").to(torch.bfloat16) for _ in range(3)]      # d = 48 is not built
    with pytest.raises(av.AvionError) as e:
        ag.attention(*bad)
    assert e.value.code == av.EUNSUPPORTED
    q, k, v = (t.requires_grad_() for t in _calls()["attention"][2])
    o = ag.attention(q, k, v)
    odd = torch.zeros(o.numel() + 1, dtype=o.dtype, device="cuda")[1:].view_as(o)              # contiguous, off by two bytes
    with pytest.raises(av.AvionError) as e:
        torch.autograd.grad(o, [q], odd)
    assert e.value.code == av.EUNSUPPORTED


@pytest.mark.gpu
def test_checkpointing_rebuilds_the_same_gradients():
    import torch
    from torch.utils.checkpoint import checkpoint
    for name in ("attention", "bias_gelu_linear"):
        front, cls, args, rest = _calls()[name]
        a = _pass(front, args, rest)
        b = _pass(lambda *t: checkpoint(front, *t, use_reentrant=False), args, rest)
        assert all(torch.equal(t, u) for t, u in zip(a, b))


def _other_strides(t):
    import torch
    wide = torch.empty((*t.shape, 2), dtype=t.dtype, device=t.device)
    wide[..., 0] = t
    return wide[..., 0]


def _other_format(t):
    import torch
    return t.to({torch.bfloat16: torch.float16, torch.float16: torch.bfloat16, torch.float32: torch.float16}[t.dtype])


UNPACKED = {"strides": _other_strides, "format": _other_format, "host": lambda t: t.cpu(), "shorter": lambda t: t[:-1]}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", UNPACKED)
@pytest.mark.parametrize("name", NAMES)
def test_saved_tensors_that_a_hook_changed_are_refused_as_by_the_classes(name, kind):
    # an unpack hook may return any tensor; where the classes go through (parameters in other strides, a torch
    # product's operand) so does the native call, with the same gradients
    import torch
    front, cls, args, rest = _calls()[name]
    apply = lambda *a: cls.apply(*(a if name != "bias_gelu_linear_no_bias" else (*a, None)))

    def outcome(f, which):
        leaves = [a.detach().requires_grad_() for a in args]
        count = iter(range(100))
        with torch.autograd.graph.saved_tensors_hooks(lambda t: (next(count), t.detach()),
                                                      lambda p: UNPACKED[kind](p[1]) if p[0] == which else p[1]):
            y = f(*leaves, *rest)
        saved = next(count)
        try:
            return saved, torch.autograd.grad(y, leaves, torch.ones_like(y))
        except (ValueError, RuntimeError) as e:
            return saved, type(e)

    saved, _ = outcome(front, -1)
    refused = 0
    for which in range(saved):
        (_, a), (_, b) = outcome(front, which), outcome(apply, which)
        assert isinstance(a, tuple) == isinstance(b, tuple), (which, a, b)
        if isinstance(a, tuple):
            assert all(torch.equal(t, u) for t, u in zip(a, b)), which
        else:
            refused += 1
    assert refused >= 1


@pytest.mark.gpu
@pytest.mark.parametrize("inside", [False, True])
@pytest.mark.parametrize("auto", ["float16", "bfloat16"])
@pytest.mark.parametrize("own", ["float16", "bfloat16"])
def test_products_under_autocast_behave_as_in_the_class(own, auto, inside):
    # autocast may give the second product (or its gradient) another 16-bit format than the activation's
    import torch
    from paper_2309_16669_amd import autograd as ag
    args = [a if a.dtype == torch.float32 else a.to(getattr(torch, own)) for a in _calls()["bias_gelu_linear"][2]]

    def outcome(f):
        leaves = [a.detach().requires_grad_() for a in args]
        with torch.autocast("cuda", dtype=getattr(torch, auto)):
            y = f(*leaves)
            try:
                if inside:
                    return [y, *torch.autograd.grad(y, leaves, torch.ones_like(y))]
            except (ValueError, RuntimeError) as e:
                return type(e)
        try:
            return [y, *torch.autograd.grad(y, leaves, torch.ones_like(y))]
        except (ValueError, RuntimeError) as e:
            return type(e)

    a, b = outcome(ag.bias_gelu_linear), outcome(ag._BiasGeluLinear.apply)
    assert isinstance(a, list) == isinstance(b, list), (a, b)
    if isinstance(a, list):
        assert all(t.dtype == u.dtype and torch.equal(t, u) for t, u in zip(a, b))
    else:
        assert a is b


ROUTES = {"native": lambda ag: ag.bias_gelu_linear, "class": lambda ag: ag._BiasGeluLinear.apply}


@pytest.mark.gpu
@pytest.mark.parametrize("route", ROUTES)
def test_the_activation_gradients_are_not_differentiated_as_the_products_they_overwrite(route):
    # dx is formed in the storage of the incoming gradient's product with the weight: neither that product's node
    # (create_graph) nor its tangent (forward mode over the backward) may come along
    import torch
    import torch.autograd.forward_ad as fwad
    from paper_2309_16669_amd import autograd as ag
    f = ROUTES[route](ag)
    x, bias, weight, out_bias = (a.detach().requires_grad_() for a in _calls()["bias_gelu_linear"][2])
    out = f(x, bias, weight, out_bias)
    dy = torch.randn_like(out).requires_grad_()
    plain = torch.autograd.grad(out, (x, bias), dy.detach(), retain_graph=True)
    recorded = torch.autograd.grad(out, (x, bias), dy, create_graph=True)
    for g, ref in zip(recorded, plain):
        assert torch.equal(g, ref) and not g.requires_grad
        with pytest.raises(RuntimeError, match="does not require grad"):
            g.float().square().sum().backward()
    with fwad.dual_level():
        dual = fwad.make_dual(dy.detach(), torch.randn_like(dy))
        for g, ref in zip(torch.autograd.grad(out, (x, bias), dual), plain):
            primal, tangent = fwad.unpack_dual(g)
            assert torch.equal(primal, ref) and tangent is None


@pytest.mark.gpu
@pytest.mark.parametrize("route", ROUTES)
def test_the_output_bias_gradient_can_be_differentiated(route):
    # the sum of the incoming gradient's rows, linear in it, with a node and a tangent of its own
    import torch
    import torch.autograd.forward_ad as fwad
    from paper_2309_16669_amd import autograd as ag
    f = ROUTES[route](ag)
    x, bias, weight, out_bias = (a.detach().requires_grad_() for a in _calls()["bias_gelu_linear"][2])
    out = f(x, bias, weight, out_bias)
    dy = torch.randn_like(out).requires_grad_()
    db, = torch.autograd.grad(out, out_bias, dy, create_graph=True)
    v = torch.randn_like(db)
    ddy, = torch.autograd.grad(db, dy, v, retain_graph=True)
    assert torch.equal(ddy, v.expand_as(dy))
    with fwad.dual_level():
        t = torch.randn_like(dy)
        db, = torch.autograd.grad(out, out_bias, fwad.make_dual(dy.detach(), t))
        assert torch.equal(fwad.unpack_dual(db).tangent, t.sum(0))


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["attention", "qkvpacked", "layer_norm", "bias_gelu", "bias_gelu_linear"])
def test_other_threads_run_during_a_call(name):
    # with a switch interval longer than the test another thread runs only when a call gives up the interpreter lock
    # (the outputs are kept: freeing a tensor gives it up too)
    import sys
    import threading
    import torch
    front, _, args, rest = _calls()[name]
    with torch.no_grad():
        front(*args, *rest)
        go, ran, kept, interval = threading.Event(), [], [], sys.getswitchinterval()
        other = threading.Thread(target=lambda: (go.wait(), ran.append(True)))
        other.start()
        try:
            sys.setswitchinterval(1000)
            go.set()
            for _ in range(10000):
                kept.append(front(*args, *rest))
                if ran:
                    break
            seen = bool(ran)
        finally:
            sys.setswitchinterval(interval)
            other.join()
    assert seen


PLAIN = ["attention_f16_causal", "qkvpacked", "layer_norm", "bias_gelu"]


def _one_pass(front, leaves, rest, dy):
    import torch
    y = front(*leaves, *rest)
    return [y.detach(), *torch.autograd.grad(y, leaves, dy)]


@pytest.mark.gpu
def test_threads_with_a_stream_each_do_not_disturb_each_other():
    # workspaces and outputs come from the allocator on each thread's stream, the backward runs on it too
    import threading
    import torch
    calls, jobs = _calls(), []
    for name in PLAIN:
        front, _, args, rest = calls[name]
        leaves = [a.detach().requires_grad_() for a in args]
        dy = torch.randn_like(front(*leaves, *rest))
        jobs.append((front, leaves, rest, dy, _one_pass(front, leaves, rest, dy)))
    torch.cuda.synchronize()
    got = [[] for _ in jobs]

    def work(i):
        front, leaves, rest, dy, _ = jobs[i]
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got[i].append(_one_pass(front, leaves, rest, dy))
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for (*_, ref), outs in zip(jobs, got):
        assert len(outs) == 20
        for out in outs:
            assert all(torch.equal(a, b) for a, b in zip(ref, out))


@pytest.mark.gpu
@pytest.mark.parametrize("name", PLAIN)
def test_forward_and_backward_can_be_captured_and_replayed(name):
    import torch
    front, _, args, rest = _calls()[name]
    leaves = [a.detach().clone().requires_grad_() for a in args]
    inputs = [[torch.randn_like(a) for a in args] for _ in range(3)]
    dy = torch.randn_like(front(*leaves, *rest))
    refs = [_one_pass(front, [t.clone().requires_grad_() for t in x], rest, dy) for x in inputs]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _one_pass(front, leaves, rest, dy)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = _one_pass(front, leaves, rest, dy)
    for i in (0, 1, 2, 1):
        with torch.no_grad():
            for leaf, t in zip(leaves, inputs[i]):
                leaf.copy_(t)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(refs[i], out)), i
        _one_pass(front, [t.clone().requires_grad_() for t in inputs[(i + 1) % 3]], rest, dy)    # eager work in between


def test_host_tensors_are_refused_as_before():
    import torch
    from paper_2309_16669_amd import autograd as ag
    q = torch.from_numpy(np.zeros((1, 40, 2, 64), np.float32)).to(torch.bfloat16)
    with pytest.raises(ValueError):
        ag.attention(q, q, q)
    with pytest.raises(ValueError):
        ag.layer_norm(q, torch.ones(64), torch.zeros(64))


def test_a_tree_without_the_native_module_serves_every_call(monkeypatch):
    # only the HIP library is needed; the classes answer (here: refuse host tensors), after a warning
    import sys
    import torch
    import paper_2309_16669_amd as av
    from paper_2309_16669_amd import autograd as ag
    monkeypatch.setattr(ag, "_native", None)
    monkeypatch.delattr(av, "_avion_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2309_16669_amd._avion_torch", None)
    q = torch.zeros(1, 40, 2, 64, dtype=torch.bfloat16)
    w, b = torch.ones(64), torch.ones(64, 64, dtype=torch.bfloat16)
    with pytest.warns(UserWarning, match="_avion_torch"):
        with pytest.raises(ValueError):
            ag.attention(q, q, q)
    for call in (lambda: ag.attention_qkvpacked(torch.stack([q] * 3, 2)), lambda: ag.layer_norm(q, w, w),
                 lambda: ag.bias_gelu(q, w), lambda: ag.bias_gelu_linear(q, w, b)):
        with pytest.raises(ValueError):
            call()


def test_a_missing_or_old_module_is_stale(monkeypatch, tmp_path):
    import os
    from paper_2309_16669_amd import build
    lib, module = tmp_path / "lib.so", tmp_path / "module.so"
    lib.touch()
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "TORCH_MODULE", str(module))
    assert build.is_stale()
    module.touch()
    assert not build.is_stale()
    os.utime(module, (0, 0))
    assert build.is_stale()
