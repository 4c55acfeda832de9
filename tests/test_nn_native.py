"""The layers' native functions against the Python ones: the same results and gradients bit for bit over the forms
an input comes in, the same refusals, and the calls they leave to Python."""
import threading

import pytest
import torch

from paper_2601_15473_amd import libsk as sk
from paper_2601_15473_amd import nn as sknn


def _layer(two_sided, dtype, bias=True):
    cls = sknn.SKLinearTwoSided if two_sided else sknn.SKLinear
    return cls(96, 80, 2, 16, bias=bias, dtype=dtype, seed=7)


def _python(layer, x):
    """The layer's forward pass through the Python functions."""
    if isinstance(layer, sknn.SKLinear):
        return sknn.SKLinearFunction.apply(x, layer.S_cat, layer.U_cat, layer.bias, layer.num_terms, layer.low_rank)
    return sknn.SKLinearTwoSidedFunction.apply(x, layer.S1_cat, layer.U1_cat, layer.U2_cat, layer.S2T_cat, layer.bias,
                                               layer.num_terms, layer.low_rank, layer._stage_matrices())


FORMS = {
    "rows": lambda x: x, "batched": lambda x: x.view(5, 26, 96), "one row": lambda x: x[3],
    "strided": lambda x: x.t().contiguous().t(), "columns": lambda x: torch.cat([x, x], 1)[:, 96:],
}


@pytest.mark.gpu
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("two_sided", [False, True])
def test_same_as_the_python_functions(two_sided, dtype, form):
    layer = _layer(two_sided, dtype, bias=form != "batched")
    base = torch.randn(130, 96, generator=torch.Generator().manual_seed(2)).to(dtype).cuda()
    got = []
    for run in (layer, lambda x: _python(layer, x)):
        x = base.clone().requires_grad_()
        y = run(FORMS[form](x))
        dY = torch.arange(y.numel(), device="cuda").remainder_(7).view(y.shape).to(dtype)
        layer.zero_grad(set_to_none=True)
        y.backward(dY)
        got.append((y.detach(), x.grad, *(p.grad for p in layer.parameters())))
        if len(got) == 1:
            assert "SKLinear" not in y.grad_fn.name(), y.grad_fn.name()   # (the Python functions' nodes bear their names)
    for a, b in zip(*got):
        assert a.shape == b.shape and a.dtype == b.dtype and torch.equal(a, b)


@pytest.mark.gpu
def test_only_the_wanted_gradients():
    layer = _layer(False, torch.bfloat16)
    x = torch.randn(40, 96, device="cuda").bfloat16()
    layer(x).float().square().sum().backward()
    want = [p.grad.clone() for p in layer.parameters()]
    layer.zero_grad(set_to_none=True)
    layer.U_cat.requires_grad_(False)
    layer(x).float().square().sum().backward()
    assert layer.U_cat.grad is None and torch.equal(layer.bias.grad, want[1])
    x.requires_grad_()
    y = layer(x)
    dx, = torch.autograd.grad(y.float().sum(), x)
    assert dx.shape == x.shape and x.grad is None
    with torch.no_grad():
        assert not layer(x).requires_grad


@pytest.mark.gpu
def test_hooks_transforms_and_tangents():
    layer = _layer(False, torch.float32)
    x = torch.randn(24, 96, device="cuda", requires_grad=True)
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t) or t.cpu(), lambda t: t.cuda()):
        y = layer(x)
    y.sum().backward()
    assert len(packed) == 3 and x.grad is not None
    z = layer(x.detach()).clone()
    # (as with the Python functions: neither has a vmap rule, a forward-mode or a second derivative)
    with pytest.raises(RuntimeError):
        torch.func.vmap(layer)(x.detach().view(2, 12, 96))
    with torch.autograd.forward_ad.dual_level(), pytest.raises(Exception):
        layer(torch.autograd.forward_ad.make_dual(x.detach(), torch.ones_like(x)))
    assert torch.equal(layer(x.detach()), z)
    y = layer(x)
    with torch.no_grad():
        layer.U_cat.add_(1.0)   # saved for the backward pass
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        y.sum().backward()

    class Tagged(torch.Tensor):
        pass

    assert sknn._native.linear(x.detach().as_subclass(Tagged), layer.S_cat, layer.U_cat, layer.bias, 2, 16) is None
    assert layer(x.detach().as_subclass(Tagged)).shape == (24, 80)


class Seen:
    """The native functions, with what each call got from them: taken or left to Python."""

    def __init__(self, native):
        self.native, self.taken = native, []

    def __getattr__(self, name):
        f = getattr(self.native, name)

        def call(*args):
            y = f(*args)
            self.taken.append(y is not None)
            return y
        return call if name.startswith("linear") else f


def _step(layer, x, around=None):
    x = x.clone().requires_grad_()
    layer.zero_grad(set_to_none=True)
    y = layer(x) if around is None else around(layer, x)
    y.backward(torch.ones_like(y))
    return [y.detach(), x.grad, *(p.grad for p in layer.parameters())]


def _dispatch_mode(layer, x):
    from torch.utils._python_dispatch import TorchDispatchMode

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            ops.append(func)
            return func(*args, **(kwargs or {}))
    ops = []
    with Mode():
        y = layer(x)
    assert ops   # (what the layer allocates, at least)
    return y


def _function_mode(layer, x):
    from torch.overrides import TorchFunctionMode

    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        return layer(x)


def _compiled(layer, x):
    torch._dynamo.reset()
    return torch.compile(layer, backend="eager")(x)


def _functional(layer, x):
    return torch.func.functional_call(layer, dict(layer.named_parameters()), (x,))


@pytest.mark.gpu
@pytest.mark.parametrize("around,taken", [(_dispatch_mode, False), (_function_mode, False), (_compiled, None), (_functional, True)],
                         ids=lambda f: getattr(f, "__name__", ""))
@pytest.mark.parametrize("two_sided", [False, True])
def test_modes_and_compilation(monkeypatch, two_sided, around, taken):
    """The same step inside torch's modes, compiled and as a functional call; the native functions leave the modes to Python."""
    layer = _layer(two_sided, torch.bfloat16)
    x = torch.randn(40, 96, generator=torch.Generator().manual_seed(3)).bfloat16().cuda()
    want = _step(layer, x)
    seen = Seen(sknn._native)
    monkeypatch.setattr(sknn, "_native", seen)
    got = _step(layer, x, around)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    assert taken is None or seen.taken == [taken], seen.taken


@pytest.mark.gpu
def test_functional_call_with_other_weights():
    layer, other = _layer(False, torch.bfloat16), _layer(False, torch.bfloat16)
    with torch.no_grad():
        other.U_cat.mul_(2.0)
    x = torch.randn(40, 96, device="cuda").bfloat16()
    with torch.no_grad():
        assert torch.equal(torch.func.functional_call(layer, dict(other.named_parameters()), (x,)), other(x))
        assert not torch.equal(layer(x), other(x))


@pytest.mark.gpu
def test_tracing(monkeypatch):
    """torch.jit.trace records a Python function's call, which the trace then makes on other inputs."""
    layer = _layer(False, torch.bfloat16)
    x = torch.randn(40, 96, device="cuda").bfloat16()
    other = torch.randn(40, 96, device="cuda").bfloat16()
    seen = Seen(sknn._native)
    monkeypatch.setattr(sknn, "_native", seen)
    with torch.no_grad():
        traced = torch.jit.trace(layer, x, check_trace=False)
        assert seen.taken == [False], seen.taken
        assert torch.equal(traced(x), layer(x)) and torch.equal(traced(other), layer(other))


@pytest.mark.gpu
def test_refusals():
    layer = _layer(False, torch.bfloat16)
    with pytest.raises(TypeError, match="dtype"):
        layer(torch.zeros(4, 96, device="cuda"))
    with pytest.raises(RuntimeError, match="GPU only"):
        layer(torch.zeros(4, 96).bfloat16())
    with pytest.raises(ValueError, match="shapes"):
        layer(torch.zeros(4, 95, device="cuda").bfloat16())
    with pytest.raises(RuntimeError):
        layer(torch.zeros(0, 96, device="cuda").bfloat16())
    odd = torch.zeros(4 * 96 + 1, device="cuda").bfloat16()[1:].view(4, 96)
    with pytest.raises(RuntimeError, match="misaligned"):
        layer(odd)


@pytest.mark.gpu
@pytest.mark.parametrize("wanted", ["all", "x", "factor"])
@pytest.mark.parametrize("two_sided", [False, True])
def test_refused_gradients(two_sided, wanted):
    """A gradient that is not 16-byte aligned: libsk's own error and status from the backward pass, as from the Python functions'."""
    layer = _layer(two_sided, torch.bfloat16)
    for p in layer.parameters():
        p.requires_grad_(wanted != "x")
    odd = torch.zeros(4 * 80 + 1, device="cuda").bfloat16()[1:].view(4, 80)
    for run in (layer, lambda x: _python(layer, x)):
        x = torch.zeros(4, 96, device="cuda").bfloat16().requires_grad_(wanted != "factor")
        y = run(x)
        with pytest.raises(sk.SkError, match="misaligned") as e:
            y.backward(odd)
        assert e.value.status == sk.SK_ERR_INVALID_ARG
    x = torch.ones(4, 96, device="cuda").bfloat16().requires_grad_()
    layer(x).sum().backward()     # (and the next pass is none the worse)
    assert x.grad is not None and torch.isfinite(x.grad).all()


@pytest.mark.gpu
def test_threads_and_streams():
    """Each thread on a stream of its own, and all on one: results as alone."""
    layer = _layer(False, torch.bfloat16)
    xs = [torch.randn(300 + 64 * i, 96, device="cuda").bfloat16() for i in range(4)]
    want = [layer(x).detach() for x in xs]
    torch.cuda.synchronize()
    shared = torch.cuda.Stream()
    for streams in ([torch.cuda.Stream() for _ in xs], [shared] * len(xs)):
        got = [None] * len(xs)

        def work(i):
            with torch.cuda.stream(streams[i]):
                for _ in range(20):
                    y = layer(xs[i].detach().requires_grad_())
                    y.backward(torch.ones_like(y))
                got[i] = y.detach()
        threads = [threading.Thread(target=work, args=(i,)) for i in range(len(xs))]
        [t.start() for t in threads]
        [t.join() for t in threads]
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    sknn.release_workspaces()
    assert torch.equal(layer(xs[0]), want[0])


@pytest.mark.gpu
@pytest.mark.parametrize("two_sided,d_in,d_out,k,beside", [
    # (fp32 sums of up to 4 MiB stay behind the workspace of a two-sided layer: 128 x (2 x 768 + 256) + 768 numbers, and 128 x (2 x 4096 + 1024) + 4096)
    (False, 256, 768, 64, 0), (True, 256, 768, 64, 920_576 + 256), (True, 1024, 4096, 64, 0),
])
def test_what_a_pass_keeps(two_sided, d_in, d_out, k, beside):
    layer = (sknn.SKLinearTwoSided if two_sided else sknn.SKLinear)(d_in, d_out, 2, k, dtype=torch.bfloat16, seed=7)
    x, dY = torch.randn(500, d_in, device="cuda").bfloat16().requires_grad_(), torch.randn(500, d_out, device="cuda").bfloat16()
    sknn.release_workspaces()     # (other tests' streams)
    op, l = (sk.SK_OP_BWD_TWO_SIDED, 4) if two_sided else (sk.SK_OP_BWD, 2)
    most = max(sk.sk_linear_workspace_bytes(o, 500, d_in, d_out, l, k, sk.SK_BF16) for o in (sk.SK_OP_FWD, op)) + beside
    for _ in range(2):
        torch.autograd.grad(layer(x), (x, *layer.parameters()), dY)
    torch.cuda.synchronize()
    held = torch.cuda.memory_allocated()
    sknn.release_workspaces()
    held -= torch.cuda.memory_allocated()
    assert 0 < held <= most + 512, (held, most)   # (the allocator's rounding)


def test_calls_left_to_python_are_not_taken():
    t = torch.zeros(4, 32)
    assert sknn._native.linear(t, t, t, None, 1, 16) is None                  # not on a GPU
    assert sknn._native.linear(t, None, t, None, 1, 16) is None
    assert sknn._native.linear(t, t, t, None, 1.0, 16) is None
    assert sknn._native.linear_two_sided(t, t, t, t, t, None, t, t, 1, 16) is None
    sknn.release_workspaces()


@pytest.mark.gpu
@pytest.mark.parametrize("counts", [(16,), (1, 1023), (4096, 3, 1040)])
def test_round_gradients(counts):
    src = [torch.randn(n, device="cuda") for n in counts]
    src[0][0] = float("inf")
    dst = [torch.full((n + 8,), 7.0, device="cuda").bfloat16() for n in counts]
    sk.check(sk.sk_round_gradients(src, dst, counts))
    torch.cuda.synchronize()
    for s, d, n in zip(src, dst, counts):
        assert torch.equal(d[:n], s.bfloat16()) and torch.equal(d[n:], torch.full((8,), 7.0, device="cuda").bfloat16())
    assert sk.sk_round_gradients([], [], []) == sk.SK_ERR_INVALID_ARG
    assert sk.sk_round_gradients(src[:1], [dst[0].data_ptr() + 4], (1,)) == sk.SK_ERR_INVALID_ARG
