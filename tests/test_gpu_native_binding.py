"""The native calls (fwd, bwd and the layer's C++ autograd node) against the
general Python path: the same results bit for bit, the same objects returned,
the same errors, in the forms where an autograd node can go wrong: strided
inputs and gradients, saved-tensor hooks, several and repeated backwards,
functorch transforms, forward-mode AD, checkpointing, other streams."""
import pytest
import torch

import paper_2202_00441_amd as P
from paper_2202_00441_amd import _lib

pytestmark = pytest.mark.gpu

LAYER = P.FewBitAct("gelu", 3)


def _general(x):
    return P.FewBitActivation.apply(x, LAYER.table)


def _x(*shape, dtype=torch.bfloat16, seed=1):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*shape, generator=gen, device="cuda").to(dtype)


def _same(a, b):
    assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride()
    assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("form", ["plain", "scalar", "empty", "transposed", "sliced", "parameter", "nonleaf"])
def test_layer_equals_the_general_path(dtype, form):
    def make():
        x = _x(33, 70, dtype=dtype)
        if form == "scalar":
            x = _x(1, dtype=dtype).reshape(())
        elif form == "empty":
            x = _x(0, 7, dtype=dtype)
        elif form == "parameter":
            return torch.nn.Parameter(x)
        return x.requires_grad_()

    outs = []
    for f in (LAYER, _general):
        leaf = make()
        x = {"transposed": leaf.t() if leaf.dim() == 2 else leaf, "sliced": leaf[:, ::2] if leaf.dim() == 2 else leaf,
             "nonleaf": leaf * 2}.get(form, leaf)
        y = f(x)
        assert y.requires_grad and not y.is_leaf and type(y) is torch.Tensor
        (g,) = torch.autograd.grad(y.sum(), leaf)          # an expanded, stride-0 gradient
        outs.append((y.detach(), g))
    _same(outs[0][0], outs[1][0])
    _same(outs[0][1], outs[1][1])


def test_without_grad():
    x = _x(1000)
    y = LAYER(x)
    assert not y.requires_grad and y.grad_fn is None
    with torch.no_grad():
        z = LAYER(x.clone().requires_grad_())
    assert not z.requires_grad
    with torch.inference_mode():
        w = LAYER(x)
    assert w.is_inference() and torch.equal(w, y)


def test_calls_return_the_buffers_passed_in():
    x = _x(1001)
    y, codes = P.fwd(LAYER.table, x)
    y2, c2 = torch.empty_like(x), torch.empty(P.packed_words(1001, 3) + 5, dtype=torch.int32, device="cuda")
    a, b = P.fwd(LAYER.table, x, y2, c2)
    assert a is y2 and b is c2 and torch.equal(a, y) and torch.equal(b[:codes.numel()], codes)
    gin = torch.empty_like(x)
    assert P.bwd(LAYER.table, x, c2, gin) is gin
    _same(gin, P.bwd(LAYER.table, x, codes))
    u = codes.view(torch.uint32)                            # other 4-byte words: the general path
    _same(gin, P.bwd(LAYER.table, x, u))


@pytest.mark.parametrize("bad", ["short", "dtype", "strided", "host", "misaligned"])
def test_errors_are_those_of_the_general_path(bad):
    x = _x(1000)
    y, codes = P.fwd(LAYER.table, x)
    if bad == "misaligned":
        with pytest.raises(P.FewbitError, match="fewbit_fwd"):
            P.fwd(LAYER.table, x[1:])
        with pytest.raises(P.FewbitError, match="fewbit_bwd"):
            P.bwd(LAYER.table, x[1:], codes)
        leaf = _x(999).requires_grad_()
        for f in (LAYER, _general):
            with pytest.raises(P.FewbitError, match="fewbit_bwd"):
                f(leaf).backward(x[1:])
        with pytest.raises(P.FewbitError, match="fewbit_fwd"):
            LAYER(x[1:])
        return
    wrong = {"short": y[:-8], "dtype": y.float(), "strided": torch.empty(2000, dtype=y.dtype, device="cuda")[::2],
             "host": y.cpu()}[bad]
    with pytest.raises(ValueError):
        P.fwd(LAYER.table, x, wrong, codes)
    with pytest.raises(ValueError):
        P.bwd(LAYER.table, x, codes, wrong)
    with pytest.raises(ValueError):
        P.bwd(LAYER.table, x, codes[:5])
    with pytest.raises((ValueError, TypeError)):
        P.fwd(LAYER.table, x.double() if bad == "dtype" else x.cpu())


def test_saved_tensor_hooks():
    x = _x(4096 + 3).requires_grad_()
    for f in (LAYER, _general):
        seen = []

        def pack(t):
            seen.append((t.dtype, t.numel()))
            return t.cpu()

        with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t.cuda()):
            y = f(x)
        assert seen == [(torch.int32, P.packed_words(x.numel(), 3))]
        (g,) = torch.autograd.grad(y, x, torch.ones_like(y))
        _same(g, torch.autograd.grad(_general(x), x, torch.ones_like(y))[0])
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t):        # left on the host
            y = f(x)
        with pytest.raises(ValueError):
            torch.autograd.grad(y, x, torch.ones_like(y))


def test_repeated_and_released_graphs():
    x = _x(2000).requires_grad_()
    y = LAYER(x)
    one = torch.ones_like(y)
    a = torch.autograd.grad(y, x, one, retain_graph=True)[0]
    b = torch.autograd.grad(y, x, one)[0]
    _same(a, b)
    with pytest.raises(RuntimeError, match="second time"):
        torch.autograd.grad(y, x, one)
    g = torch.autograd.grad(LAYER(x), x, one, create_graph=True)[0]
    h = torch.autograd.grad(_general(x), x, one, create_graph=True)[0]
    assert g.requires_grad == h.requires_grad and torch.equal(g, h)


def test_transforms_are_refused_as_before():
    x = _x(4, 64, dtype=torch.float32)
    for f in (LAYER, _general):
        with pytest.raises(RuntimeError):
            torch.func.vmap(f)(x)
        with pytest.raises(RuntimeError):
            torch.func.grad(lambda t: f(t).sum())(x)
        with pytest.raises(RuntimeError):
            with torch.autograd.forward_ad.dual_level():
                f(torch.autograd.forward_ad.make_dual(x, torch.ones_like(x)))


@pytest.mark.parametrize("reentrant", [False, True])
def test_checkpoint(reentrant):
    from torch.utils.checkpoint import checkpoint
    x = _x(3000).requires_grad_()
    (a,) = torch.autograd.grad(LAYER(x).sum(), x)
    x2 = x.detach().clone().requires_grad_()
    checkpoint(LAYER, x2, use_reentrant=reentrant).sum().backward()
    _same(a, x2.grad)


def test_backward_runs_on_the_forwards_stream():
    # the forward waits on its stream behind a delay, in memory that held other
    # bytes before: a backward on any other stream would read those
    side = torch.cuda.Stream()
    x = _x(1 << 20).requires_grad_()
    ones = torch.ones_like(x)
    (ref,) = torch.autograd.grad(_general(x), x, ones)
    side.wait_stream(torch.cuda.current_stream())
    for delay in (0, 20_000_000):                  # the first pass loads and allocates
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            stale = [torch.full((P.packed_words(x.numel(), 3),), 0x2D2D2D2D, dtype=torch.int32, device="cuda")
                     for _ in range(2)]
            stale += [torch.full_like(x, -3.0) for _ in range(3)]
            where = {t.data_ptr() for t in stale}
            del stale
            torch.cuda._sleep(delay)
            y = LAYER(x)
            g = torch.ones_like(y)
        (codes,) = y.grad_fn.saved_tensors
        assert codes.data_ptr() in where and g.data_ptr() in where
        (got,) = torch.autograd.grad(y, x, g)
        busy = not side.query()
        torch.cuda.synchronize()
        _same(got, ref)
        del y, g, codes, got
    assert busy, "the delay was over before the backward was launched"


def test_dispatch_and_function_modes_see_the_general_path():
    from torch.utils._python_dispatch import TorchDispatchMode

    class Count(TorchDispatchMode):
        ops = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Count.ops += 1
            return func(*args, **(kwargs or {}))

    x = _x(1000)
    y, codes = P.fwd(LAYER.table, x)
    with Count():
        y2, c2 = P.fwd(LAYER.table, x)
    assert Count.ops > 0 and torch.equal(y, y2) and torch.equal(codes, c2)
    assert _lib._native.fwd(LAYER.table.c, x.cpu(), None, None) is None


def test_compiled_autograd():
    # two layers with tables of their own, saved-tensor hooks, and a second
    # backward that reuses the compiled graph
    from torch._dynamo import compiled_autograd
    other = P.FewBitAct("silu", 2)
    fs = [(LAYER, other), (_general, lambda t: P.FewBitActivation.apply(t, other.table))]
    for seed in (1, 2):
        grads = []
        for f, g in fs:
            for compiled in (False, True):
                x = _x(3001, seed=seed).requires_grad_()
                with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
                    y = g(f(x) * 2).sum() + f(x).float().square().sum()
                if compiled:
                    with compiled_autograd._enable(torch.compile(backend="eager")):
                        y.backward()
                else:
                    y.backward()
                grads.append(x.grad)
        for g in grads[1:]:
            _same(g, grads[0])


def test_grad_fn_shows_the_saved_codes():
    x = _x(1000).requires_grad_()
    codes = P.fwd(LAYER.table, x.detach())[1]
    for f in (LAYER, _general):
        y = f(x)
        assert y.grad_fn.name().startswith("FewBitActivation") and len(y.grad_fn.next_functions) == 1
        (saved,) = y.grad_fn.saved_tensors
        assert torch.equal(saved, codes)
        seen = []
        y.grad_fn.register_hook(lambda gi, go: seen.append((gi[0].shape, go[0].shape)))
        y.sum().backward()
        assert seen == [(x.shape, x.shape)]
        with pytest.raises(RuntimeError, match="second time"):
            y.grad_fn.saved_tensors


def test_the_profiler_sees_the_layer():
    x = _x(1000).requires_grad_()
    for f in (LAYER, _general):
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU], record_shapes=True) as p:
            f(x).sum().backward()
        shapes = {e.name: e.input_shapes for e in p.events()}
        assert shapes["FewBitActivation"][0] == [1000] and "FewBitActivationBackward" in shapes
        seq = {e.name: e.sequence_nr for e in p.events()}
        assert seq["FewBitActivation"] == seq["FewBitActivationBackward"] >= 0
