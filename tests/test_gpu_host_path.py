"""The host path of ordinary calls (csrc/ktanh_torch.cpp) against the Python code that takes all others:
the same results, the same graph, and the calls that have to go to the Python code go there."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1909_07729_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1909_07729_amd import autograd, binding
    binding.load_library()
    torch.cuda.set_device(0)
    return binding, autograd, torch


@pytest.fixture
def python_only(gpu, monkeypatch):
    """Switches the host path off inside a `with`."""
    binding, _, _ = gpu

    class Off:
        def __enter__(self):
            self.patch = pytest.MonkeyPatch()
            self.patch.setattr(binding, "_host", None)
            self.patch.setattr(binding, "_calls", {})

        def __exit__(self, *exc):
            self.patch.undo()
    return Off


def _same(torch, a, b):
    assert type(a) is type(b)
    if isinstance(a, (tuple, list)):
        assert len(a) == len(b)
        for x, y in zip(a, b):
            _same(torch, x, y)
        return
    assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.requires_grad == b.requires_grad
    assert a.is_leaf == b.is_leaf and a._is_view() == b._is_view()
    bits = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
    assert torch.equal(a.detach().view(bits), b.detach().view(bits))


def _values(torch, shape, dtype, seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    return (torch.randn(shape, generator=gen, device="cuda:0") * 2).to(dtype)


def test_every_entry_point_gives_the_same_through_both_paths(gpu, python_only):
    binding, _, torch = gpu
    tables = {"l": binding.ktanh_fit_lut_bmin0(), "L": binding.ktanh_fit_lut64()}
    tried = 0
    for name, kinds in binding.SIGNATURES.items():
        if not kinds.startswith("pp") or "klstm" in name:
            continue
        assert name in binding._calls, name
        dtype = torch.float32 if "_f32" in name else torch.bfloat16
        ins = [_values(torch, (7, 41), dtype, seed) for seed in range(2 if kinds.startswith("ppp") else 1)]
        table = [tables[k] for k in kinds if k in tables]
        for shape in ((7, 41), (0, 3), (1,)):
            xs = [t.flatten()[:int(np.prod(shape))].view(shape) for t in ins]
            for kwargs in ({}, *({"lut": t} for t in table)):
                fast = getattr(binding, name)(*xs, **kwargs)
                with python_only():
                    _same(torch, fast, getattr(binding, name)(*xs, **kwargs))
                out = torch.empty_like(fast)
                keyword = "dx" if len(xs) == 2 else "out"
                assert getattr(binding, name)(*xs, **kwargs, **{keyword: out}) is out
                _same(torch, fast, out)
                assert binding._calls[name](*xs, None, *([kwargs.get("lut")])) is not None
                tried += 1
    assert tried > 100
    for entry, table in (("klstm_cell", tables["l"]), ("klstm_cell64", tables["L"])):
        gates, c = _values(torch, (3, 2, 32), torch.bfloat16, 5), _values(torch, (2, 8), torch.float32, 6)
        dh, dc = _values(torch, (2, 8), torch.bfloat16, 7), _values(torch, (2, 8), torch.float32, 8)
        for kwargs in ({}, {"lut": table}):
            fast = getattr(binding, entry)(gates, c, **kwargs)
            back = getattr(binding, entry + "_backward")(gates[0], c, dh, dc, **kwargs)
            with python_only():
                _same(torch, fast, getattr(binding, entry)(gates, c, **kwargs))
                _same(torch, back, getattr(binding, entry + "_backward")(gates[0], c, dh, dc, **kwargs))
            given = getattr(binding, entry)(gates, c, c_out=fast[0], h_out=fast[1], **kwargs)
            assert given[0] is fast[0] and given[1] is fast[1]
            outs = torch.empty_like(back[0]), torch.empty_like(back[1])
            given = getattr(binding, entry + "_backward")(gates[0], c, dh, dc, dgates=outs[0], dc_prev=outs[1], **kwargs)
            assert given[0] is outs[0] and given[1] is outs[1]
            _same(torch, given, back)


def test_ordinary_calls_are_taken(gpu):
    """None of the functions declines what it is there for: else the other tests would hold the Python code against itself."""
    binding, autograd, torch = gpu
    host = binding._host
    x, g = _values(torch, (4, 8), torch.bfloat16, 1), _values(torch, (2, 32), torch.bfloat16, 2)
    c, dh = _values(torch, (2, 8), torch.float32, 3), _values(torch, (2, 8), torch.bfloat16, 4)
    for wide in (False, True):
        assert host.cell(g.unsqueeze(0), c, None, None, None, wide) is not None
        assert host.cell(g.unsqueeze(0), c, torch.empty_like(c), dh.unsqueeze(0).clone(), None, wide) is not None
        assert host.cell_backward(g, c, dh, c, None, None, None, wide) is not None
        assert host.cell_backward(g, c, dh, c, torch.empty_like(g), torch.empty_like(c), None, wide) is not None
        assert host.train_cell(g, c, wide) is not None
        cell = host.train_cell(g.clone().requires_grad_(), c, wide)
        assert all("KLstmCell" not in type(t.grad_fn).__name__ for t in cell) and all(t.requires_grad for t in cell)
    for code in range(8):
        for t in (x, x.float()):
            assert host.train(code, t) is not None
            y = host.train(code, t.clone().requires_grad_())
            assert y.requires_grad and type(y.grad_fn).__name__ not in ("_FromOutputBackward", "_FromInputBackward")
    with torch.no_grad():
        assert host.train(0, x.clone().requires_grad_()) is not None
    # and through the functions that programs call
    for fn in (autograd.ktanh, autograd.ksigmoid, autograd.kswish, autograd.kgelu):
        assert type(fn(x.clone().requires_grad_()).grad_fn).__name__ not in ("_FromOutputBackward", "_FromInputBackward")
    assert "KLstmCell" not in type(autograd.klstm_cell(g.clone().requires_grad_(), c)[0].grad_fn).__name__


def test_calls_that_are_not_ordinary_go_to_the_python_code(gpu):
    binding, _, torch = gpu
    x = _values(torch, (4, 8), torch.bfloat16, 1)
    call, grad, host = binding._calls["kgelu"], binding._calls["kgelu_backward"], binding._host

    class Other(torch.Tensor):
        pass

    for bad in (x.cpu(), x.float(), x.t(), x.view(torch.int16), x.as_subclass(Other), None, 3, torch.empty(0)):
        assert call(bad, None, None) is None
        assert grad(bad, x, None, None) is None and grad(x, bad, None, None) is None
        assert host.train(6, bad) is None or (isinstance(bad, torch.Tensor) and bad.dtype == torch.float32 and bad.is_cuda)
    assert call(x, torch.empty(31, device=x.device, dtype=x.dtype), None) is None
    assert call(x, None, binding.ktanh_fit_lut64()) is None and call(x, None, 5) is None
    assert grad(x, x[:2], None, None) is None
    with pytest.raises(ValueError):
        binding.kgelu(x.t())
    with pytest.raises(TypeError):
        binding.kgelu(x.float())
    with pytest.raises(ValueError):
        binding.kgelu(x.cpu())
    with pytest.raises(ctypes.ArgumentError):
        binding.kgelu(x, lut=binding.ktanh_fit_lut64())
    # a table the library refuses, through the host path
    rows = binding.ktanh_default_lut().as_tuples()
    rows[3] = (126, 8, 0)
    with pytest.raises(binding.KtanhError) as err:
        binding.kgelu(x, lut=binding.KtanhLut.from_tuples(rows))
    assert err.value.status == 3 and "kgelu" in str(err.value)
    # cell shapes that do not agree
    c = _values(torch, (2, 8), torch.float32, 2)
    for gates in (x, _values(torch, (1, 2, 31), torch.bfloat16, 3), _values(torch, (1, 3, 32), torch.bfloat16, 3)):
        assert host.cell(gates, c, None, None, None, False) is None
        with pytest.raises(ValueError):
            binding.klstm_cell(gates, c)
    with pytest.raises(binding.KtanhError):     # H not a multiple of 8
        binding.klstm_cell(_values(torch, (1, 2, 16), torch.bfloat16, 3), c[:, :4].contiguous())


def test_modes_and_transforms_see_the_python_code(gpu, python_only):
    binding, autograd, torch = gpu
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode
    x = _values(torch, (4, 8), torch.bfloat16, 1)
    seen = []

    class Functions(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    for mode in (Functions, Dispatch):
        seen.clear()
        with mode():
            y = binding.kgelu(x)
        assert seen and torch.equal(y, binding.kgelu(x))
    leaf = x.clone().requires_grad_()
    for attempt in (lambda: torch.func.vmap(autograd.kgelu)(x), lambda: torch.func.grad(lambda v: autograd.kgelu(v).sum())(x)):
        with pytest.raises(Exception) as fast:
            attempt()
        with python_only(), pytest.raises(type(fast.value)):
            attempt()
    with torch.autograd.forward_ad.dual_level():
        dual = torch.autograd.forward_ad.make_dual(x, torch.ones_like(x))
        assert binding._host.train(6, dual) is None
    traced = torch.jit.trace(autograd.kgelu, (x,), check_trace=False)
    other = _values(torch, (4, 8), torch.bfloat16, 9)
    assert torch.equal(traced(other), autograd.kgelu(other))
    # a batched gradient has no memory of its own: refused as before
    y = autograd.kgelu(leaf)
    with pytest.raises(RuntimeError):
        torch.autograd.grad(y, leaf, torch.stack([x, x]), is_grads_batched=True)


@pytest.mark.parametrize("dtype", ["bfloat16", "float32"])
@pytest.mark.parametrize("intervals", [32, 64])
def test_gradients_of_activations(gpu, python_only, dtype, intervals):
    _, autograd, torch = gpu
    dtype = getattr(torch, dtype)
    dy = _values(torch, (5, 33), dtype, 4)
    for fn in (autograd.ktanh, autograd.ksigmoid, autograd.kswish, autograd.kgelu):
        def step(grad=dy, make=lambda y, x: y):
            x = _values(torch, (5, 33), dtype, 3).requires_grad_()
            y = fn(x, intervals=intervals)
            return [y, *torch.autograd.grad(make(y, x), x, grad)]
        fast = step()
        summed = step(None, lambda y, x: y.sum())        # an expanded gradient, stride 0
        twice = step(dy, lambda y, x: y * x)
        with python_only():
            _same(torch, fast, step())
            _same(torch, summed, step(None, lambda y, x: y.sum()))
            _same(torch, twice, step(dy, lambda y, x: y * x))
        with torch.no_grad():
            y = fn(_values(torch, (5, 33), dtype, 3).requires_grad_(), intervals=intervals)
            assert not y.requires_grad
            _same(torch, y, fast[0].detach())
        # saved tensors are released, checked for changes in place, and go through saved-tensor hooks
        x = _values(torch, (5, 33), dtype, 3).requires_grad_()
        y = fn(x, intervals=intervals)
        y.backward(dy)
        with pytest.raises(RuntimeError):
            y.backward(dy)
        x = _values(torch, (5, 33), dtype, 3).requires_grad_()
        inner = x * 1
        y = fn(inner, intervals=intervals)
        saved, other = (y, inner) if fn in (autograd.ktanh, autograd.ksigmoid) else (inner, y)
        other.detach().add_(1)                           # the one that is not saved may change
        (g,) = torch.autograd.grad(y, x, dy, retain_graph=True)
        _same(torch, g, fast[1])
        saved.detach().add_(1)
        with pytest.raises(RuntimeError, match="modified by an inplace operation"):
            y.backward(dy)
        packed = []
        with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t) or t.cpu(), lambda t: t.to("cuda:0")):
            x = _values(torch, (5, 33), dtype, 3).requires_grad_()
            y = fn(x, intervals=intervals)
        assert len(packed) == 1
        _same(torch, list(torch.autograd.grad(y, x, dy)), fast[1:])
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t.cpu()):
            y = fn(x, intervals=intervals)
        with pytest.raises(ValueError):                  # what comes back has to be on the GPU
            torch.autograd.grad(y, x, dy)
        # a gradient of a gradient has no graph, as before
        y = fn(x, intervals=intervals)
        (g,) = torch.autograd.grad(y, x, dy, create_graph=True)
        assert not g.requires_grad


@pytest.mark.parametrize("intervals", [32, 64])
def test_gradients_of_the_cell(gpu, python_only, intervals):
    _, autograd, torch = gpu
    B, H = 3, 16

    def leaves():
        return (_values(torch, (B, 4 * H), torch.bfloat16, 1).requires_grad_(),
                _values(torch, (B, H), torch.float32, 2).requires_grad_())

    def step(use):
        g, c = leaves()
        h, c1 = autograd.klstm_cell(g, c, intervals=intervals)
        h2, c2 = autograd.klstm_cell(g.detach() * 1, c1, intervals=intervals)
        outs = {"h": [h, h2], "c": [c2], "both": [h, h2, c2], "sum": [h2.float().sum() + c2.sum()]}[use]
        return [h, c1, h2, c2, *torch.autograd.grad(outs, [g, c], [torch.ones_like(o) for o in outs])]
    for use in ("h", "c", "both", "sum"):        # an output that takes no part arrives as zeros
        fast = step(use)
        with python_only():
            _same(torch, fast, step(use))
    for needs in (0, 1):
        g, c = leaves()
        (g, c)[needs].requires_grad_(False)
        out = autograd.klstm_cell(g, c, intervals=intervals)
        assert out[0].requires_grad and out[1].requires_grad
        (grad,) = torch.autograd.grad(out, (g, c)[1 - needs], [torch.ones_like(o) for o in out])
        assert grad.shape == (g, c)[1 - needs].shape
    g, c = leaves()
    h, _ = autograd.klstm_cell(g, c, intervals=intervals)
    with pytest.raises(RuntimeError):            # h is a view of the multi-step result, as before
        h.add_(1)


def test_streams_and_threads(gpu):
    """Each thread's calls and their gradients run on the stream that the thread has made current."""
    binding, autograd, torch = gpu
    n, rounds = 1 << 20, 20
    x = [_values(torch, n, torch.bfloat16, seed) for seed in range(4)]
    want = []
    for t in x:
        leaf = t.clone().requires_grad_()
        y = autograd.kgelu(leaf)
        want.append((y.detach(), *torch.autograd.grad(y, leaf, t)))
    torch.cuda.synchronize()
    wrong, ended = [], []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(rounds):
                    leaf = torch.empty_like(x[k]).copy_(x[k]).requires_grad_()
                    y = autograd.kgelu(leaf)
                    (dx,) = torch.autograd.grad(y, leaf, x[k])
                    if not (torch.equal(y.detach(), want[k][0]) and torch.equal(dx, want[k][1])):
                        wrong.append(k)
            ended.append(k)
        except BaseException as error:
            wrong.append((k, repr(error)))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not wrong and sorted(ended) == [0, 1, 2, 3]
    graph = torch.cuda.CUDAGraph()               # a captured call, replayed on new values
    src = x[0].clone()
    with torch.cuda.graph(graph):
        y = binding.kgelu(src)
    for k in (1, 2, 3):
        src.copy_(x[k])
        graph.replay()
        assert torch.equal(y, want[k][0])
