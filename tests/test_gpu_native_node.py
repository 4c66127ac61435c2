"""GPU: the native autograd node of the LoRA layer against the Python node it stands in for: the same bits over layouts,
types, options and skipped gradients, the same saved tensors, errors and refusals, and the Python node where it must run."""
import pytest

from paper_2312_03415_amd import binding as rl

pytestmark = pytest.mark.gpu


def layer(dtype, n=70, i=136, o=264, r=16, seed=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    mk = lambda *s: (torch.randn(*s, generator=g, device="cuda") / s[0] ** 0.5).to(dtype)
    return mk(n, i), mk(i, o), mk(i, r), mk(r, o), mk(o), mk(n, o)


def run(fn, x, W, A, B, dy, extra, want=(True, True, True)):
    import torch
    xs, As, Bs = (t.detach().requires_grad_(w) for t, w in zip((x, A, B), want))
    y = fn(xs, W, As, Bs, *extra)
    ins = [t for t, w in zip((xs, As, Bs), want) if w]
    return [y.detach(), *torch.autograd.grad(y, ins, dy.reshape(y.shape))], y


def python_node(*args):
    """RunLoRAFunction's Python node (what a subclass of it runs)."""
    from paper_2312_03415_amd.module import RunLoRAFunction

    class Sub(RunLoRAFunction):
        pass
    return Sub.apply(*args)


@pytest.mark.parametrize("dtype", ["bfloat16", "float16", "float32"])
@pytest.mark.parametrize("pair,merged,drop,keep_t", [((1, 1), False, None, False), ((0, 0), False, None, False), ((2, 5), True, None, False),
                                                     ((1, 5), False, None, True), ((1, 1), False, (0.25, 77), True), ((3, 6), False, None, False)])
def test_native_node_gives_the_python_nodes_bits(dtype, pair, merged, drop, keep_t):
    import torch
    from paper_2312_03415_amd.module import RunLoRAFunction, _native
    dt = getattr(torch, dtype)
    x, W, A, B, bias, dy = layer(dt)
    forms = [x, x.view(2, 35, 136), torch.cat([x, x], 1)[:, :136], x.t().contiguous().t(), torch.cat([x[:1, :8], x[:1, :8]], 1).new_zeros(70, 144)[:, 4:140]]
    for k, xf in enumerate(forms):
        for b in (bias, None):
            extra = (b, 0.5, pair, merged, drop, keep_t)
            assert _native().lora(xf, W, A, B, *extra) is not None
            got, y = run(RunLoRAFunction.apply, xf, W, A, B, dy, extra)
            want, yp = run(python_node, xf, W, A, B, dy, extra)
            assert "LoRANode" in type(y.grad_fn).__name__ or "LoRANode" in y.grad_fn.name()
            for g, w in zip(got, want):
                assert g.shape == w.shape and torch.equal(g, w), (k, b is None)
    # a strided upstream gradient, single gradients
    wide = torch.cat([dy, dy], 1)[:, 264:]
    for want_g in ((True, False, False), (False, True, False), (False, False, True)):
        got, _ = run(RunLoRAFunction.apply, x, W, A, B, wide, extra, want_g)
        want, _ = run(python_node, x, W, A, B, wide, extra, want_g)
        assert all(torch.equal(g, w) for g, w in zip(got, want)), want_g


def test_saved_tensors_errors_and_refusals_are_the_python_nodes():
    import torch
    from paper_2312_03415_amd.module import RunLoRAFunction, _native
    x, W, A, B, bias, dy = layer(torch.bfloat16)
    extra = (None, 1.0, (1, 1), False)

    def packed(fn):
        seen = []
        with torch.autograd.graph.saved_tensors_hooks(lambda t: (seen.append(tuple(t.shape)), t.cpu())[1], lambda t: t.cuda()):
            out, _ = run(fn, x, W, A, B, dy, extra)
        return seen, out
    (sa, ga), (sb, gb) = packed(RunLoRAFunction.apply), packed(python_node)
    assert sa == sb == [(70, 136), (136, 264), (136, 16), (16, 264)]
    messages = []
    for fn in (RunLoRAFunction.apply, python_node):
        xs = x.clone().requires_grad_(True)
        z = xs * 1.0
        y = fn(z, W, A, B, *extra)
        with pytest.raises(RuntimeError, match="view"):       # the output is a view made inside the node
            y.add_(1.0)
        y = fn(z, W, A, B, *extra)
        z.add_(1.0)                                            # a saved tensor changed in place
        with pytest.raises(RuntimeError, match="inplace") as e:
            y.sum().backward()
        messages.append(str(e.value))
        with pytest.raises(rl.RunLoRAError) as e:              # the default backward needs the default forward's T
            y = fn(xs, W, A, B, None, 1.0, (1, 0), False)
            y.sum().backward()
        assert e.value.code == rl.RL_ERR_SAVED_MISMATCH
        with pytest.raises(rl.RunLoRAError) as e:              # refused by the forward: no merged weight under dropout
            fn(xs, W, A, B, None, 1.0, (2, 1), False, (0.5, 1))
        assert e.value.code == rl.RL_ERR_UNSUPPORTED
        messages.append(str(e.value))
        with torch.no_grad():
            assert not fn(xs, W, A, B, *extra).requires_grad
    assert messages[:2] == messages[2:], messages

    # what has to see a Python-level function, or a message of the Python path, does not take the native node
    class Sub(torch.Tensor):
        pass
    assert _native().lora(x.as_subclass(Sub), W, A, B, *extra) is None
    assert _native().lora(x.cpu(), W, A, B, *extra) is None
    assert _native().lora(x.double(), W, A, B, *extra) is None
    assert _native().lora(x, W.t().contiguous().t(), A, B, *extra) is None
    assert _native().lora(x[:, :128], W, A, B, *extra) is None
    assert _native().lora(x[:0], W, A, B, *extra) is None
    seen = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))
    with Mode():
        assert _native().lora(x, W, A, B, *extra) is None
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: RunLoRAFunction.apply(t, W, A, B, *extra).float().sum())(x)


def under_hooks(fn, unpack, x, W, A, B, dy, extra):
    """A pass whose saved tensors leave as host copies (their device memory is free for others) and come back as unpack(t)."""
    import torch
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), unpack):
        xs, As, Bs = (t.detach().clone().requires_grad_(True) for t in (x, A, B))
        y = fn(xs * 1.0, W, As, Bs, *extra)
    churn = [torch.full((1 << k,), 7.0, device="cuda", dtype=x.dtype) for k in range(9, 18)]
    grads = torch.autograd.grad(y, (xs, As, Bs), dy)
    del churn
    return grads


@pytest.mark.parametrize("node", ["native", "python"])
def test_saved_tensors_that_come_back_changed(node):
    """What a saved-tensor hook returns is what the backward reads: moved to the host and back, or laid out anew, it gives the
    plain pass's bits; a type, layout or device that the forward would refuse is refused."""
    import torch
    from paper_2312_03415_amd.module import RunLoRAFunction
    fn = RunLoRAFunction.apply if node == "native" else python_node
    x, W, A, B, bias, dy = layer(torch.bfloat16)
    extra = (None, 0.5, (1, 1), False)
    plain, _ = run(fn, x, W, A, B, dy, extra)

    def wide(t):   # rows apart
        return torch.cat([t, t], 1)[:, :t.shape[1]]
    for unpack in (lambda t: t.cuda(), lambda t: wide(t.cuda()), lambda t: t.cuda().t().contiguous().t() if t.shape == x.shape else t.cuda()):
        got = under_hooks(fn, unpack, x, W, A, B, dy, extra)
        assert all(torch.equal(g, w) for g, w in zip(got, plain[1:]))
    only = lambda like, change: lambda t: change(t.cuda()) if t.shape == like.shape else t.cuda()
    for like, change, error in ((W, lambda t: t.t().contiguous().t(), ValueError), (A, lambda t: t.repeat_interleave(2, 1)[:, ::2], ValueError),
                                (W, lambda t: t.cpu(), ValueError), (x, lambda t: t.cpu(), ValueError),
                                (W, lambda t: t.float(), rl.RL_ERR_DTYPE), (B, lambda t: t.half(), rl.RL_ERR_DTYPE),
                                (x, lambda t: t.float(), rl.RL_ERR_DTYPE)):
        with pytest.raises(ValueError if error is ValueError else rl.RunLoRAError) as e:
            under_hooks(fn, only(like, change), x, W, A, B, dy, extra)
        assert error is ValueError or e.value.code == error, (tuple(like.shape), e.value)


def test_other_layers_read_what_a_saved_tensor_hook_returns():
    import torch
    from paper_2312_03415_amd.module import RunDoRALinear, RunVeRALinear
    x, W, A, B, bias, dy = layer(torch.bfloat16)
    dora, vera = RunDoRALinear(W, 16, bias=bias), RunVeRALinear(W, A, B, bias)
    with torch.no_grad():
        dora.lora_A.copy_(A), dora.lora_B.copy_(B), vera.vera_b.copy_(bias)
    for mod in (dora, vera):
        params = [p for p in mod.parameters() if p.requires_grad]
        xs = x.clone().requires_grad_(True)
        want = torch.autograd.grad(mod(xs * 1.0), [xs, *params], dy)
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
            y = mod(xs * 1.0)
        churn = [torch.full((1 << k,), 7.0, device="cuda", dtype=x.dtype) for k in range(9, 18)]
        got = torch.autograd.grad(y, [xs, *params], dy)
        assert all(torch.equal(g, w) for g, w in zip(got, want)), type(mod).__name__
        del churn


def test_native_node_on_streams_and_threads():
    """Two streams and two threads at once, each with passes of its own: every result is the one computed alone (no scratch
    is shared between calls)."""
    import threading

    import torch
    from paper_2312_03415_amd.module import RunLoRAFunction
    cases = [layer(torch.bfloat16, 300 + 40 * k, 520, 776, 16, seed=k) for k in range(4)]
    extra = (None, 1.0, (1, 1), False)
    alone = [run(RunLoRAFunction.apply, c[0], c[1], c[2], c[3], c[5], extra)[0] for c in cases]
    torch.cuda.synchronize()
    out, errors = {}, []

    def work(k):
        try:
            s = torch.cuda.Stream()
            s.wait_stream(torch.cuda.default_stream())
            with torch.cuda.stream(s):
                for rep in range(8):
                    c = cases[k]
                    out[k] = run(RunLoRAFunction.apply, c[0], c[1], c[2], c[3], c[5], extra)[0]
            s.synchronize()
        except Exception as e:   # noqa: BLE001 - reported by the main thread
            errors.append(e)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(4):
        assert all(torch.equal(a, b) for a, b in zip(out[k], alone[k])), k


@pytest.mark.parametrize("kind", ["lora", "vera", "dora"])
def test_python_nodes_on_streams_and_threads(kind):
    """The same for the nodes in Python, DoRA and VeRA among them."""
    import threading

    import torch
    from paper_2312_03415_amd.module import RunDoRALinear, RunVeRALinear
    jobs = []
    for k in range(4):
        x, W, A, B, bias, dy = layer(torch.bfloat16, 300 + 40 * k, 520, 776, 16, seed=k)
        if kind == "lora":
            jobs.append(lambda x=x, W=W, A=A, B=B, dy=dy: run(python_node, x, W, A, B, dy, (None, 1.0, (1, 1), False))[0])
            continue
        mod = RunVeRALinear(W, A, B, bias) if kind == "vera" else RunDoRALinear(W, 16, bias=bias)
        with torch.no_grad():
            mod.vera_b.copy_(bias) if kind == "vera" else (mod.lora_A.copy_(A), mod.lora_B.copy_(B))

        def job(mod=mod, x=x, dy=dy):
            xs = x.detach().requires_grad_(True)
            y = mod(xs)
            return [y.detach(), *torch.autograd.grad(y, [xs, *(p for p in mod.parameters() if p.requires_grad)], dy)]
        jobs.append(job)
    alone = [job() for job in jobs]
    torch.cuda.synchronize()
    out, errors = {}, []

    def work(k):
        try:
            s = torch.cuda.Stream()
            s.wait_stream(torch.cuda.default_stream())
            with torch.cuda.stream(s):
                for rep in range(8):
                    out[k] = jobs[k]()
            s.synchronize()
        except Exception as e:   # noqa: BLE001 - reported by the main thread
            errors.append(e)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(4):
        assert all(torch.equal(a, b) for a, b in zip(out[k], alone[k])), (kind, k)
