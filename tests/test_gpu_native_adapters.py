"""GPU: the native autograd nodes of the VeRA and DoRA layers against the Python nodes they stand in for: the same bits over layouts, types
and skipped gradients, the same saved tensors, errors and refusals, threads and streams, and the Python node where it must run."""
import pytest

from paper_2312_03415_amd import binding as rl

pytestmark = pytest.mark.gpu

N, I, O, R = 70, 136, 264, 16


def functions(kind):
    """(function, the same on its Python node: what a subclass runs)"""
    from paper_2312_03415_amd import module
    base = module.RunVeRAFunction if kind == "vera" else module.RunDoRAFunction

    class Sub(base):
        pass
    return base.apply, Sub.apply


def native(kind, *args):
    from paper_2312_03415_amd.module import _native
    return getattr(_native(), kind)(*args)


def operands(kind, dtype, seed=0, n=N, i=I, o=O):
    """x, W, [A, B, vectors ...], bias, dy"""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    mk = lambda *s: (torch.randn(*s, generator=g, device="cuda") / s[0] ** 0.5).to(dtype)
    x, W, A, B = mk(n, i), mk(i, o), mk(i, R), mk(R, o)
    vectors = [mk(R) + 0.5, mk(o)] if kind == "vera" else [W.float().norm(dim=0).to(dtype)]
    return x, W, [A, B, *vectors], mk(o), mk(n, o)


def tail(kind, bias, pair):
    return (bias, 0.5, pair) if kind == "vera" else (bias, 0.5, pair[1])


def run(fn, kind, x, W, params, bias, dy, pair, want=None):
    import torch
    first = 2 if kind == "vera" else 0       # VeRA's A and B are frozen
    want = [True] * (1 + len(params) - first) if want is None else want
    xs = x.detach().requires_grad_(want[0])
    ps = [p.detach().requires_grad_(k >= first and want[1 + k - first]) for k, p in enumerate(params)]
    y = fn(xs, W, *ps, *tail(kind, bias, pair))
    ins = [t for t in (xs, *ps) if t.requires_grad]
    return [y.detach(), *torch.autograd.grad(y, ins, dy.reshape(y.shape))], y


PAIRS = {"vera": [(1, 1), (0, 0), (2, 5), (3, 6)], "dora": [(2, 4), (2, 5), (2, 7), (2, 8)]}


@pytest.mark.parametrize("kind,dtype", [("vera", "bfloat16"), ("vera", "float16"), ("vera", "float32"), ("dora", "bfloat16"), ("dora", "float16")])
def test_native_nodes_give_the_python_nodes_bits(kind, dtype):
    import torch
    fn, py = functions(kind)
    x, W, params, bias, dy = operands(kind, getattr(torch, dtype))
    forms = [x, x.view(2, 35, I), torch.cat([x, x], 1)[:, :I], x.t().contiguous().t(), x.new_zeros(N, 144)[:, 4:140]]
    for pair in PAIRS[kind]:
        for k, xf in enumerate(forms):
            for b in (bias, None):
                assert native(kind, xf, W, *params, *tail(kind, b, pair)) is not None
                got, y = run(fn, kind, xf, W, params, b, dy, pair)
                want, _ = run(py, kind, xf, W, params, b, dy, pair)
                assert ("VeRANode" if kind == "vera" else "DoRANode") in y.grad_fn.name()
                for g, w in zip(got, want):
                    assert g.shape == w.shape and torch.equal(g, w), (pair, k, b is None)
    wide = torch.cat([dy, dy], 1)[:, O:]     # a strided upstream gradient, single gradients
    count = len(got) - 1
    for one in range(count):
        want_g = [k == one for k in range(count)]
        got, _ = run(fn, kind, x, W, params, bias, wide, PAIRS[kind][1], want_g)
        want, _ = run(py, kind, x, W, params, bias, wide, PAIRS[kind][1], want_g)
        assert all(torch.equal(g, w) for g, w in zip(got, want)), want_g


@pytest.mark.parametrize("kind", ["vera", "dora"])
def test_saved_tensors_errors_and_refusals(kind):
    import torch
    fn, py = functions(kind)
    x, W, params, bias, dy = operands(kind, torch.bfloat16)
    pair, td = PAIRS[kind][0], torch.bfloat16

    def packed(f, unpack=lambda t: t.cuda()):
        seen = []
        with torch.autograd.graph.saved_tensors_hooks(lambda t: (seen.append((tuple(t.shape), t.dtype)), t.cpu())[1], unpack):
            out, _ = run(f, kind, x, W, params, bias, dy, pair)
        return seen, out
    (sa, ga), (sb, gb) = packed(fn), packed(py)
    assert sa == sb and all(torch.equal(a, b) for a, b in zip(ga, gb))
    # what a hook returns is what the backward reads, or refuses
    vec = params[-1]
    for change, shape in ((lambda t: t.t().contiguous().t(), (I, O)), (lambda t: t.cpu(), (I, O)), (lambda t: t.float(), tuple(vec.shape)),
                          (lambda t: t.repeat_interleave(2)[::2], tuple(vec.shape)), (lambda t: t.cpu(), (N, I))):
        only = lambda t: change(t.cuda()) if tuple(t.shape) == shape and t.dtype == td else t.cuda()
        for f in (fn, py):
            with pytest.raises(ValueError):
                packed(f, only)
    wide = lambda t: torch.cat([t.cuda()] * 2, 1)[:, :t.shape[1]] if t.dim() == 2 else t.cuda()
    for f in (fn, py):
        assert all(torch.equal(a, b) for a, b in zip(packed(f, wide)[1], ga))
    messages = []
    for f in (fn, py):
        z = x.clone().requires_grad_(True) * 1.0
        y = f(z, W, *params, *tail(kind, bias, pair))
        with pytest.raises(RuntimeError, match="view"):       # the output is a view made inside the node
            y.add_(1.0)
        y = f(z, W, *params, *tail(kind, bias, pair))
        z.add_(1.0)                                            # a saved tensor changed in place
        with pytest.raises(RuntimeError, match="inplace") as e:
            y.sum().backward()
        messages.append(str(e.value))
        if kind == "dora":                                     # the output is saved too
            y = f(x.clone().requires_grad_(True) * 1.0, W, *params, *tail(kind, bias, pair))
            y.detach().add_(1.0)
            with pytest.raises(RuntimeError, match="inplace"):
                y.sum().backward()
        with pytest.raises(rl.RunLoRAError) as e:
            y = f(x.clone().requires_grad_(True), W, *params, *tail(kind, None, (1, 0) if kind == "vera" else (2, 1)))
            y.sum().backward()
        assert e.value.code == (rl.RL_ERR_SAVED_MISMATCH if kind == "vera" else rl.RL_ERR_UNSUPPORTED)
        with torch.no_grad():
            assert not f(x.clone().requires_grad_(True), W, *params, *tail(kind, bias, pair)).requires_grad
    assert messages[0] == messages[1]

    class Sub(torch.Tensor):
        pass
    args = lambda xx=x, ww=W, pp=params: (xx, ww, *pp, *tail(kind, bias, pair))
    assert native(kind, *args(x.as_subclass(Sub))) is None
    assert native(kind, *args(x.cpu())) is None and native(kind, *args(x.double())) is None and native(kind, *args(x[:0])) is None
    assert native(kind, *args(ww=W.t().contiguous().t())) is None
    assert native(kind, *args(pp=[*params[:-1], vec.float()])) is None
    assert native(kind, *args(pp=[*params[:-1], vec.repeat_interleave(2)[::2]])) is None
    assert native(kind, *args(pp=[*params[:-1], vec[:-8]])) is None

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, a=(), kw=None):
            return func(*a, **(kw or {}))
    with Mode():
        assert native(kind, *args()) is None
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: fn(t, W, *params, *tail(kind, bias, pair)).float().sum())(x)


@pytest.mark.parametrize("kind", ["vera", "dora"])
def test_both_nodes_on_streams_and_threads(kind):
    """Four threads with a stream each: every pass gives the bits of one computed alone, on the native node and on the Python one."""
    import threading

    import torch
    for f in functions(kind):
        cases = [operands(kind, torch.bfloat16, k, 300 + 40 * k, 520, 776) for k in range(4)]
        one = lambda c: run(f, kind, c[0], c[1], c[2], c[3], c[4], PAIRS[kind][0])[0]
        alone = [one(c) for c in cases]
        torch.cuda.synchronize()
        out, errors = {}, []

        def work(k):
            try:
                s = torch.cuda.Stream()
                s.wait_stream(torch.cuda.default_stream())
                with torch.cuda.stream(s):
                    for _ in range(8):
                        out[k] = one(cases[k])
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
