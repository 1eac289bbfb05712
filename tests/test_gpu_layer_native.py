"""The layer's C++ autograd function against its Python twin: the same bits for every choice of what is learned, in steps,
without gradients, with a graph of the backward pass and over batches of upstream gradients; what one of them refuses the
other refuses as well."""
import weakref

import pytest

torch = pytest.importorskip("torch")

from paper_2510_20271_amd import api, layer, synth
from paper_2510_20271_amd.layer import SoftECCLayer

pytestmark = pytest.mark.gpu


def _layer(ndim, T, tilted=False, learn_tau=True, learn_theta=True, lam=20.0):
    angles = [0.3] if ndim == 2 else [0.3, 1.1]
    return SoftECCLayer(ndim, T, -1.0, 1.0, lam=lam, theta=angles, learn_tau=learn_tau, learn_theta=learn_theta,
                        tilted_c=tilted).cuda()


def _grid(shape):
    return torch.from_numpy(synth.grf_batch(shape[0], shape[1:], 2.0, 17)).cuda()


def _both(monkeypatch, fn):
    """fn through the C++ function, which has to return (the Python one is not there to step in), then through Python."""
    returned = []
    real = layer._native()

    def counted(*args):
        chi = real(*args)
        returned.append(chi)
        assert chi.grad_fn is None or "SoftECCAngles" not in type(chi.grad_fn).__name__
        return chi

    def absent(*args):
        raise AssertionError("the Python function was taken")

    with monkeypatch.context() as m:
        m.setattr(layer, "_native", lambda: counted)
        m.setattr(layer._SoftECCAngles, "apply", absent)
        a = fn()
    assert returned
    monkeypatch.setattr(layer, "_native_takes", lambda *args: False)
    return a, fn()


@pytest.mark.parametrize("shape", [(1, 30, 40), (3, 61, 67), (2, 12, 20, 33)])
@pytest.mark.parametrize("T", [1, 37, 300])
@pytest.mark.parametrize("learn", [(True, True, True), (False, True, False), (False, False, True), (True, False, False)])
def test_same_bits(monkeypatch, shape, T, learn):
    need_x, need_tau, need_theta = learn

    def step():
        m = _layer(len(shape) - 1, T, tilted=T == 37, learn_tau=need_tau, learn_theta=need_theta)
        x = _grid(shape).requires_grad_(need_x)
        chi = m(x)
        g = torch.linspace(-1.0, 2.0, chi.numel(), device="cuda").view_as(chi)
        chi.backward(g)
        with torch.no_grad():
            plain = m(x)
        assert not plain.requires_grad
        return chi.detach(), plain, x.grad, m.tau.grad, m.theta.grad

    a, b = _both(monkeypatch, step)
    for p, q, wanted in zip(a, b, (True, True, need_x, need_tau, need_theta)):
        assert (p is None) == (q is None) == (not wanted)
        assert p is None or torch.equal(p, q)


def test_graph_of_the_backward_pass_and_batched_gradients(monkeypatch):
    def run():
        m = _layer(3, 20)
        chi = m(_grid((2, 12, 20, 33)))
        g = torch.ones_like(chi).requires_grad_()
        gt, ga = torch.autograd.grad(chi, [m.tau, m.theta], g, create_graph=True)
        second = torch.autograd.grad(gt.sum() + ga.sum(), g, retain_graph=True)[0]
        m = _layer(3, 20, learn_theta=False)  # (a batch of upstream gradients: the thresholds alone)
        chi = m(_grid((2, 12, 20, 33)))
        many = torch.autograd.grad(chi, [m.tau], torch.stack([g.detach(), 2 * g.detach()]), is_grads_batched=True)[0]
        return gt.detach(), ga.detach(), second, many

    for p, q in zip(*_both(monkeypatch, run)):
        torch.testing.assert_close(p, q, rtol=1e-6, atol=1e-6)


def test_saved_tensors(monkeypatch):
    m, x = _layer(2, 9), _grid((2, 20, 30)).requires_grad_()
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: (packed.append(t.shape), t.clone())[1], lambda t: t):
        chi = m(x)
    assert packed
    chi.sum().backward()
    with pytest.raises(RuntimeError):  # a second time through a freed graph
        chi.sum().backward()
    chi = m(x)
    with torch.no_grad():
        x.add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        chi.sum().backward()


def test_refusals_stay(monkeypatch):
    with pytest.raises(api.EccError):
        _layer(2, 5, lam=-1.0)(_grid((1, 20, 30)))
    m, x = _layer(2, 5), _grid((1, 20, 30))
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: m(t).sum())(x)
    with pytest.raises(RuntimeError):
        torch.func.vmap(m)(x[None])
    with pytest.raises(ValueError):
        m(x[0])
    # other layouts and types go the Python way, with the same result
    want = m(x)
    assert torch.equal(m(x.transpose(1, 2).contiguous().transpose(1, 2)), want)
    assert torch.equal(m(x.double()), want)


@pytest.mark.parametrize("how", ["host", "strided", "short", "other type"])
@pytest.mark.parametrize("which", range(5))  # the input, the derivatives, the thresholds, the state, the angles
def test_what_a_hook_hands_back_is_checked(which, how):
    """A saved-tensor hook that returns something else than was saved is refused before any kernel sees it."""
    change = {"host": lambda t: t.cpu(), "strided": lambda t: torch.stack([t, t], -1)[..., 0],
              "short": lambda t: t.reshape(-1)[: t.numel() // 2].clone(),
              "other type": lambda t: t.double() if t.is_floating_point() else t.short()}[how]
    m = SoftECCLayer(3, 9, -1.0, 1.0, theta=[0.3, 1.1]).cuda()
    x, seen = _grid((2, 12, 20, 33)).requires_grad_(), []

    def pack(t):
        seen.append(t)
        return len(seen) - 1, t

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: change(p[1]) if p[0] == which else p[1]):
        chi = m(x)
    assert len(seen) == 5
    with pytest.raises(ValueError if how != "short" or which != 3 else RuntimeError):
        chi.sum().backward()


def test_a_refusal_in_the_backward_pass_has_its_status():
    m, x, seen = _layer(2, 9), _grid((2, 20, 30)).requires_grad_(), []

    def pack(t):
        seen.append(t)
        return len(seen) - 1, t

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: p[1][:256].clone() if p[0] == 3 else p[1]):
        chi = m(x)  # (number 3 is the state)
    with pytest.raises(api.EccError, match="state") as e:
        chi.sum().backward()
    assert e.value.status == -3


def test_errors_of_the_native_function_are_the_callers(monkeypatch):
    """No second run through Python: memory that has run out, a hook's own error, a fault of the function itself."""
    m, x, calls = _layer(2, 9), _grid((2, 20, 30)), []

    def pack(t):
        calls.append(1)
        raise RuntimeError("of the hook")

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t):
        with pytest.raises(RuntimeError, match="of the hook"):
            m(x)
    assert len(calls) == 1
    for error in (torch.OutOfMemoryError("no memory"), RuntimeError("fault"), api.EccError(-1, "refused")):
        calls.clear()

        def fails(*args):
            calls.append(1)
            raise error

        monkeypatch.setattr(layer, "_native", lambda: fails)
        with pytest.raises(type(error)) as e:
            m(x)
        assert e.value is error and len(calls) == 1


def test_a_graph_keeps_no_workspace():
    """A step's workspace is the stream's: one that was replaced by a larger one goes, though a graph that used it is alive."""
    torch.cuda.synchronize()
    api._WS_CACHE.clear()
    m, x = _layer(2, 9), _grid((2, 20, 30)).requires_grad_()
    m(x).sum().backward()
    want, x.grad = x.grad, None
    chi = m(x)
    (kept,) = [weakref.ref(ws) for ws in api._WS_CACHE.values()]
    api.soft_step_workspace((300, 300), 4, 64, x.device)
    assert kept() is None
    chi.sum().backward()
    assert torch.equal(x.grad, want)


def test_a_node_run_on_another_stream_has_a_workspace_of_its_own():
    torch.cuda.synchronize()
    api._WS_CACHE.clear()
    m, x = _layer(2, 1000), _grid((40, 30, 40)).requires_grad_()
    g = torch.ones(40, 1000, device="cuda")  # (the contraction takes several blocks, whose sums go through the workspace)
    m(x).backward(g)
    chi = m(x)
    (ws,) = api._WS_CACHE.values()
    ws.fill_(0xAB)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()), torch.no_grad():
        grad_x, grad_theta, grad_tau = chi.grad_fn(g)[:3]
    torch.cuda.synchronize()
    assert bool((ws == 0xAB).all())
    assert torch.equal(grad_x, x.grad) and torch.equal(grad_tau, m.tau.grad) and torch.equal(grad_theta, m.theta.grad)


def test_parameters_of_other_types():
    """alpha, lam and tilted_c may be whatever float() and bool() take, as through the Python function."""
    m, x = _layer(2, 9), _grid((2, 20, 30))
    want = m(x)
    m.alpha, m.lam, m.tilted_c = torch.tensor(m.alpha), "20.0", ""
    assert torch.equal(m(x), want)
