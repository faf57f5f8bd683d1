"""The Python functions behind the native ones: what they serve when the native
functions are not there or not meant, and the same behaviour of both."""
import pytest
import torch

from tests.gpu_util import dev
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2006_12838_amd as P
    return P


@pytest.mark.parametrize("neighbours", [False, True])
@pytest.mark.parametrize("contiguous", [True, False])
def test_second_backward(P, neighbours, contiguous):
    """The workspace goes with the first backward; a second one scans again."""
    phi, _ = workloads.sphere_lattice(N=30, R=9.0, seed=6)
    tp = dev(phi)
    tp = (tp if contiguous else tp.transpose(0, 2)).detach().requires_grad_(True)
    k = P.curvature(tp, neighbour_normals=neighbours)
    w = torch.randn_like(k)
    first, = torch.autograd.grad(k, tp, w, retain_graph=True)
    second, = torch.autograd.grad(k, tp, w, retain_graph=True)
    third, = torch.autograd.grad(k, tp, w)
    assert first.abs().max() > 0 and torch.equal(first, second) and torch.equal(first, third)


FORMS = ("rows", "parts", "curvature")


def call(P, form, seed=7):
    """(differentiable inputs, their function, the Python autograd function's result on them)"""
    if form == "curvature":
        tp = dev(workloads.sphere_lattice(N=24, R=7.0, seed=seed)[0]).requires_grad_(True)
        return [tp], lambda p: P.curvature(p, "sz"), lambda p: P.PlicCurvature.apply(p, "sz")
    nx, ny, nz, V0 = dev(*workloads.plic_problems(2001, seed=seed, edge_frac=0.0))
    if form == "parts":
        return ([t.requires_grad_(True) for t in (nx, ny, nz, V0)], lambda x, y, z, v: P.offset((x, y, z), v),
                lambda x, y, z, v: P.PlicOffset.apply(x, y, z, v))
    n = torch.stack([nx, ny, nz], -1).requires_grad_(True)
    return [n, V0.requires_grad_(True)], lambda n, v: P.offset(n, v), lambda n, v: P.PlicOffset.apply(*n.unbind(-1), v)


def gradients(result, inputs):
    g = torch.Generator(device="cuda").manual_seed(1)
    return torch.autograd.grad(result, inputs, torch.randn(result.shape, generator=g, device="cuda"))


def equal(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("form", FORMS)
def test_both_functions_agree(P, form, monkeypatch):
    inputs, native, python = call(P, form)
    a, b = native(*inputs), python(*inputs)
    assert type(a.grad_fn) is not type(b.grad_fn)              # the native function made its own node
    want = gradients(b, inputs)
    assert torch.equal(a, b) and equal(gradients(a, inputs), want)
    if form == "rows":
        plain = [t.detach() for t in inputs]
        V0 = P._native.volume_rows(plain[0], a.detach(), 0)
        assert isinstance(V0, torch.Tensor) and torch.equal(V0, P.volume(tuple(plain[0].unbind(-1)), a.detach()))
    monkeypatch.setattr(P, "_native_may", lambda: False)       # as where it is not built
    c = native(*inputs)
    assert type(c.grad_fn) is not type(a.grad_fn) and torch.equal(a, c) and equal(gradients(c, inputs), want)


@pytest.mark.parametrize("form", FORMS)
def test_saved_tensors_on_the_host(P, form):
    inputs, native, _ = call(P, form)
    want = gradients(native(*inputs), inputs)
    with torch.autograd.graph.save_on_cpu():
        d = native(*inputs)
    assert equal(gradients(d, inputs), want)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("wrong", [lambda t: t.cpu(), lambda t: t.double(), lambda t: t[..., :1], lambda t: t.to_sparse(),
                                   lambda t: torch.stack([t, t], -1)[..., 0]],
                         ids=["host", "dtype", "short", "sparse", "strided"])
def test_a_hook_that_returns_another_tensor_is_refused(P, form, wrong):
    inputs, native, _ = call(P, form)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, wrong):
        d = native(*inputs)
    with pytest.raises(RuntimeError, match="saved tensor"):
        gradients(d, inputs)


@pytest.mark.parametrize("form", FORMS)
def test_errors_of_hooks_keep_their_type(P, form):
    class Own(Exception):
        pass

    def fail(t):
        raise Own("pack")

    inputs, native, _ = call(P, form)
    with torch.autograd.graph.saved_tensors_hooks(fail, lambda t: t):
        with pytest.raises(Own, match="pack"):
            native(*inputs)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("reentrant", [False, True])
def test_checkpointing(P, form, reentrant):
    from torch.utils.checkpoint import checkpoint

    inputs, native, _ = call(P, form)
    want = gradients(native(*inputs), inputs)
    d = checkpoint(native, *inputs, use_reentrant=reentrant)
    g = torch.Generator(device="cuda").manual_seed(1)
    d.backward(torch.randn(d.shape, generator=g, device="cuda"))
    assert equal([t.grad for t in inputs], want)


@pytest.mark.parametrize("form", FORMS)
def test_backward_on_another_thread_and_stream(P, form):
    import threading

    inputs, native, _ = call(P, form)
    want = gradients(native(*inputs), inputs)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        d = native(*inputs)
    got = []
    t = threading.Thread(target=lambda: got.extend(gradients(d, inputs)))
    t.start()
    t.join()
    torch.cuda.synchronize()
    assert equal(got, want)


@pytest.mark.parametrize("form", FORMS)
def test_dispatch_modes_see_the_python_path(P, form):
    from torch.utils._python_dispatch import TorchDispatchMode

    class Count(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.seen += 1
            return func(*args, **(kwargs or {}))

    inputs, native, python = call(P, form)
    want = native(*inputs)
    with Count() as mode:
        d = native(*inputs)
    assert mode.seen > 0 and type(d.grad_fn) is not type(want.grad_fn) and torch.equal(d, want)
