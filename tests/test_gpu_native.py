"""The native torch functions behind offset, volume and curvature: the bits of
the Python autograd functions (PlicOffset, PlicCurvature) on the same tensors,
and the same behaviour around them: what needs no gradient makes no node, a
changed input is noticed, a second backward works, function transforms and
unknown options are refused as before, side streams."""
import pytest
import torch

from tests.gpu_util import dev
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2006_12838_amd as P
    return P


def problems(dtype, m=3001):
    import numpy as np
    nx, ny, nz, V0 = workloads.plic_problems(m, seed=21, dtype=np.float64 if dtype == torch.float64 else np.float32)
    return dev(nx, ny, nz, V0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("form", ["rows", "parts"])
def test_offset_equals_the_python_function(P, dtype, form):
    t = [x.requires_grad_(True) for x in problems(dtype)]
    w = torch.randn_like(t[3])
    want = P.PlicOffset.apply(*t, "sz", "mixed")
    gw = torch.autograd.grad(want, t, w)
    n = torch.stack([x.detach() for x in t[:3]], -1).requires_grad_(True) if form == "rows" else tuple(t[:3])
    got = P.offset(n, t[3], "sz", "mixed")
    assert type(got.grad_fn) is not type(want.grad_fn) and torch.equal(got, want)
    gg = torch.autograd.grad(got, (n, t[3]) if form == "rows" else t, w)
    if form == "rows":
        gg = (*gg[0].unbind(-1), gg[1])
    for a, b in zip(gg, gw):
        assert torch.equal(a, b)
    with torch.no_grad():
        assert P.offset(n, t[3]).grad_fn is None
    if form == "rows":
        plain = n.detach()
        assert P.offset(plain, t[3].detach()).grad_fn is None
        assert torch.equal(P.volume(plain, want.detach()), P.volume(tuple(plain.unbind(-1)), want.detach()))


def test_options_and_transforms(P):
    nx, ny, nz, V0 = problems(torch.float32, 64)
    n = torch.stack([nx, ny, nz], -1)
    with pytest.raises(ValueError):
        P.offset(n, V0, "bisection")
    with pytest.raises(ValueError):
        P.offset(n, V0, "sz", "double")
    P.offset(n.double(), V0.double(), "sz", "double")            # float64 never looked at the precision
    with pytest.raises(RuntimeError, match="PLIC_EINVAL"):
        P.offset(n, V0, 99)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda v: P.offset(n, v).sum())(V0)
    with pytest.raises(Exception):
        torch.vmap(lambda a, v: P.offset(a, v))(n, V0)
    with pytest.raises(ValueError):
        P.offset(n.cpu(), V0.cpu())
    e = P.offset(n[:0], V0[:0])
    assert e.shape == (0,)
    with torch.autograd.forward_ad.dual_level():
        with pytest.raises(Exception):
            P.offset(n, torch.autograd.forward_ad.make_dual(V0, torch.ones_like(V0)))
    v = V0.clone().requires_grad_(True)
    d0 = P.offset(n, v * 1.0)
    x = v * 1.0
    d0 = P.offset(n, x)
    x.mul_(0.5)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        d0.sum().backward()


@pytest.mark.parametrize("neighbours", [False, True])
def test_curvature_equals_the_python_function(P, neighbours):
    phi, _ = workloads.sphere_lattice(N=30, R=9.0, seed=4)
    tp = dev(phi).requires_grad_(True)
    w = torch.randn_like(tp)
    want = P.PlicCurvature.apply(tp, "sz", "mixed", "cm", neighbours)
    gw, = torch.autograd.grad(want, tp, w)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = P.curvature(tp, "sz", "mixed", "cm", neighbours)
        g1, = torch.autograd.grad(got, tp, w, retain_graph=True)
        g2, = torch.autograd.grad(got, tp, w)
    side.synchronize()
    assert torch.equal(got, want) and torch.equal(g1, gw) and torch.equal(g2, gw)
    with pytest.raises(RuntimeError, match="PLIC_EINVAL"):
        P.curvature(tp, "sz_kawano")
    with pytest.raises(ValueError):
        P.curvature(tp, "sz", "half")
    assert torch.equal(P.curvature(tp.detach().transpose(0, 2), "sz"),          # not contiguous: the Python path
                       P.curvature(tp.detach().transpose(0, 2).contiguous(), "sz"))
