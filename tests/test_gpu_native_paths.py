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
