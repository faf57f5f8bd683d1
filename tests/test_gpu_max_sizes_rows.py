"""The row entry points on 2^30 + 4099 problems: the library launches chunks of
2^30 problems, from one to the next of which rows advance three times as far as
single elements.  A seeded set of 2^20 problems is repeated on the device, and
every copy of the outputs equals the first, bit for bit, the ragged tail too."""
import pytest
import torch

import workloads
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu

BASE = 1 << 20
BIG = (1 << 30) + 4099


def repeated(t):
    return t.repeat(BIG // BASE + 1, *[1] * (t.dim() - 1))[:BIG].contiguous()


def same(big, base):
    body, tail = big[:BIG // BASE * BASE].view(BIG // BASE, *base.shape), big[BIG // BASE * BASE:]
    return all(torch.equal(body[k:k + 64], base.expand(64, *base.shape)) for k in range(0, BIG // BASE, 64)) \
        and torch.equal(tail, base[:tail.shape[0]])


@pytest.fixture
def free_memory():
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_rows_beyond_one_dispatch(free_memory, precision):
    import paper_2006_12838_amd as P

    nx, ny, nz, V0 = dev(*workloads.plic_problems(BASE, seed=9, edge_frac=0.0))
    n, V0, g = torch.stack([nx, ny, nz], 1), V0 * 0.98 + 0.01, dev(workloads.upstream_grad(BASE, seed=10))
    bn, bV0, bg = (repeated(t) for t in (n, V0, g))
    print(f"problems: {BIG}", flush=True)

    def forward(n, V0):
        d0, copy, back = torch.empty_like(V0), torch.empty_like(n), torch.empty_like(V0)
        P.plic_offset_rows_f32(n, V0, d0, copy, "sz", precision)
        P.plic_volume_rows_f32(n, d0, back, precision)
        return d0, copy, back

    def backward(n, V0, g):
        gn, gv = torch.empty_like(n), torch.empty_like(V0)
        P.plic_offset_backward_rows_f32(n, V0, g, gn, gv, "sz", precision)
        return gn, gv

    for f, big, base in ((forward, (bn, bV0), (n, V0)), (backward, (bn, bV0, bg), (n, V0, g))):
        for k, (b, s) in enumerate(zip(f(*big), f(*base))):
            assert torch.isfinite(s).all() and same(b, s), (f.__name__, k)
