"""A lattice of 64 x 2052 x 2052 cells (263,169 tiles of 64 x 4 x 4): its groups are
48 tiles, three rounds of their scan; a lane that looks for work items owns runs
of groups; and the gather looks for its tiles in two stretches of 262,144.  Two
copies of a small perturbed sphere, one in the first tiles and one that ends in
the second stretch, give the bits of the small lattice alone, and zero is
everywhere else: forward, the backward that scans, the one that reuses the
forward's records, with and without neighbour normals."""
import pytest
import torch

import workloads
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu

BIG = (2052, 2052, 64)                        # (Z, Y, X)
N = 40
CORNERS = ((8, 8, 12), (2012, 2008, 12))      # (z, y, x); the second copy's last interface cells lie in z >= 2044


@pytest.fixture
def free_memory():
    yield
    torch.cuda.empty_cache()


def blocks(big):
    return [big[z:z + N, y:y + N, x:x + N] for z, y, x in CORNERS]


def embed(small, big):
    for b in blocks(big):
        b.copy_(small)
    return big


def check(big, small, what):
    for k, b in enumerate(blocks(big)):
        assert torch.equal(b, small), (what, k)
        b.zero_()
    assert not big.any(), what


@pytest.mark.parametrize("neighbours", [False, True])
def test_embedded_copies(free_memory, neighbours):
    import paper_2006_12838_amd as P

    phi, _, _ = workloads.perturbed_sphere_lattice(N=N, R=12.0, seed=13, ss=4)
    assert ((phi[32:36] > 0) & (phi[32:36] < 1)).any()           # z = 2044 .. 2047 of the second copy: tiles past 262,144
    sp, sg = dev(phi), dev(workloads.upstream_grad(phi.shape, seed=14))
    cells = int(((sp > 0) & (sp < 1)).sum())
    o = ("sz", "mixed", "py", neighbours)
    ks, gs = torch.empty_like(sp), torch.empty_like(sp)
    # every row fits: the gather that recomputes rows adds dense tiles in another order
    ws = torch.empty(P.plic_curvature_workspace_bytes_ex(N, N, N, neighbours) + cells * 432, dtype=torch.uint8, device="cuda")
    P.plic_curvature_ex_f32(sp, ks, *o, ws)
    P.plic_curvature_backward_ex_f32(sp, sg, gs, *o, ws)
    assert torch.count_nonzero(ks) > 500 and torch.count_nonzero(gs) > 1000

    Z, Y, X = BIG
    bp, bg = embed(sp, torch.zeros(BIG, device="cuda")), embed(sg, torch.randn(BIG, device="cuda"))
    ws = torch.empty(P.plic_curvature_workspace_bytes_ex(X, Y, Z, neighbours), dtype=torch.uint8, device="cuda")
    out = torch.full(BIG, float("nan"), device="cuda")
    P.plic_curvature_ex_f32(bp, out, *o, ws)
    torch.cuda.synchronize()
    print("forward", flush=True)
    check(out, ks, "kappa")
    P.plic_curvature_backward_reuse_f32(bp, bg, out.fill_(float("nan")), *o, ws)
    check(out, gs, "reusing backward")
    P.plic_curvature_backward_ex_f32(bp, bg, out.fill_(float("nan")), *o, ws)
    check(out, gs, "backward")
    assert P.plic_curvature_status(ws, X, Y, Z, neighbours)[:2] == (0, 2 * cells)
