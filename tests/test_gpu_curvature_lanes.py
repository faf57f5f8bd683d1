"""Interface cells on 16 lanes (few work items on the lattice) and on 4 lanes
(many): the same bits.  A drop with specks (fits that are ill-conditioned, of
few points, without a normal) alone and among copies of itself, forward and
backward."""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev
import workloads

pytestmark = pytest.mark.gpu


def drop(seed):
    phi, _ = workloads.sphere_lattice(N=40, R=11.0, seed=seed)
    rng = np.random.default_rng(seed)
    a = np.zeros((40, 40, 64), np.float32)
    a[:, :, 12:52] = np.asarray(phi).reshape(40, 40, 40)
    speck = rng.random(a.shape) < 0.02
    speck[[0, -1]] = speck[:, [0, -1]] = speck[:, :, [0, 1, -2, -1]] = False
    return np.where(speck, rng.random(a.shape).astype(np.float32), a)


@pytest.mark.parametrize("neighbours", [False, True])
@pytest.mark.parametrize("solver,precision,normal", [("sz", "fp32", "py"), ("analytic", "mixed", "cm"),
                                                     ("nested", "mixed", "py"), ("newton", "fp64", "py")])
def test_few_cells_equal_many(solver, precision, normal, neighbours):
    import paper_2006_12838_amd as P

    one = drop(3)
    copies = 12                                   # about 500 work items a copy; the line lies at 1024 or 2048
    w = np.random.default_rng(5).standard_normal(one.shape).astype(np.float32)
    res = []
    for n in (1, 2, 3, copies):
        phi, up = (dev(np.concatenate([a] * n, axis=2)) for a in (one, w))
        kappa, g = torch.empty_like(phi), torch.empty_like(phi)
        # room for every row: the gather that recomputes rows adds in another order in crowded tiles
        size = P.plic_curvature_workspace_bytes_ex(*phi.shape[::-1], neighbours) + phi.numel() * 4 * 111
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        P.plic_curvature_ex_f32(phi, kappa, solver, precision, normal, neighbours, ws)
        P.plic_curvature_backward_ex_f32(phi, up, g, solver, precision, normal, neighbours, ws)
        res.append((n, kappa, g))
    _, k1, g1 = res[0]
    assert k1.nan_to_num().abs().max() > 0 and g1.nan_to_num().abs().max() > 0
    for n, k, g in res[1:]:
        for c in range(n):
            for want, got in ((k1, k), (g1, g)):
                assert torch.allclose(want[:, :, 2:-2], got[:, :, 64 * c + 2:64 * c + 62], rtol=0, atol=0,
                                      equal_nan=True), (n, c)
