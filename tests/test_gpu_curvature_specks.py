"""Lattices of specks, whose fits are ill-conditioned or of few points in most
cells: on 16 lanes (few work items) such a cell forms its sums again in the same
call, on 4 lanes (many) it is done again on 16; the same bits."""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("neighbours", [False, True])
@pytest.mark.parametrize("solver,precision", [("sz", "fp32"), ("analytic", "mixed"), ("newton", "fp64")])
@pytest.mark.parametrize("share,shape", [(0.2, (20, 20, 64)), (0.9, (12, 12, 64))])
def test_few_cells_equal_many(share, shape, solver, precision, neighbours):
    import paper_2006_12838_amd as P

    rng = np.random.default_rng(7)
    a = np.where(rng.random(shape) < share, rng.random(shape), rng.random(shape) < 0.5).astype(np.float32)
    a[:, :, [0, 1, -2, -1]] = 0.0
    w = rng.standard_normal(shape).astype(np.float32)
    cells = int(((a > 0) & (a < 1))[1:-1, 1:-1].sum())
    copies = 6
    assert cells < 900 * 8 and copies * cells > 2560 * 8      # the lines lie at 900 to 2560 items of 8 cells
    res = []
    for n in (1, copies):
        phi, up = (dev(np.concatenate([x] * n, axis=2)) for x in (a, w))
        kappa, g = torch.empty_like(phi), torch.empty_like(phi)
        size = P.plic_curvature_workspace_bytes_ex(*phi.shape[::-1], neighbours) + phi.numel() * 4 * 111
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        P.plic_curvature_ex_f32(phi, kappa, solver, precision, "py", neighbours, ws)
        P.plic_curvature_backward_ex_f32(phi, up, g, solver, precision, "py", neighbours, ws)
        res.append((kappa, g))
    assert all(x.nan_to_num().abs().max() > 0 for x in res[0])
    for want, got in zip(*res):
        for c in range(copies):
            assert torch.allclose(want[:, :, 3:-3], got[:, :, 64 * c + 3:64 * c + 61], rtol=0, atol=0, equal_nan=True), c
