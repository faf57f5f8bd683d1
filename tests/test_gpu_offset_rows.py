"""Normals as rows (one (..., 3) tensor): offset, volume and backward through
the row kernels against the FP64 oracle at the sizes where the blocks and the
row staging can go wrong (a wavefront's 3 KiB of rows, a last block that is not
whole, unaligned pointers), and through the public functions against the path
of three separate components.  Tolerances as for those: |d0 - oracle| <= 1e-5 /
1e-12, |V0 - oracle| <= 1e-6 / 1e-14, dd0/dV0 relative 1e-5 / 1e-9, centroid
2e-5 / 1e-11 times the largest upstream gradient."""
import numpy as np
import pytest
import torch

import workloads
from tests.gpu_util import dev, host, max_abs_err

pytestmark = pytest.mark.gpu

KINDS = {"f32": (np.float32, torch.float32, 1e-5, 1e-6, 1e-5, 2e-5),
         "f64": (np.float64, torch.float64, 1e-12, 1e-14, 1e-9, 1e-11)}


@pytest.fixture(scope="module")
def P():
    import paper_2006_12838_amd as P
    return P


def problems(count, dtype, seed):
    nx, ny, nz, V0 = workloads.plic_problems(count, seed=seed, edge_frac=0.0, dtype=dtype)
    V0 = (0.01 + 0.98 * V0.astype(np.float64)).astype(dtype)
    return np.ascontiguousarray(np.stack([nx, ny, nz], 1)), V0


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("count", [1, 63, 256, 511, 512, 1024, 1025, 2048, 2050, 70_003, 300_007])
def test_rows_match_oracle(P, orc, kind, shift, count):
    npdt, dt, tol_d, tol_v, tol_dv, tol_c = KINDS[kind]
    n, V0 = problems(count, npdt, seed=count)
    gd = workloads.upstream_grad(count, seed=count + 1, dtype=npdt)
    place = lambda a: torch.cat([dev(a).new_zeros(shift), dev(a).reshape(-1)])[shift:]   # noqa: E731
    tn, tv, tg = place(n), place(V0), place(gd)
    new = lambda m: torch.full((m + shift + 8,), 7.0, dtype=dt, device="cuda")[shift:]   # noqa: E731
    d0, copy, back, gn, gv = new(count), new(3 * count), new(count), new(3 * count), new(count)
    more = {} if kind == "f64" else {"precision": "mixed"}
    f = {k: getattr(P, f"plic_{k}_{kind}") for k in ("offset_rows", "volume_rows", "offset_backward_rows")}
    f["offset_rows"](tn, tv, d0[:count], copy[:3 * count], solver="sz", **more)
    f["volume_rows"](tn, d0[:count], back[:count])
    f["offset_backward_rows"](tn, tv, tg, gn[:3 * count], gv[:count], solver="sz", **more)
    for t, m in ((d0, count), (copy, 3 * count), (back, count), (gn, 3 * count), (gv, count)):
        assert (t[m:] == 7.0).all()                       # nothing past the end
    ref, dv, gx, gy, gz = orc.offset_grad(n[:, 0], n[:, 1], n[:, 2], V0)
    assert torch.equal(copy[:3 * count], tn)
    assert max_abs_err(host(d0[:count]), ref) <= tol_d
    vref = orc.volume(n[:, 0], n[:, 1], n[:, 2], host(d0[:count]))
    assert max_abs_err(host(back[:count]), vref) <= tol_v
    g = gd.astype(np.float64)
    assert np.max(np.abs(host(gv[:count]) - g * dv) / np.abs(g * dv)) <= tol_dv
    want = g[:, None] * np.stack([gx, gy, gz], 1)
    assert np.max(np.abs(host(gn[:3 * count]).reshape(-1, 3) - want)) <= tol_c * max(1.0, np.abs(g).max())


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("form", ["rows", "columns", "broadcast", "shaped"])
def test_public_functions_over_forms(P, kind, form):
    """Every form of the normals gives the results of three separate arrays."""
    npdt, dt, tol_d, tol_v, _, tol_c = KINDS[kind]
    n, V0 = problems(6000, npdt, seed=3)
    if form == "broadcast":
        n = n[:1]
    tn, tv = dev(n), dev(V0)
    if form == "columns":
        tn = tn.t().contiguous().t()                      # (m, 3), the columns contiguous
    if form == "shaped":
        tn, tv = tn.reshape(10, 20, 30, 3), tv.reshape(10, 20, 30)
    tn.requires_grad_(True)
    tv.requires_grad_(True)
    w = dev(workloads.upstream_grad(tuple(tv.shape), seed=4, dtype=npdt))
    parts = [tn.detach()[..., k].expand(tv.shape).contiguous().requires_grad_(True) for k in range(3)]
    tv2 = tv.detach().clone().requires_grad_(True)
    a, b = P.offset(tn, tv), P.offset(tuple(parts), tv2)
    assert a.shape == b.shape == tv.shape and (a - b).abs().max() <= tol_d
    assert (P.volume(tn, a) - P.volume(tuple(parts), b)).abs().max() <= 2 * tol_v
    ga, gv = torch.autograd.grad(a, (tn, tv), w)
    gb = torch.autograd.grad(b, (*parts, tv2), w)
    want = torch.stack(gb[:3], -1)
    if form == "broadcast":
        want = want.sum(0, keepdim=True)
    assert ga.shape == tn.shape
    assert (ga - want).abs().max() <= tol_c * (1 if form != "broadcast" else 6000)
    assert ((gv - gb[3]).abs() <= KINDS[kind][4] * gb[3].abs()).all()


def test_normals_may_change_before_the_backward(P):
    """The gradient is that of the normals the forward saw."""
    n, V0 = problems(5000, np.float32, seed=5)
    tn, tv = dev(n), dev(V0).requires_grad_(True)
    want, = torch.autograd.grad(P.offset(tn, tv).sum(), tv)
    d0 = P.offset(tn, tv)
    tn.zero_()
    got, = torch.autograd.grad(d0.sum(), tv)
    assert torch.equal(got, want)
