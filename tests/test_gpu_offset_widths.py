"""Two problems per thread (float batches up to 4 or 8 million) and four (more):
a batch beyond the line equals its two halves, bit for bit, forward and
backward, whole and not whole last blocks."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solver,precision", [("sz", "fp32"), ("analytic", "mixed"), ("newton", "fp64")])
@pytest.mark.parametrize("layout,count", [("rows", 8_000_003), ("arrays", 4_000_003), ("arrays", 8_000_768)])
def test_large_batch_equals_its_halves(layout, count, solver, precision):
    import paper_2006_12838_amd as P

    g = torch.Generator(device="cuda").manual_seed(count)
    n = torch.randn((count, 3), generator=g, device="cuda")
    V0, up = (torch.rand((count,), generator=g, device="cuda") for _ in range(2))
    parts = [c.contiguous() for c in n.unbind(-1)]

    def run(lo, hi):
        v, w = V0[lo:hi], up[lo:hi]
        d0 = torch.empty_like(v)
        if layout == "rows":
            r, keep, gn, gv = n[lo:hi], torch.empty_like(n[lo:hi]), torch.empty_like(n[lo:hi]), torch.empty_like(v)
            P.plic_offset_rows_f32(r, v, d0, keep, solver, precision)
            P.plic_offset_backward_rows_f32(keep, v, w, gn, gv, solver, precision)
            return d0, keep, gn, gv
        xs = [c[lo:hi] for c in parts]
        out = [torch.empty_like(v) for _ in range(4)]
        P.plic_offset_f32(*xs, v, d0, solver, precision)
        P.plic_offset_backward_f32(*xs, v, w, *out, solver, precision)
        return d0, *out

    half = count // 2 // 4 * 4                      # the halves' arrays stay 16-byte aligned
    for whole, a, b in zip(run(0, count), run(0, half), run(half, count)):
        assert torch.allclose(whole, torch.cat([a, b]), rtol=0, atol=0, equal_nan=True)
        assert torch.isfinite(whole).float().mean() > 0.99
