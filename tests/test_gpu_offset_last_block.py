"""Forward offsets of FP64 arithmetic on float arrays, whose last blocks take
ways of their own: a batch equals its pieces of a million problems (which go
two to a thread), bit for bit, for every remainder of a block, and nothing is
written past the end."""
import pytest
import torch

pytestmark = pytest.mark.gpu

PIECE = 1_000_000


def batch(count, shift=0):
    g = torch.Generator(device="cuda").manual_seed(count + shift)
    n = torch.randn((3 * count + shift,), generator=g, device="cuda")[shift:]
    V0 = torch.rand((count + shift,), generator=g, device="cuda")[shift:]
    V0[::97] = 0.0
    V0[::101] = 1.0
    return n, V0


def offsets(P, layout, n, V0, solver, d0=None):
    """d0, and the copy of n that rows leave, each with 8 more elements that stay 7"""
    shift = (V0.data_ptr() // 4) % 4
    new = lambda m: torch.full((m + shift + 8,), 7.0, device="cuda")[shift:]     # noqa: E731
    m = V0.numel()
    out, copy = new(m) if d0 is None else d0, new(3 * m)
    if layout == "rows":
        P.plic_offset_rows_f32(n, V0, out[:m], copy[:3 * m], solver, "fp64")
    else:
        c = n.view(m, 3).t()
        parts = [torch.cat([c.new_zeros(shift), c[k]])[shift:] for k in range(3)]
        P.plic_offset_f32(*parts, V0, out[:m], solver, "fp64")
    return out, copy


def check(P, layout, n, V0, solver):
    out, copy = offsets(P, layout, n, V0, solver)
    m = V0.numel()
    for a in range(0, m, PIECE):
        b = min(m, a + PIECE)
        want, _ = offsets(P, layout, n[3 * a:3 * b].clone(), V0[a:b].clone(), solver)
        assert torch.equal(out[a:b], want[:b - a]), (a, b)
    assert torch.isfinite(out).all() and (out[m:] == 7.0).all() and out.numel() == m + 8
    if layout == "rows":
        assert torch.equal(copy[:3 * m], n) and (copy[3 * m:] == 7.0).all()


@pytest.mark.parametrize("solver", ["sz", "analytic"])
@pytest.mark.parametrize("layout", ["rows", "arrays"])
@pytest.mark.parametrize("rest", [0, 1, 255, 256, 257, 1023])
def test_four_to_a_thread(layout, rest, solver):
    import paper_2006_12838_amd as P
    check(P, layout, *batch(8_000_512 + rest), solver)


@pytest.mark.parametrize("solver", ["sz", "analytic", "newton", "nested", "sz_kawano"])
@pytest.mark.parametrize("layout", ["rows", "arrays"])
@pytest.mark.parametrize("count", [1, 63, 255, 256, 257, 70_001])
def test_unaligned(layout, count, solver):
    import paper_2006_12838_amd as P
    n, V0 = batch(count, shift=1)
    if solver == "sz_kawano":                     # NaN for some fill levels of 0 and 1
        V0.clamp_(0.01, 0.99)
    check(P, layout, n, V0, solver)
    want, _ = offsets(P, layout, n, V0, solver)
    m = V0.numel()
    own = torch.cat([V0.new_zeros(1), V0, V0.new_full((8,), 7.0)])[1:]
    got, _ = offsets(P, layout, n, own[:m], solver, d0=own)          # d0 is V0
    assert torch.equal(got, want)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("count", [1, 3, 4, 5, 1021, 1023, 1024, 1025, 1027, 5003])
def test_volume_of_arrays(count, precision):
    """aligned arrays (four problems a thread) and the same unaligned (one)"""
    import paper_2006_12838_amd as P

    g = torch.Generator(device="cuda").manual_seed(count)
    n = [torch.randn(count, generator=g, device="cuda") for _ in range(3)]
    d0 = torch.rand(count, generator=g, device="cuda") * 2.0 - 1.0
    res = []
    for shift in (0, 1):
        a = [torch.cat([t.new_zeros(shift), t])[shift:] for t in (*n, d0)]
        out = torch.full((count + shift + 8,), 7.0, device="cuda")[shift:]
        P.plic_volume_f32(*a, out[:count], precision)
        assert (out[count:] == 7.0).all()
        res.append(out[:count])
    assert torch.equal(*res) and (res[0] >= 0).all() and (res[0] <= 1).all()
